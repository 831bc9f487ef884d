"""The two row-blocked forms of the 2-D sweep (few cases: 16 velocity quadruples by 16 columns a
wave; many: 64 quadruples a wave) at the edges of their columns and rows, with mirror ghosts
(ducts) and with periodic wraps and solids, against the oracle's sweep; then the velocity
equation's right sides over several workgroups through a solve.

The recurrence is the oracle's up to the rounding of a few operations a cell; 1e-12 of the
largest value is what the other tests of the sweep hold at up to 128 cells a side."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import collision, duct
from oracle.velocity import VelocityGrid
from paper_1612_04488_amd import inputs, sis

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def rel(a, b):
    return float(np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300))


def faces(n, length=0.5):
    return inputs.duct_faces(n, length)


def cross_sections(kind):
    if kind == "duct":      # 33 columns: three waves, the last group of one column
        return [(faces(12), faces(10, 1.0), None), (faces(9), faces(3, 0.25), None), (faces(7), faces(33), None),
                (faces(5), faces(17), None)]
    if kind == "wide":      # 65 and 112 columns: five and seven waves
        return [(faces(6), faces(65), None), (faces(9), faces(112), None)]
    out = []
    for n1, n2 in ((18, 20), (16, 16), (23, 31)):
        mask = np.zeros((n1, n2), bool)
        mask[3:6, 4:9] = mask[n1 - 4:, 8:10] = mask[8, n2 - 3:] = True
        out.append((np.linspace(0.0, 1.0, n1 + 1), np.linspace(0.0, 1.0, n2 + 1), mask))
    return out


@pytest.mark.parametrize("kind,copies", [("duct", 1), ("duct", 30), ("wide", 1), ("wide", 20), ("periodic", 1),
                                         ("periodic", 12)])
def test_sweep_forms(kind, copies):
    print("sweep2d", kind, copies, flush=True)
    n_v, l_v, m = 8, 4.0, 3
    p = sis.Plan(n_v, l_v, m_angle=m)
    f = collision.FSM(VelocityGrid(n_v, l_v), m_angle=m)
    geo = "periodic" if kind == "periodic" else "duct"
    base = cross_sections(kind)
    deltas = [3.0, 0.0, 0.5, 8.0][:len(base)]
    geom = sis.Geometry2D(p, geo, base * copies, deltas * copies, [1] * (len(base) * copies))
    assert geom.sweep_form() == 1
    edges = (duct.WALL, duct.SYM, duct.WALL, duct.SYM) if geo == "duct" else (duct.PERIODIC,) * 4
    grids = [duct.Grid2D(a, b, edges, mask) for a, b, mask in base]
    nc = sum(len(g.cells) for g in grids)
    assert geom.n_cells == nc * copies
    rhs = inputs.smooth_h(n_v, l_v, nc, seed=5) + 0.1 * inputs.rough_h(n_v, l_v, nc, seed=3)
    prev = inputs.rough_h(n_v, l_v, nc, seed=9)
    dev = lambda x: torch.tensor(x.reshape(nc, -1), dtype=torch.float64, device=DEV).repeat(copies, 1)
    h, mom = dev(prev), torch.empty((nc * copies, 8), dtype=torch.float64, device=DEV)
    sis.transport_sweep(p, geom, dev(rhs), h, mom)
    torch.cuda.synchronize()
    h = h.cpu().numpy().reshape(copies, nc, -1)
    assert all(np.array_equal(h[0], h[c]) for c in range(copies))
    o = 0
    for c, g in enumerate(grids):
        s = slice(o, o + len(g.cells))
        o += len(g.cells)
        ref = duct.sweep_2d(rhs[s], deltas[c] * f.nu, g, f.grid, prev[s])
        assert rel(h[0, s], ref.reshape(len(g.cells), -1)) < 1e-12, c
