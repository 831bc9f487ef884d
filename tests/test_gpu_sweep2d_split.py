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
    if kind == "two waves":
        return [(faces(8), faces(20), None), (faces(11), faces(17), None)]
    if kind == "five waves":
        return [(faces(7), faces(70), None)]
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


@pytest.mark.parametrize("species,n1,n2", [(1, 47, 44), (1, 46, 45), (2, 50, 43), (2, 9, 5)])
def test_moments_of_the_swept_cells(species, n1, n2):
    """2068, 2070, 2150 cells and 45, short rows (one cell a workgroup): sums of n^3 terms in any order, against
    the sums of their magnitudes."""
    n, l_v = 6, 4.0
    mix = dict(masses=(1.0, 2.0), diameters=(1.0, 0.8), chi=(0.4, 0.6), m_rho=3) if species == 2 else None
    p = sis.Plan(n, l_v, m_angle=2, mixture=mix)
    geom = sis.Geometry2D(p, "duct", [(faces(n1), faces(n2), None)], [0.7], [1])
    nc = n1 * n2
    g = torch.Generator(device=DEV).manual_seed(n2)
    rhs = torch.randn((nc, p.n_dof), dtype=torch.float64, device=DEV, generator=g)
    h, mom = torch.zeros_like(rhs), torch.full((nc, species, 8), np.nan, dtype=torch.float64, device=DEV)
    sis.transport_sweep(p, geom, rhs, h, mom)
    torch.cuda.synchronize()
    vg = VelocityGrid(n, l_v)
    v1, v2, v3 = (np.broadcast_to(a, (n, n, n)) for a in (vg.V1, vg.V2, vg.V3))
    h, mom = h.cpu().numpy().reshape(nc, species, n, n, n), mom.cpu().numpy().reshape(nc, species, 8)
    for s in range(species):
        ms = (1.0, 2.0)[s]
        f = [v3, (ms * (v1 ** 2 + v2 ** 2 + v3 ** 2) - 2.5) * v3, v3 * (2 * v1 ** 2 - 1), 2 * v1 * v2 * v3,
             v3 * (2 * v2 ** 2 - 1), 2 * ms * v1 * v3, 2 * ms * v2 * v3]
        for k, fk in enumerate(f):
            ref = np.array([vg.integrate(fk * x) for x in h[:, s]])
            size = np.array([vg.integrate(np.abs(fk * x)) for x in h[:, s]])
            assert np.all(np.abs(mom[:, s, k] - ref) <= (n ** 3 + 16) * np.finfo(float).eps * size), (s, k)


@pytest.mark.parametrize("n,parity,species,n1,n2", [(24, 1, 1, 77, 47), (24, 1, 1, 47, 76), (16, 0, 1, 74, 109), (16, 0, 2, 37, 109),
                                                    (16, 0, 1, 74, 108)])
def test_moments_of_long_rows(n, parity, species, n1, n2):
    """Rows of 6912 and 4096 values at the size from which four cells share a workgroup: 3619 cells (three left over),
    3572 (one cell a workgroup); 8066 (two left over), 4033 of two species (one left over), 7992 (one a workgroup)."""
    l_v = 5.0
    mix = dict(masses=(1.0, 2.0), diameters=(1.0, 0.8), chi=(0.4, 0.6), m_rho=3) if species == 2 else None
    p = sis.Plan(n, l_v, m_angle=2, parity=parity, mixture=mix)
    geom = sis.Geometry2D(p, "duct", [(faces(n1), faces(n2), None)], [0.7], [1])
    nc, n3 = n1 * n2, p.n_dof // species
    g = torch.Generator(device=DEV).manual_seed(n2)
    rhs = torch.randn((nc, p.n_dof), dtype=torch.float64, device=DEV, generator=g)
    h, mom = torch.zeros_like(rhs), torch.full((nc, species, 8), np.nan, dtype=torch.float64, device=DEV)
    sis.transport_sweep(p, geom, rhs, h, mom)
    torch.cuda.synchronize()
    vg = VelocityGrid(n, l_v)
    v1, v2, v3 = (np.broadcast_to(a, (n, n, n)).astype(float)[:, :, n // 2 if parity else 0:].reshape(-1) for a in (vg.V1, vg.V2, vg.V3))
    w = (2 * l_v / n) ** 3 * (2 if parity else 1)
    h, mom = h.cpu().numpy().reshape(nc, species, n3), mom.cpu().numpy().reshape(nc, species, 8)
    for s in range(species):
        ms = (1.0, 2.0)[s]
        f = w * np.stack([v3, (ms * (v1 ** 2 + v2 ** 2 + v3 ** 2) - 2.5) * v3, v3 * (2 * v1 ** 2 - 1), 2 * v1 * v2 * v3,
                          v3 * (2 * v2 ** 2 - 1), 2 * ms * v1 * v3, 2 * ms * v2 * v3], 1)
        ref, size = h[:, s] @ f, np.abs(h[:, s]) @ np.abs(f)
        assert np.all(np.abs(mom[:, s, :7] - ref) <= (n3 + 16) * np.finfo(float).eps * size), s


@pytest.mark.parametrize("kind,copies", [("two waves", 16), ("two waves", 17), ("five waves", 32), ("five waves", 33)])
def test_sweep_forms_at_the_widths_limits(kind, copies):
    """The last batch that goes by lanes and the first that goes by rows, for workgroups of two and of five waves
    (8^3 velocities: 8 groups of quadruples a case)."""
    test_sweep_forms(kind, copies)
