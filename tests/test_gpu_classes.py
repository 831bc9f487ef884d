"""The contraction on reflection classes: collide against the plan's own matrix applied in
float64, where the index arithmetic can go wrong -- grids with an odd number of orbits along the
third axis (no 16-byte pairs, an odd class row), the smallest grid, every parity storage, two
species, the polar grid, tiles that read class rows and the few-cell tile that reads the cells'
rows, split-K;
then the workspace rules: capture before any eager call, a captured buffer that a larger batch
would replace, and the fixed-workspace call over several passes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1612_04488_amd import sis

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EPS = np.finfo(np.float64).eps
MIX = dict(masses=(1.0, 2.0), diameters=(1.0, 0.8), chi=(0.4, 0.6), m_rho=3)


def make(grid):
    kind, n, parity = grid
    if kind == "polar":
        return sis.Plan(0, 2.0, m_angle=2, polar=dict(n_vr=3, vr_max=2.0, n_th=n, n_vz=4))
    return sis.Plan(n, 4.0, m_angle=2, parity=parity, mixture=MIX if kind == "mix" else None)


def inputs(p, nc, seed=1):
    g = torch.Generator(device=DEV).manual_seed(seed)
    h = torch.randn((nc, p.n_dof), dtype=torch.float64, device=DEV, generator=g)
    return h, torch.rand(nc, dtype=torch.float64, device=DEV, generator=g) + 0.5


def bound(op, h, delta, unit):
    """Rounding of a sum of K products in any order and grouping, each operand of which was itself
    summed over at most 8 images: (K + 32) units of sum |K| |h| over the reflected images.  The
    matrix commutes with the reflections only to rounding, K eps of its largest entry per row."""
    K = op.shape[1]
    big = np.abs(op).max(axis=1)
    return delta[:, None] * (K + 32) * unit * (np.abs(h).sum(axis=1)[:, None] * big[None, :])


def check(p, op, h, delta, rhs, unit=EPS, cells=None):
    hn, dn, out = (t.cpu().numpy() for t in (h, delta, rhs))
    ref = dn[:, None] * (hn @ op.T)
    assert np.all(np.isfinite(out))
    assert np.all(np.abs(out - ref) <= bound(op, hn, dn, unit))


@pytest.mark.parametrize("grid", [("one", 4, 0), ("one", 4, 2), ("one", 6, 0), ("one", 6, 1), ("one", 6, 2), ("one", 8, 0),
                                  ("one", 10, 1), ("mix", 6, 2), ("mix", 8, 1), ("mix", 4, 0), ("polar", 6, 0), ("polar", 4, 0)],
                         ids=str)
def test_collide_on_classes_is_the_matrix(grid):
    p = make(grid)
    op = p.tables(operator=True)["op"]
    for nc in (1, 33, 300):
        h, delta = inputs(p, nc)
        rhs = torch.full_like(h, np.nan)
        p.collide(h, delta, rhs)                       # tuned
        check(p, op, h, delta, rhs)
    for k, (rows, depth) in enumerate([(128, 16), (64, 16), (32, 16), (128, 32), (64, 32)]):
        for splits in (1, 3):
            nc = 129 + 2 * k + splits
            h, delta = inputs(p, nc, seed=k)
            p.set_contraction_config(nc, rows, depth, splits)
            rhs = torch.full_like(h, np.nan)
            p.collide(h, delta, rhs)
            check(p, op, h, delta, rhs)


@pytest.mark.parametrize("grid", [("one", 4, 0), ("one", 8, 0), ("one", 8, 1), ("one", 12, 2), ("mix", 8, 2), ("polar", 6, 0)],
                         ids=str)
def test_low_precision_on_classes(grid):
    p = make(grid)
    op = p.tables(operator=True)["op"]
    h, delta = inputs(p, 37)
    for precision, unit in (("fp32", 2.0 ** -23), ("bf16x3", 2.0 ** -15), ("bf16", 2.0 ** -7)):
        if precision == "bf16" and grid[0] == "mix":
            continue
        p.set_precision(precision)
        outs = []
        for rows in (128, 64, 32):
            p.set_contraction_config(37, rows, 16 if precision == "fp32" else 64, 1, precision=precision)
            rhs = torch.full_like(h, np.nan)
            p.collide(h, delta, rhs)
            check(p, op, h, delta, rhs, unit=unit)
            outs.append(rhs)
        if precision != "fp32":   # the tile that splits the cells' rows itself agrees to the last bit
            assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    p.set_precision("fp64")


def test_capture_without_workspace_and_growth_after_capture():
    p = make(("one", 8, 1))
    op = p.tables(operator=True)["op"]
    h, delta = inputs(p, 300)
    rhs, rhs2 = torch.empty_like(h), torch.empty_like(h)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    g1, g2 = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(g1, stream=s):               # nothing allocated yet
        p.collide(h, delta, rhs)
    p.collide(h, delta, rhs2)                          # eager: workspace made
    with torch.cuda.graph(g2, stream=s):
        p.collide(h, delta, rhs2)
    big, dbig = inputs(p, 2000, seed=3)
    rbig = torch.empty_like(big)
    for it in range(3):
        p.collide(big, dbig, rbig)                     # replaces the workspace the first time
        check(p, op, big, dbig, rbig)
        h.copy_(inputs(p, 300, seed=10 + it)[0])
        rhs.fill_(np.nan)
        rhs2.fill_(np.nan)
        torch.cuda.synchronize()
        g1.replay()
        g2.replay()
        torch.cuda.synchronize()
        check(p, op, h, delta, rhs)
        check(p, op, h, delta, rhs2)


def test_fixed_workspace_over_several_passes():
    p = make(("one", 8, 0))
    op = p.tables(operator=True)["op"]
    nc = 9001                                          # 2 x 8 bytes x 512 unknowns: 8191 cells fit
    h, delta = inputs(p, nc)
    rhs, am = torch.full_like(h, np.nan), torch.full((nc, 4), np.nan, dtype=torch.float64, device=DEV)
    flow = torch.ones(nc, dtype=torch.int32, device=DEV)
    rhs2, am2 = torch.full_like(h, np.nan), torch.full_like(am, np.nan)
    p.collide_noalloc(h, delta, rhs)
    check(p, op, h, delta, rhs)
    p.collide_noalloc(h, delta, rhs, flow=flow, amom_out=am)
    p.collide(h, delta, rhs2, flow=flow, amom_out=am2)
    d = (am - am2).abs().max().item()
    assert d <= 1e-12 * am2.abs().max().item()
