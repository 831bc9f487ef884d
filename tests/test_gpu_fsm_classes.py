"""The per-cell transform path on grids that take each of its kernels (tiles per wave, k-steps, guards),
with odd and even angle counts (directions that are their own mirror image), every slab width, few cells
(terms split over workgroups) and many: against the assembled operator, which the other tests pin to the
oracle.  Both sum about 10^4 products per unknown in float64: 1e-12 of the largest value, the bound of the
other transform tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1612_04488_amd import sis

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def compare(p, cells, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    h = torch.randn((cells, p.n_dof), dtype=torch.float64, device=DEV, generator=g)
    delta = torch.rand(cells, dtype=torch.float64, device=DEV, generator=g) + 0.5
    a, b = torch.full_like(h, np.nan), torch.full_like(h, np.nan)
    p.collide_fsm(h, delta, a)
    p.collide(h, delta, b)
    err = ((a - b).abs().max() / b.abs().max()).item()
    assert err < 1e-12, err


@pytest.mark.parametrize("n,n_pad,m,parity", [(4, 8, 1, 2), (6, 12, 2, 0), (10, 26, 3, 1), (18, 36, 4, 2), (20, 42, 2, 1),
                                              (22, 44, 5, 2), (24, 48, 3, 1), (26, 52, 2, 2), (28, 54, 3, 2), (30, 60, 2, 2),
                                              (32, 64, 2, 2), (34, 64, 3, 2), (36, 64, 2, 2)])
def test_transforms_match_the_operator(n, n_pad, m, parity):
    p = sis.Plan(n, 5.0, n_pad=n_pad, m_angle=m, parity=parity)
    for cells in (1, 3, 150):
        compare(p, cells, n + cells)


@pytest.mark.parametrize("n,n_pad,parity", [(12, 24, 1), (24, 48, 2), (30, 64, 2), (36, 64, 2)])
def test_every_slab_width(n, n_pad, parity):
    p = sis.Plan(n, 5.0, n_pad=n_pad, m_angle=2, parity=parity)
    for slab in range(1, 9):
        p.set_fsm_slab(slab)
        assert p.fsm_info()["slab_l1"] == slab
        compare(p, 5, slab)


def test_many_cells_of_the_smallest_grid():
    """4^3 velocities in eight classes: 2 200 000 cells are more threads than a launch takes (2^32), although
    their rows and sums are within the 2 GiB of a chunk."""
    p = sis.Plan(4, 5.0, n_pad=8, m_angle=2)
    nc = 2_200_000
    g = torch.Generator(device=DEV).manual_seed(4)
    h = torch.randn((nc, p.n_dof), dtype=torch.float64, device=DEV, generator=g)
    delta = torch.rand(nc, dtype=torch.float64, device=DEV, generator=g) + 0.5
    out = torch.full_like(h, np.nan)
    p.collide_fsm(h, delta, out)
    assert bool(torch.isfinite(out).all())
    at = torch.tensor([0, 65_534, 65_535, 65_536, 131_069, 131_070, 2_097_151, 2_097_152, nc - 1], device=DEV)
    ref = torch.empty((len(at), p.n_dof), dtype=torch.float64, device=DEV)
    p.collide(h[at].contiguous(), delta[at].contiguous(), ref)
    assert (out[at] - ref).abs().max() <= 1e-12 * ref.abs().max()
