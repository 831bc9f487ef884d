"""The finish step with more threads a row (no more rows than compute units) against the same rows in
a larger batch, every class count: the right sides and L element by element are the same
arithmetic; the moments and the projection's coefficients are sums in another order."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1612_04488_amd import sis

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("parity", [0, 1, 2])
@pytest.mark.parametrize("project", [False, True])
def test_few_rows_equal_many(parity, project):
    p = sis.Plan(18, 5.0, m_angle=2, parity=parity)      # 729 orbits a class: an odd count, no pairs at parity 1
    few, many = 256, 257
    g = torch.Generator(device=DEV).manual_seed(parity)
    rnd = lambda *s: torch.randn(s, dtype=torch.float64, device=DEV, generator=g)
    h, dU = rnd(many, p.n_dof), rnd(many)
    delta = torch.rand(many, dtype=torch.float64, device=DEV, generator=g) + 0.5
    flow = (torch.arange(many, device=DEV) % 3).to(torch.int32)
    out = {}
    for nc in (few, many):
        p.set_contraction_config(nc, 128, 16, 2)
        r = [torch.full((nc, p.n_dof), np.nan, dtype=torch.float64, device=DEV) for _ in range(2)]
        am = torch.full((nc, 4), np.nan, dtype=torch.float64, device=DEV)
        p.collide(h[:nc], delta[:nc], r[0], dU=dU[:nc], flow=flow[:nc], project=project, lh_out=r[1], amom_out=am)
        out[nc] = (*r, am)
    for k in range(2):
        a, b = out[few][k], out[many][k][:few]
        if not project:
            assert torch.equal(a, b), k
        else:                                            # five sums of n_dof terms in another order
            assert (a - b).abs().max() <= 1e-12 * b.abs().max(), k
    a, b = out[few][2], out[many][2][:few]
    assert (a - b).abs().max() <= 1e-12 * b.abs().max()


@pytest.mark.parametrize("n,parity,splits", [(16, 2, 8), (16, 2, 11), (12, 1, 9), (12, 0, 3)])
def test_many_splits_of_few_rows(n, parity, splits):
    """Few short rows load more splits at once: the same sums in the same order as in a larger batch."""
    p = sis.Plan(n, 5.0, m_angle=2, parity=parity)
    few, many = 17, 300
    g = torch.Generator(device=DEV).manual_seed(splits)
    h = torch.randn((many, p.n_dof), dtype=torch.float64, device=DEV, generator=g)
    delta = torch.rand(many, dtype=torch.float64, device=DEV, generator=g) + 0.5
    out = {}
    for nc in (few, many):
        p.set_contraction_config(nc, 128, 16, splits)
        r = torch.full((nc, p.n_dof), np.nan, dtype=torch.float64, device=DEV)
        am = torch.full((nc, 4), np.nan, dtype=torch.float64, device=DEV)
        p.collide(h[:nc], delta[:nc], r, amom_out=am)
        out[nc] = (r, am)
    assert torch.equal(out[few][0], out[many][0][:few])
    assert torch.equal(out[few][1], out[many][1][:few])


@pytest.mark.parametrize("n,parity", [(20, 2), (18, 2), (24, 2), (20, 0), (22, 0), (10, 1), (18, 1)])
@pytest.mark.parametrize("splits", [1, 2, 3, 4, 6, 8])
def test_rows_and_splits_at_the_forms_limits(n, parity, splits):
    """500 pairs, 729 orbits and 864 pairs of two classes, 1000 and 1331 orbits of eight (256 threads below, 1024
    above), 125 and 729 of four (512), and split counts of one round or less with more splits at once: the same
    sums in the same order as in a larger batch, element by element."""
    p = sis.Plan(n, 5.0, m_angle=2, parity=parity)
    few, many = 5, 300
    g = torch.Generator(device=DEV).manual_seed(splits)
    h = torch.randn((many, p.n_dof), dtype=torch.float64, device=DEV, generator=g)
    delta = torch.rand(many, dtype=torch.float64, device=DEV, generator=g) + 0.5
    out = {}
    for nc in (few, many):
        p.set_contraction_config(nc, 128, 16, splits)
        r = torch.full((nc, p.n_dof), np.nan, dtype=torch.float64, device=DEV)
        am = torch.full((nc, 4), np.nan, dtype=torch.float64, device=DEV)
        p.collide(h[:nc], delta[:nc], r, amom_out=am)
        out[nc] = (r, am)
    assert torch.equal(out[few][0], out[many][0][:few])
    assert (out[few][1] - out[many][1][:few]).abs().max() <= 1e-12 * out[many][1].abs().max()
