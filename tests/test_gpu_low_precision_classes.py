"""The low-precision contractions on reflection classes against the plan's own matrix in float64, with a bound per
element that a wrong block, operand layout or sum cannot meet.

With the class sums x_b of a cell and the blocks B_b of the matrix, an output is the signed sum over the classes of
B_b x_b, so the rounding of operands and sums is bounded by E = sum_b |B_b| |x_b| times
  FP32     2 u + K u' (both operands to u = 2^-24, K additions at u' = 2^-23 each),
  3xBF16   3 x 2^-18 (each operand short by 2^-18 after two parts of 2^-9, the product of the low parts left out)
           and 3 K additions,
  BF16     2 x 2^-9 and K additions.
The last lines of the check hold the bound itself to account: against the outputs' own size, a result of zeros and
the result of the next cell fail almost everywhere."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1612_04488_amd import sis

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MIX = dict(masses=(1.0, 2.0), diameters=(1.0, 0.8), chi=(0.4, 0.6), m_rho=3)


def fold(a, axes):
    """Sums over the images along the reflected axes, even and odd: [class][the other axes, halved]."""
    out = [a]
    for ax in axes:
        n = a.shape[ax] // 2
        up, lo = slice(n, None), slice(n - 1, None, -1)
        cut = lambda x, s: x[(slice(None),) * ax + (s,)]
        out = [f(cut(x, up), cut(x, lo)) for f in (np.add, np.subtract) for x in out]
    return np.stack(out)


def blocks_and_rows(op, h, dims, axes, species):
    """B_b [class][K][K] and x_b [class][cells][K] (the matrix is symmetric under the reflections to rounding)."""
    K = species * int(np.prod(dims)) // 2 ** len(axes)
    x = fold(h.reshape((-1, species) + dims), [2 + a for a in axes])
    both = op.reshape((species,) + dims + (species,) + dims)
    B = []
    rows = fold(both, [1 + a for a in axes])                     # [class of the output]
    for b, r in enumerate(rows):
        B.append(fold(r, [2 + len(dims) + a for a in axes])[b])  # the same class of the input
    return np.stack(B).reshape(len(rows), K, K) / 4.0 ** len(axes), x.reshape(len(rows), -1, K)


def make(grid):
    kind, n, parity = grid
    if kind == "polar":
        p = sis.Plan(0, 2.0, m_angle=2, polar=dict(n_vr=4, vr_max=2.0, n_th=n, n_vz=4))
        return p, (4, n, 4), (1,), 1
    p = sis.Plan(n, 4.0, m_angle=2, parity=parity, mixture=MIX if kind == "mix" else None)
    dims = (n, n // 2 if parity == 2 else n, n // 2 if parity else n)
    return p, dims, (0, 1, 2)[:3 - parity], 2 if kind == "mix" else 1


@pytest.mark.parametrize("grid", [("one", 4, 0), ("one", 8, 0), ("one", 8, 1), ("one", 12, 1), ("one", 12, 2), ("mix", 8, 2),
                                  ("mix", 8, 1), ("polar", 6, 0), ("polar", 12, 0)], ids=str)
@pytest.mark.parametrize("precision,operands,products", [("fp32", 2.0 ** -23, 1), ("bf16x3", 3 * 2.0 ** -18, 3), ("bf16", 2.0 ** -8, 1)])
def test_low_precision_holds_its_own_bound(grid, precision, operands, products):
    p, dims, axes, species = make(grid)
    op = p.tables(operator=True)["op"]
    try:
        p.set_precision(precision)
    except sis.SisError as e:
        assert precision == "bf16" and species == 2 and e.code == -7
        return
    nc = 37
    g = torch.Generator(device=DEV).manual_seed(len(str(grid)))
    h = torch.randn((nc, p.n_dof), dtype=torch.float64, device=DEV, generator=g)
    delta = torch.rand(nc, dtype=torch.float64, device=DEV, generator=g) + 0.5
    hn, dn = h.cpu().numpy(), delta.cpu().numpy()
    B, x = blocks_and_rows(op, hn, dims, axes, species)
    K = B.shape[1]
    E = sum(np.abs(xb) @ np.abs(b).T for b, xb in zip(B, x))                       # [cell][orbit]
    E = E.reshape((nc, species) + tuple(d // 2 if a in axes else d for a, d in enumerate(dims)))
    for a in axes:                                                                 # the same for every image
        E = np.concatenate([np.flip(E, 2 + a), E], 2 + a)
    ref = dn[:, None] * (hn @ op.T)
    bound = dn[:, None] * E.reshape(nc, -1) * (operands + products * (K + 8) * 2.0 ** -23)
    size = np.abs(ref)
    for a in (np.zeros_like(ref), np.roll(ref, 1, 0)):                             # what the bound has to refuse
        assert np.mean(np.abs(a - ref) > bound) > 0.8
    assert np.median(bound) < 0.2 * np.median(size)
    for rows, depth in ((128, 16), (64, 16), (32, 16)) + (((256, 32),) if precision == "bf16x3" else ()):
        for splits in (1, 2):
            p.set_contraction_config(nc, rows, depth if precision == "fp32" or depth == 32 else 64, splits, precision=precision)
            rhs = torch.full_like(h, np.nan)
            p.collide(h, delta, rhs)
            assert np.all(np.abs(rhs.cpu().numpy() - ref) <= bound), (rows, splits)
