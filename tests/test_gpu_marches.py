"""The serial marches (planar sweep, tube sweep, velocity equations) against the oracle: node
counts around a group of the sweep (8 nodes) and a chunk of the velocity equation (256), and
th columns of one strip of the tube sweep (62 a pass) and two.

The recurrences are stable (positive upwind weights), so n steps of a few roundings each
keep n * 1e-15 relative: 1e-11 covers the largest here (300 nodes + 66 columns) with the
sums of the moments and integrals, which take no part in the marches."""
import functools

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import collision, mixture, polar
from oracle import transport as tr
from oracle.velocity import VelocityGrid
from paper_1612_04488_amd import inputs, sis

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-11
MIX = dict(masses=inputs.MIX_NEAR["mixture"]["masses"], diameters=inputs.MIX_NEAR["mixture"]["diameters"],
           chi=(0.4, 0.6))


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def rel(a, b):
    return float(np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300))


@functools.lru_cache(maxsize=None)
def planar():
    return sis.Plan(6, 4.0, m_angle=2), collision.FSM(VelocityGrid(6, 4.0), n_pad=12, m_angle=2)


@functools.lru_cache(maxsize=None)
def mix():
    return (sis.Plan(6, 4.0, m_angle=2, mixture=dict(m_rho=3, **MIX)),
            mixture.MixtureFSM(VelocityGrid(6, 4.0), MIX["masses"], MIX["diameters"], MIX["chi"], m_angle=2, m_rho=3))


@pytest.mark.parametrize("sections", [1, 8, 9, 16, 17, 255, 256, 299])
def test_planar_marches(sections):
    print("planar", sections, flush=True)
    p, f = planar()
    x, d, N = inputs.nodes_tanh(sections), 0.8, 1.1
    geom = sis.Geometry(p, [x], [d], [1])
    n = geom.n_cells
    rng = np.random.default_rng(sections)
    rhs = rng.standard_normal((n, 6, 6, 6))
    hh, mom = dev(np.zeros((n, 216))), dev(np.zeros((n, 4)))
    sis.transport_sweep(p, geom, dev(rhs.reshape(n, -1)), hh, mom)
    amom = rng.standard_normal((n, 4))
    U, dU = dev(np.zeros(n)), dev(np.zeros(n))
    sis.diffusion_correct(p, geom, mom, dev(amom), N, U, dU)
    torch.cuda.synchronize()
    assert rel(hh.cpu().numpy(), tr.sweep_1d(rhs, d * f.nu, x, f.grid).reshape(n, -1)) < TOL
    m = mom.cpu().numpy()
    ref = tr.diffusion_1d(x, m[0, 0], m[:, 2], amom[:, 0] + N * d * amom[:, 1], d, N, 1)
    assert rel(U.cpu().numpy(), ref) < TOL and rel(dU.cpu().numpy(), ref - m[:, 0]) < TOL
    for scheme in ("SIS", "CIS"):
        r = sis.solve(p, geom, scheme=scheme, eps=0.0, max_it=2, raise_not_converged=False)
        for k, field in (("M", "U"), ("Q", "q")):
            assert abs(r[k][0] - tr.flow_rate_1d(x, r[field])) < TOL * np.max(np.abs(r[field])), (scheme, k)


@pytest.mark.parametrize("sections", [1, 8, 255, 256, 299])
def test_mixture_marches(sections):
    print("mixture", sections, flush=True)
    p, o = mix()
    x, d, N = inputs.nodes_tanh(sections), 0.8, 1.1
    geom = sis.Geometry(p, [x], [d], [1])
    n = geom.n_cells
    rng = np.random.default_rng(sections)
    rhs = rng.standard_normal((n, 2, 6, 6, 6))
    hh, mom = dev(np.zeros((n, 432))), dev(np.zeros((n, 2, 4)))
    sis.transport_sweep(p, geom, dev(rhs.reshape(n, -1)), hh, mom)
    amom = rng.standard_normal((n, 2, 4))
    U, dU = dev(np.zeros((n, 2))), dev(np.zeros((n, 2)))
    sis.diffusion_correct(p, geom, mom, dev(amom), N, U, dU)
    torch.cuda.synchronize()
    h_o = mixture.sweep_1d(o, rhs, x, d)
    assert rel(hh.cpu().numpy(), h_o.reshape(n, -1)) < TOL
    m = mom.cpu().numpy()
    ref = mixture.velocity_1d(o, x, m, amom[:, :, :2], d, np.array([N, N]))
    assert rel(U.cpu().numpy(), ref) < TOL
    r = sis.solve(p, geom, eps=0.0, max_it=2, raise_not_converged=False)
    scale = [tr.flow_rate_1d(x, r["U"][:, s]) for s in range(2)]
    for k, field in (("M", "U"), ("Q", "q")):      # one common factor sqrt(m / m_A)
        want = [tr.flow_rate_1d(x, r[field][:, s]) for s in range(2)]
        f = r["M"][0][0] / scale[0]
        assert all(abs(r[k][0][s] - f * want[s]) < TOL * f * np.max(np.abs(r[field])) for s in range(2)), k


@pytest.mark.parametrize("n_th,n_vr,n_vz,nodes", [(4, 2, 2, 3), (6, 6, 6, 4), (12, 4, 2, 300), (126, 2, 2, 5),
                                                  (128, 2, 4, 9), (130, 2, 2, 9), (132, 2, 2, 70)])
def test_tube_marches(n_th, n_vr, n_vz, nodes):
    print("tube", n_th, n_vr, n_vz, nodes, flush=True)
    p = sis.Plan(0, 3.0, m_angle=2, polar=dict(n_vr=n_vr, vr_max=3.0, n_th=n_th, n_vz=n_vz))
    g = polar.PolarGrid(n_vr, 3.0, n_th, n_vz, 3.0)
    nu = p.tables()["nu"].reshape(g.shape)
    r, d, N = np.sin(0.5 * np.pi * (np.arange(nodes) + 1.0) / nodes), 0.8, 1.1
    geom = sis.Geometry(p, [r, r], [d, 3.0], [1, 1], kind="tube")
    n, nv = geom.n_cells, g.VR.size
    rng = np.random.default_rng(n_th)
    rhs = rng.standard_normal((n,) + g.shape)
    hh, mom = dev(np.zeros((n, nv))), dev(np.zeros((n, 8)))
    sis.transport_sweep(p, geom, dev(rhs.reshape(n, nv)), hh, mom)
    amom = rng.standard_normal((n, 4))
    U, dU = dev(np.zeros(n)), dev(np.zeros(n))
    sis.diffusion_correct(p, geom, mom, dev(amom), N, U, dU)
    torch.cuda.synchronize()
    h, m = hh.cpu().numpy().reshape(rhs.shape), mom.cpu().numpy()
    for c, dc in enumerate((d, 3.0)):
        s = slice(c * nodes, (c + 1) * nodes)
        assert rel(h[s], polar.sweep_tube(rhs[s], dc * nu, r, g)) < TOL, c
        assert rel(U.cpu().numpy()[s], polar.velocity_tube(r, m[s], amom[s], dc, N)) < TOL, c
    out = sis.solve(p, geom, eps=0.0, max_it=2, raise_not_converged=False)
    for c in range(2):
        s = slice(c * nodes, (c + 1) * nodes)
        for k, field in (("M", "U"), ("Q", "q")):
            assert abs(out[k][c] - polar.flow_rate_tube(r, out[field][s])) < TOL * np.max(np.abs(out[field])), (c, k)
