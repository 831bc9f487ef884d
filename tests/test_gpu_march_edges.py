"""The serial marches at the edges they are built with: the planar sweep takes 24 nodes a chunk, the tube sweep 62
columns a strip (th nodes in pairs of passes: 124), with loads 24 diagonals ahead; and the planar sweep of many cases
on rows whose halves are not whole cache lines, which takes four waves a workgroup.

Tolerances as in the other tests of the marches: stable recurrences of a few roundings a node, 1e-11."""
import functools

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import transport as tr
from oracle.velocity import VelocityGrid
from paper_1612_04488_amd import inputs, sis
from test_gpu_marches import DEV, TOL, dev, rel, test_mixture_marches, test_planar_marches, test_tube_marches

pytestmark = pytest.mark.gpu
march_planar, march_mixture, march_tube = test_planar_marches, test_mixture_marches, test_tube_marches
del test_planar_marches, test_mixture_marches, test_tube_marches


@pytest.mark.parametrize("sections", [23, 24, 25, 47, 48, 49, 72])
def test_planar_chunks(sections):
    march_planar(sections)


@pytest.mark.parametrize("sections", [23, 24, 25, 48, 49])
def test_mixture_chunks(sections):
    march_mixture(sections)


@pytest.mark.parametrize("n_th,n_vr,n_vz,nodes", [(122, 2, 2, 9), (124, 2, 2, 9), (124, 2, 2, 25), (124, 2, 4, 70), (126, 2, 2, 24),
                                                  (248, 2, 2, 7), (250, 2, 2, 7), (20, 2, 2, 23), (20, 2, 2, 24), (20, 2, 2, 25),
                                                  (20, 2, 2, 26), (6, 2, 2, 48), (6, 2, 2, 49)])
def test_tube_strips(n_th, n_vr, n_vz, nodes):
    march_tube(n_th, n_vr, n_vz, nodes)


@functools.lru_cache(maxsize=None)
def plan(n, parity, species):
    mix = dict(masses=(1.0, 2.0), diameters=(1.0, 0.8), chi=(0.4, 0.6), m_rho=3) if species == 2 else None
    return sis.Plan(n, 4.0, m_angle=2, parity=parity, mixture=mix)


@pytest.mark.parametrize("n,parity,species,cases", [(12, 2, 1, 511), (12, 2, 1, 512), (12, 2, 2, 256), (18, 2, 1, 171), (14, 2, 1, 400),
                                                    (14, 1, 1, 190), (16, 2, 1, 300)])
@pytest.mark.parametrize("nodes", [2, 25, 26])
def test_planar_sweep_of_many_cases(n, parity, species, cases, nodes):
    """216 velocities of a half row (one workgroup of four waves from 512 cases on, or of 256 with two species), 729
    (three), 686 (three), 343 (two thirds of two: one wave a workgroup), 512 (whole lines: one wave): every case alike,
    and the march of the stored half against the oracle's of the full grid."""
    p = plan(n, parity, species)
    x = inputs.nodes_tanh(nodes - 1)
    geom = sis.Geometry(p, [x] * cases, [0.8] * cases, [1] * cases)
    nv = p.n_vel
    rhs = np.random.default_rng(n + nodes).standard_normal((nodes, species, nv))
    h = torch.full((cases, nodes, species, nv), np.nan, dtype=torch.float64, device=DEV)
    sis.transport_sweep(p, geom, dev(rhs).repeat(cases, 1, 1), h)
    torch.cuda.synchronize()
    assert torch.equal(h, h[:1].expand_as(h))
    got = h[0].cpu().numpy()
    nu = p.tables()["nu"].reshape(species, n, -1)
    v = VelocityGrid(n, 4.0)
    lo2, lo3 = (n // 2 if parity == 2 else 0), (n // 2 if parity else 0)
    full = np.zeros((nodes, n, n, n))
    fnu = np.ones((n, n, n))
    for s in range(species):
        full[:, :, lo2:, lo3:] = rhs[:, s].reshape(nodes, n, n - lo2, n - lo3)
        fnu[:, lo2:, lo3:] = nu[s].reshape(n, n - lo2, n - lo3)
        ref = tr.sweep_1d(full, 0.8 * fnu, x, v)[:, :, lo2:, lo3:]
        assert rel(got[:, s], ref.reshape(nodes, nv)) < TOL, s
