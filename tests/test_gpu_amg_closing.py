"""The coarse GMRES where its Krylov space is exhausted before its steps are:
lattices of one and two blocks with one to three test vectors (2 to 12
unknowns), up to 32 steps, against the direct solution.  The bound is the
solution's own conditioning, 200 eps cond(D_c + m0)."""
import numpy as np
import pytest

from gpu_util import Lattice, rel, to_dev, to_host
from paper_1710_07041_amd import synth
from test_gpu_amg import dense_from_blocks
from test_gpu_amg_shapes import f16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[((4, 4, 4, 4), 1), ((4, 4, 4, 4), 2), ((4, 4, 4, 4), 3), ((8, 4, 4, 4), 1),
                                        ((8, 4, 4, 4), 2), ((8, 4, 4, 4), 3)],
                ids=lambda p: "x".join(map(str, p[0])) + f"-{p[1]}")
def lat(request):
    from paper_1710_07041_amd import ddsap
    dims, n = request.param
    lat = Lattice(dims, eps=0.3, seed=3, oracle_clover=False)
    p = ddsap.default_amg_params()
    p.nvec, p.setup_iters, p.setup_ncy, p.setup_nmr, p.setup_prec, p.adapt = n, 1, 1, 2, ddsap.DD_F64, 0
    lat.ctx.amg_setup(-0.2, to_dev(synth.gaussian_spinor(dims, nrhs=n, seed=85)), p)
    lat.Dc = dense_from_blocks(dims, f16(lat.ctx.amg_coarse_operator()))
    return lat


def solve_all(lat, scale, k):
    """Three right-hand sides of one call: scale times a random one, zero, and a random one."""
    import torch
    nc = lat.Dc.shape[0]
    rng = np.random.default_rng(86)
    b = rng.standard_normal((3, nc)) + 1j * rng.standard_normal((3, nc))
    b[0] *= scale
    b[1] = 0
    m0 = np.array([-0.2, 0.0, 0.1])
    x = torch.empty((3, nc), dtype=torch.complex128, device="cuda")
    lat.ctx.amg_coarse_solve(m0, to_dev(b), x, k, 3)
    lat.ctx.synchronize()
    x = to_host(x)
    assert np.all(x[1] == 0)
    for r in (0, 2):
        A = lat.Dc + m0[r] * np.eye(nc)
        assert rel(x[r], np.linalg.solve(A, b[r])) <= 200 * np.finfo(float).eps * np.linalg.cond(A), (scale, k, r)


@pytest.mark.parametrize("k", [13, 32])
def test_exhausted_space(lat, k):
    solve_all(lat, 1.0, k)


@pytest.mark.parametrize("scale", [1e-12, 1e-6, 1e6, 1e16])
def test_any_scale(lat, scale):
    """The solution is linear in b: the step at which the space counts as
    exhausted must not depend on |b|."""
    solve_all(lat, scale, 16)
