"""Restriction and prolongation in groups of right-hand sides (one, two and four
a workgroup, whole and ragged groups) and on a count of blocks that is no multiple
of the eight XCDs: each right-hand side bitwise as alone (its own sums do not
depend on the group), and alone P^+ P = 1 to the precision's rounding."""
import numpy as np
import pytest

from gpu_util import Lattice, rel, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[(16, 16, 16, 16), (4, 4, 8, 24), (8, 16, 16, 24)],
                ids=lambda d: "x".join(map(str, d)))
def lat(request):
    """256, 12 and 192 blocks."""
    import torch
    from paper_1710_07041_amd import ddsap
    lat = Lattice(request.param, eps=0.3, seed=5, oracle_clover=False)
    p = ddsap.default_amg_params()
    p.nvec, p.setup_iters, p.setup_ncy, p.setup_nmr, p.setup_prec, p.adapt = 5, 1, 1, 2, ddsap.DD_F32, 0
    lat.ctx.amg_setup(-0.2, torch.randn((5, lat.V, 4, 3), dtype=torch.complex128, device="cuda"), p)
    return lat


@pytest.mark.parametrize("nrhs", [2, 3, 4, 5, 7, 16])
@pytest.mark.parametrize("prec,tol", [("f64", 1e-14), ("f32", 2e-6)])
def test_groups(lat, prec, tol, nrhs):
    import torch
    ctx = lat.ctx
    x = torch.randn((nrhs, ctx.amg_coarse_size()), dtype=torch.complex128, device="cuda")
    fine, y = ctx.empty_blocked(prec, nrhs), torch.empty_like(x)
    ctx.amg_prolong(x, fine, prec, nrhs)
    ctx.amg_restrict(fine, y, prec, nrhs)
    back = torch.empty((nrhs, lat.V, 4, 3), dtype=torch.complex128, device="cuda")
    ctx.unpack(fine, back, prec, nrhs)
    for r in sorted({0, 1, nrhs // 2, nrhs - 1}):
        one, yo, bo = ctx.empty_blocked(prec, 1), torch.empty_like(x[:1]), torch.empty_like(back[:1])
        ctx.amg_prolong(x[r:r + 1].contiguous(), one, prec, 1)
        ctx.amg_restrict(one, yo, prec, 1)
        ctx.unpack(one, bo, prec, 1)
        ctx.synchronize()
        assert torch.equal(torch.view_as_real(back[r]), torch.view_as_real(bo[0])), r
        assert torch.equal(torch.view_as_real(y[r]), torch.view_as_real(yo[0])), r
        assert rel(to_host(yo)[0], to_host(x)[r]) < tol
    assert np.all(np.isfinite(to_host(y)))
