"""The FP32 gather form, which one right-hand side with an explicit clover term
runs on a lattice of more than 512 blocks: the operator against the oracle, and the
residual inside the two-level preconditioner against the block-wise form's (the
same clover term to rounding, so the results agree to FP32 rounding)."""
import numpy as np
import pytest

import oracle
from gpu_util import BC, REL_TOL_APPLY, Lattice, rel, site_err, to_dev, to_host
from paper_1710_07041_amd import synth

pytestmark = pytest.mark.gpu

DIMS = (16, 16, 16, 40)


def test_f32_gather_explicit_clover():
    import torch
    from paper_1710_07041_amd import ddsap
    lat = Lattice(DIMS, eps=0.4, seed=101)
    p = ddsap.default_amg_params()
    p.nvec, p.setup_iters, p.setup_ncy, p.setup_nmr, p.setup_prec, p.adapt = 2, 1, 1, 2, ddsap.DD_F32, 0
    lat.ctx.amg_setup(-0.2, torch.randn((2, lat.V, 4, 3), dtype=torch.complex128, device="cuda"), p)
    psi = synth.gaussian_spinor(DIMS, seed=102)

    def precondition():
        x = to_dev(psi)
        a, b = lat.ctx.empty_blocked("f32"), lat.ctx.empty_blocked("f32")
        lat.ctx.pack(x, a, "f32")
        lat.ctx.amg_precondition(-0.2, a, b, "f32")
        y = torch.empty_like(x)
        lat.ctx.unpack(b, y, "f32")
        lat.ctx.synchronize()
        return to_host(y)

    mirrored = precondition()
    C = np.ascontiguousarray(np.stack([lat.C[:, :6, :6], lat.C[:, 6:, 6:]], axis=1))
    lat.ctx.set_clover(C)  # the oracle's, mirrored to rounding only
    assert rel(precondition(), mirrored) <= 1e-5
    C[5, 1, 4, 5] += 0.5
    C[5, 1, 5, 4] = np.conj(C[5, 1, 4, 5])
    lat.ctx.set_clover(C)
    full = np.zeros_like(lat.C)
    full[:, :6, :6], full[:, 6:, 6:] = C[:, 0], C[:, 1]
    for compressed in (True, False):
        lat.ctx.set_link_compression(compressed)
        out = lat.apply(psi, -0.2, "f32")
        assert site_err(out, oracle.apply_D(DIMS, lat.U, full, -0.2, psi, BC)) <= 10 * REL_TOL_APPLY["f32"]
