"""The Schwarz sweep deals the right-hand sides of a block to several
workgroups when one workgroup per block would leave CUs idle.  On 16^4 (128
blocks of a colour) the group holds two right-hand sides of FP32 or FP16 data
and four of FP64 (one workgroup per CU instead of two), so these counts leave
a ragged last group; every right-hand side has to equal its lone run (a group
of one) bitwise, since the arithmetic per right-hand side is the same."""
import numpy as np
import pytest

from gpu_util import Lattice, to_dev
from paper_1710_07041_amd import synth

pytestmark = pytest.mark.gpu

DIMS = (16, 16, 16, 16)


@pytest.fixture(scope="module")
def lat():
    return Lattice(DIMS, eps=0.4, seed=41, oracle_clover=False)


@pytest.mark.parametrize("eo", [False, True])
@pytest.mark.parametrize("prec,nrhs", [("f32", 3), ("f32", 7), ("f16", 7), ("f64", 7), ("f32", 16)])
def test_groups_match_lone(lat, prec, nrhs, eo):
    eta = synth.gaussian_spinor(DIMS, nrhs=nrhs, seed=42)
    m0 = np.linspace(-0.3, 0.1, nrhs)

    def sap(x, m, n):
        eb, pb = lat.ctx.empty_blocked(prec, n), lat.ctx.empty_blocked(prec, n)
        lat.ctx.pack(x, eb, prec, n)
        lat.ctx.sap(m, eb, pb, 2, 4, prec, n, eo=eo)
        lat.ctx.synchronize()
        return pb.cpu().numpy().reshape(-1, n, pb.numel() // (n * (lat.V // 256)))  # [block][rhs][bytes]

    out = sap(to_dev(eta), m0, nrhs)
    for r in (0, 1, nrhs // 2, nrhs - 2, nrhs - 1):
        assert np.array_equal(out[:, r], sap(to_dev(eta[r:r + 1]), m0[r:r + 1], 1)[:, 0]), r
