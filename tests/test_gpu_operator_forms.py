"""The two forms of the operator: block-wise (FP32 always, FP16 with several
right-hand sides, anything whose workgroups fit in two per CU, 512 pairs of a
4^4 block and a right-hand side on the card) and gather.  Every kernel variant
(a direction that one block spans or none, all link entries or two rows,
mirrored or explicit clover term) and both sides of the line between the forms
against the oracle, at the largest site's error."""
import numpy as np
import pytest

import oracle
from gpu_util import BC, REL_TOL_APPLY, Lattice, site_err
from paper_1710_07041_amd import synth

pytestmark = pytest.mark.gpu

# whole-lattice bound of one application, on the largest site error: the worst
# of up to 150k sites over the root mean square (x 10, as for the clover mirror)
SITE = {p: 10 * t for p, t in REL_TOL_APPLY.items()}


def check(lat, C, prec, nrhs, seed):
    psi = synth.gaussian_spinor(lat.dims, nrhs=nrhs, seed=seed)
    m0 = np.linspace(-0.3, 0.2, nrhs)
    out = lat.apply(psi, m0, prec, nrhs)
    for r in sorted({0, 1, nrhs // 2, nrhs - 1} & set(range(nrhs))):
        ref = oracle.apply_D(lat.dims, lat.U, C, m0[r], psi[r], BC)
        assert site_err(out[r], ref) <= SITE[prec], (lat.dims, prec, nrhs, r)


@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (4, 8, 8, 8), (8, 4, 4, 8), (4, 4, 4, 4)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
def test_variants(dims, prec):
    lat = Lattice(dims, eps=0.4, seed=61)
    C = np.ascontiguousarray(np.stack([lat.C[:, :6, :6], lat.C[:, 6:, 6:]], axis=1))
    C[-1, 1, 4, 5] += 0.5  # one mirrored entry of one site
    C[-1, 1, 5, 4] = np.conj(C[-1, 1, 4, 5])
    full = np.zeros_like(lat.C)
    full[:, :6, :6], full[:, 6:, 6:] = C[:, 0], C[:, 1]
    for explicit in (False, True):
        if explicit:
            lat.ctx.set_clover(C)
        for compressed in (True, False):
            lat.ctx.set_link_compression(compressed)
            for nrhs in (1, 2, 3):
                check(lat, full if explicit else lat.C, prec, nrhs, 62 + nrhs)


@pytest.mark.parametrize("dims,prec,nrhs", [
    ((16, 16, 16, 32), "f64", 1), ((16, 16, 16, 40), "f64", 1),  # 512 and 640 blocks
    ((16, 16, 16, 32), "f16", 1), ((16, 16, 16, 40), "f16", 1),
    ((16, 16, 16, 16), "f64", 2), ((16, 16, 16, 16), "f64", 3),
    ((4, 16, 16, 16), "f64", 8), ((4, 16, 16, 16), "f64", 9),
    ((16, 16, 16, 16), "f32", 7), ((16, 16, 16, 16), "f16", 7),  # a ragged last workgroup
])
def test_line_between_forms(dims, prec, nrhs):
    lat = Lattice(dims, eps=0.4, seed=71)
    check(lat, lat.C, prec, nrhs, 72)
