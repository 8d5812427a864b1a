"""The clover term of a gauge field mirrors the upper-left 3x3 block of each
chiral half in the lower-right one, and the kernels then skip the mirrored
entries.  An explicit clover term that breaks the mirror on a single site, in
a single entry, has to be read in full: the diagonal (slot 2 and half of slot
1) and the off-diagonal mirrored entries (slots 15-17) are each broken on the
last site and compared with the oracle."""
import numpy as np
import pytest

import oracle
from gpu_util import BC, REL_TOL_APPLY, Lattice, check_sap, gpu_sap, site_err
from paper_1710_07041_amd import synth

pytestmark = pytest.mark.gpu

DIMS = (8, 8, 4, 8)


@pytest.fixture(scope="module")
def lat():
    return Lattice(DIMS, eps=0.4, seed=51)


def halves(C):
    """The two chiral 6x6 halves (V, 2, 6, 6) of the oracle's clover term."""
    return np.ascontiguousarray(np.stack([C[:, :6, :6], C[:, 6:, 6:]], axis=1))


def test_clover_term_mirrors(lat):
    """The property itself, on the oracle's clover term (to its rounding)."""
    C = halves(lat.C)
    assert np.abs(C[:, :, :3, :3] + C[:, :, 3:, 3:]).max() <= 1e-14


@pytest.mark.parametrize("entry", [None, (3, 3), (4, 4), (5, 5), (3, 4), (3, 5), (4, 5)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
def test_broken_mirror_is_read(lat, prec, entry):
    m0, psi = -0.2, synth.gaussian_spinor(DIMS, seed=52)
    C = halves(lat.C)
    C[:, :, 3:, 3:] = -C[:, :, :3, :3]  # exactly, as the kernels may assume
    if entry is not None:
        i, j = entry
        C[-1, 1, i, j] += 0.5
        C[-1, 1, j, i] = np.conj(C[-1, 1, i, j])
    lat.ctx.set_clover(C)
    full = np.zeros_like(lat.C)  # (V, 12, 12), block diagonal in chirality
    full[:, :6, :6], full[:, 6:, 6:] = C[:, 0], C[:, 1]
    out = lat.apply(psi, m0, prec)
    ref = oracle.apply_D(DIMS, lat.U, full, m0, psi, BC)
    # the largest site error: one site's entry does not hide in the lattice norm
    assert site_err(out, ref) <= 10 * REL_TOL_APPLY[prec]
    sap = oracle.sap(DIMS, (4, 4, 4, 4), lat.U, full, m0, psi, 2, 4, BC)
    check_sap(gpu_sap(lat.ctx, psi, m0, 2, 4, prec), sap, prec, f"mirror {entry}")
