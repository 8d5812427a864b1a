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


@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (4, 8, 8, 8)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
def test_smoother_forms(dims, prec):
    """The four forms of the sweep (with and without a direction that one
    block spans, mirrored and explicit clover term), with all nine link
    entries read too, two right-hand sides each, against the oracle."""
    lat = Lattice(dims, eps=0.4, seed=53)
    eta, m0 = synth.gaussian_spinor(dims, nrhs=2, seed=54), np.array([-0.25, 0.1])
    broken = halves(lat.C)
    broken[0, 0, 3, 4] += 0.25
    broken[0, 0, 4, 3] = np.conj(broken[0, 0, 3, 4])
    full = np.zeros_like(lat.C)
    full[:, :6, :6], full[:, 6:, 6:] = broken[:, 0], broken[:, 1]
    for clover in (None, broken):
        if clover is not None:
            lat.ctx.set_clover(clover)
        for compressed in (True, False):
            lat.ctx.set_link_compression(compressed)
            out = gpu_sap(lat.ctx, eta, m0, 3, 4, prec, nrhs=2)
            for r in range(2):
                C = lat.C if clover is None else full
                ref = oracle.sap(dims, (4, 4, 4, 4), lat.U, C, m0[r], eta[r], 3, 4, BC)
                check_sap(out[r], ref, prec, f"form {dims} {clover is None} {compressed} r={r}")
