"""The FP64 smoother's rounding does not add up over its cycles: it forms the
block residual from psi as stored every eight cycles, so the error against the
oracle after 32 cycles is the error after four.  Root mean squares over 98304
numbers of one distribution, alike to under 2%; rounding that adds up makes them
grow by a factor of 1.19.  Counts of cycles on both sides of a fresh residual,
one and two right-hand sides, and every form of the kernel stay at the bound of
the smoother's other tests."""
import numpy as np
import pytest

import oracle
from gpu_util import BC, Lattice, check_sap, gpu_sap, rel
from paper_1710_07041_amd import synth

pytestmark = pytest.mark.gpu


def test_rounding_does_not_add_up():
    lat = Lattice((8, 8, 8, 8), eps=0.4, seed=2)
    eta, m0 = synth.gaussian_spinor(lat.dims, seed=3), -0.2
    err = {}
    for ncy in (4, 32):
        ref = oracle.sap(lat.dims, (4, 4, 4, 4), lat.U, lat.C, m0, eta, ncy, 4, BC)
        err[ncy] = rel(gpu_sap(lat.ctx, eta, m0, ncy, 4, "f64"), ref)
    print(f"SAPGROWTH {err}", flush=True)
    assert err[32] <= 1.08 * err[4]


@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (4, 8, 8, 8), (4, 4, 4, 4)])
@pytest.mark.parametrize("explicit", [False, True])
def test_cycle_counts(dims, explicit):
    lat = Lattice(dims, eps=0.4, seed=12)
    eta, m0 = synth.gaussian_spinor(dims, nrhs=2, seed=13), np.array([-0.25, 0.1])
    C = np.ascontiguousarray(np.stack([lat.C[:, :6, :6], lat.C[:, 6:, 6:]], axis=1))
    if explicit:
        C[0, 0, 3, 4] += 0.25
        C[0, 0, 4, 3] = np.conj(C[0, 0, 3, 4])
        lat.ctx.set_clover(C)
    full = np.zeros_like(lat.C)
    full[:, :6, :6], full[:, 6:, 6:] = C[:, 0], C[:, 1]
    for ncy, nmr in ((8, 4), (9, 4), (10, 1), (17, 3), (9, 0)):
        out = gpu_sap(lat.ctx, eta, m0, ncy, nmr, "f64", nrhs=2)
        for r in range(2):
            ref = oracle.sap(dims, (4, 4, 4, 4), lat.U, full if explicit else lat.C, m0[r], eta[r], ncy, nmr, BC)
            if nmr == 0:
                assert not np.any(out[r]) and not np.any(ref)
            else:
                check_sap(out[r], ref, "f64", f"{dims} ncy={ncy} nmr={nmr} r={r}")
