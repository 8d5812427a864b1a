"""The even-odd sweep's forms: mirrored and explicit clover term (which feeds the
Cholesky factors and the even sites' products), two and three link rows, with and
without a direction that one block spans, at one and two workgroups per CU; the
plain sweep on FP16 fields with an explicit clover term; and the bytes that the
profile counts for an even-odd call."""
import numpy as np
import pytest

import oracle
from gpu_util import BC, Lattice, check_sap, gpu_sap, round_fp16
from paper_1710_07041_amd import synth
from test_gpu_sap_eo import gpu_sap_eo

pytestmark = pytest.mark.gpu


def explicit_clover(lat, size):
    """The lattice's clover term with one mirrored entry changed: (halves, full)."""
    C = np.ascontiguousarray(np.stack([lat.C[:, :6, :6], lat.C[:, 6:, 6:]], axis=1))
    for half, i, j in ((0, 3, 4), (1, 4, 5)):
        C[-1, half, i, j] += size
        C[-1, half, j, i] = np.conj(C[-1, half, i, j])
    C[0, 1, 5, 5] += size
    full = np.zeros_like(lat.C)
    full[:, :6, :6], full[:, 6:, 6:] = C[:, 0], C[:, 1]
    return C, full


@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (4, 8, 8, 8)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
def test_even_odd_forms(dims, prec):
    lat = Lattice(dims, eps=0.4, seed=53)
    eta, m0 = synth.gaussian_spinor(dims, nrhs=2, seed=54), np.array([-0.25, 0.1])
    C, full = explicit_clover(lat, 0.25)
    for ref_clover in (lat.C, full):
        if ref_clover is full:
            lat.ctx.set_clover(C)
        for compressed in (True, False):
            lat.ctx.set_link_compression(compressed)
            out = gpu_sap_eo(lat, eta, m0, 3, 4, prec, nrhs=2)
            for r in range(2):
                ref = oracle.sap(dims, (4, 4, 4, 4), lat.U, ref_clover, m0[r], eta[r], 3, 4, BC, eo=True)
                check_sap(out[r], ref, "eo-" + prec, f"form {dims} {ref_clover is full} {compressed} r={r}")


@pytest.mark.parametrize("prec", ["f32", "f16"])
def test_even_odd_two_workgroups_per_cu(prec):
    """A wrapping lattice of 256 blocks a colour (one workgroup per CU with one
    right-hand side, two with two): each right-hand side against the oracle."""
    dims = (4, 16, 32, 64)
    lat = Lattice(dims, eps=0.4, seed=55)
    eta, m0 = synth.gaussian_spinor(dims, nrhs=2, seed=56), np.array([-0.25, 0.1])
    ref = [oracle.sap(dims, (4, 4, 4, 4), lat.U, lat.C, m0[r], eta[r], 2, 3, BC, eo=True) for r in range(2)]
    out = gpu_sap_eo(lat, eta, m0, 2, 3, prec, nrhs=2)
    for r in range(2):
        check_sap(out[r], ref[r], "eo-" + prec, f"two r={r}")
        check_sap(gpu_sap_eo(lat, eta[r], m0[r], 2, 3, prec), ref[r], "eo-" + prec, f"one r={r}")


@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (4, 8, 8, 8)])
def test_half_fields_explicit_clover(dims):
    """FP16 links and clover under the FP32 sweep against the SAP of the rounded fields."""
    lat = Lattice(dims, eps=0.4, seed=57)
    eta, m0 = synth.gaussian_spinor(dims, nrhs=2, seed=58), np.array([-0.25, 0.1])
    C, full = explicit_clover(lat, 0.25)
    lat.ctx.set_sap_half_fields(True)
    lat.ctx.set_link_compression(False)
    for ref_clover in (lat.C, full):
        if ref_clover is full:
            lat.ctx.set_clover(C)
        out = gpu_sap(lat.ctx, eta, m0, 3, 4, "f32", nrhs=2)
        for r in range(2):
            ref = oracle.sap(dims, (4, 4, 4, 4), round_fp16(lat.U), round_fp16(ref_clover), m0[r], eta[r], 3, 4, BC)
            check_sap(out[r], ref, "f32h-rounded", f"{dims} {ref_clover is full} r={r}")


@pytest.mark.parametrize("prec,size", [("f64", 8), ("f32", 4), ("f16", 2)])
def test_even_odd_bytes(prec, size):
    """Per site: links and clover 72 reals each, and per right-hand side eta read,
    psi written and, but on a colour's first visit, psi read, 24 reals each."""
    dims, n, ncy = (8, 8, 8, 8), 3, 5
    lat = Lattice(dims, eps=0.4, seed=59, oracle_clover=False)
    eta, psi = lat.ctx.empty_blocked(prec, n), lat.ctx.empty_blocked(prec, n)
    eta.zero_()
    lat.ctx.profile_enable()
    lat.ctx.sap(-0.2, eta, psi, ncy, 4, prec, n, eo=True)
    lat.ctx.synchronize()
    got = lat.ctx.profile_read()["sap_sweep_eo_" + prec]
    assert got["launches"] == 2 * ncy
    half = lat.V / 2  # one colour
    assert got["bytes"] == size * half * (2 * ncy * (144 + n * 48) + 2 * (ncy - 1) * n * 24)
