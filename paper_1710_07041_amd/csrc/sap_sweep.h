// The plain Schwarz colour sweep (included by sap.hip): one 256-thread
// workgroup per block, one thread per site.
//
// What bounds it: two workgroups fit a CU (registers, LDS), i.e. two wavefronts
// per SIMD, and a workgroup's visit is a chain of its loads (8 us of a visit of
// 35 us at 32^3x64 in FP32), the face trips (5 us), the MR steps (4 x 3.9 us)
// and its stores.  One wavefront issues a VALU instruction per 5.3 cycles, two
// per SIMD one per 2.7, four one per 1.8 (a loop of independent FMAs), so an MR
// step takes what its 1400 instructions take to issue, whether or not another
// workgroup shares the CU; HBM idles meanwhile (FP32: 3.7 of 5.8 TB/s).
// Hence few instructions and branches in the step: a lattice without a
// direction that one block spans takes a kernel without the wrap tests (WRAP),
// y hops shift zeros in instead of testing lanes, lane moves carry no old
// value, and with a sigma . F clover term (SIG) both its halves stay in
// registers (FP32 arithmetic), so no memory load sits inside the step.
// Measured together, twelve FP32 cycles at 32^3x64: 7.07 -> 6.70 ms a call,
// ten FP16 ones at 48^3x96: 23.4 -> 22.5 ms, twelve FP64 ones at 24^3x48, which
// now carry the residual: 6.60 -> 6.05 ms.  The faces are published by the
// even-odd sweep's routine, a whole half spinor at a time: 6.70 -> 6.64 and 6.14
// -> 6.01 ms against one that goes spin by spin; forming FP64's residual anew
// every eighth cycle takes 0.06 ms of that back.
// More wavefronts did not pay: three workgroups per CU (168 registers, link
// rows rebuilt at each use) spill, 15.4 ms in FP32; two threads per site (512
// threads a block at 128 registers) double the LDS traffic and the barriers,
// 10.9 ms.
#pragma once

#include "block_ops.h"

namespace dd {

// FP64 data read psi again at the end of the visit and take the faces in an
// unrolled loop; FP32 arithmetic, at half the registers a thread, spills with
// either: it keeps psi in LDS meanwhile (PL) and one face trip in flight.
// 24^3x48, FP64: 6.05 against 6.75 ms, with an explicit clover term (eight
// registers spilled) 6.54 against 7.07; 4x24^2x48 with four right-hand sides 3.54
// against 3.85, explicit (twenty spilled) 3.77 against 4.16; 32^3x64, FP32: 8.98
// against 6.70 ms.
template <typename S> constexpr bool PSI_LDS = sizeof(S) < 8;

// The carried residual lets the rounding of psi add up from visit to visit.  FP64
// arithmetic, which formed it anew at every visit before it was carried, does so
// every FRESH_EVERY cycles: the error against exact sums is then at every count
// of cycles what it was (8^4: 3.9e-16; carried throughout, 4.5e-16 after 32) for
// 2% of the time of twelve cycles.  FP32 and FP16 have always carried it.
template <typename S> constexpr bool FRESH = sizeof(S) == 8;
constexpr int FRESH_EVERY = 8;

template <typename S, typename A, bool PL> struct SweepLds {
    cx<A> tf[6][BS];   // projected half spinors for the +t hops
    cx<A> tb[6][BS];   // U^+ times projected half spinors for the -t hops
    cx<A> del[12][BS]; // MR accumulator (each thread its own site's entries)
    vec2_t<S> psi[PL ? 12 : 1][BS]; // psi before the visit
    A red[4][4];
};

// ---- faces of direction MU (layout and contents: block_ops.h)
template <int MU, typename S, typename A>
__device__ __forceinline__ void blk_face_load(const Geom &g, int b, const int bc[4], int s, int r, int nrhs,
                                               const vec2_t<S> *__restrict__ F, vec2_t<S> raw[6])
{
    const int l = (s >> (2 * MU)) & 3;
    if (g.nb[MU] == 1 || (l != 0 && l != BEXT - 1)) return;
    const int dir = l == 0 ? -1 : 1;
    int bn, sn, sign;
    bool inb;
    neighbour_rt(g, b, bc, s, MU, dir, bn, sn, sign, inb);
    const vec2_t<S> *fp = F + ((long)bn * nrhs + r) * FACE_ELEMS + (2 * MU + (dir < 0 ? 1 : 0)) * 6 * 64 + face_index(s, MU);
#pragma unroll
    for (int e = 0; e < 6; ++e) raw[e] = fp[e * 64];
}
template <int MU, typename S, typename A>
__device__ __forceinline__ void blk_face_add(const Geom &g, const int bc[4], int s, const vec2_t<S> raw[6],
                                              const cx<A> W[9], cx<A> qu[6], cx<A> ql[6])
{
    if (g.nb[MU] == 1) return; // uniform: the in-block exchange wraps
    const int l = (s >> (2 * MU)) & 3;
    // the link and the published half spinors carry -1/2: only the boundary sign remains
    if (l == 0) {
        const A k = bc[MU] == 0 ? (A)g.bcs[MU] : (A)1;
        cx<A> h[6];
#pragma unroll
        for (int e = 0; e < 6; ++e) h[e] = ldc<A>(&raw[e]);
        recon_spin<MU, +1, 0, false>(qu, ql, h, k);
        recon_spin<MU, +1, 1, false>(qu, ql, h + 3, k);
    } else if (l == BEXT - 1) {
        const A k = bc[MU] + 1 == g.nb[MU] ? (A)g.bcs[MU] : (A)1;
        cx<A> h[6], t[3];
#pragma unroll
        for (int e = 0; e < 6; ++e) h[e] = ldc<A>(&raw[e]);
        su3_spin(W, h, t);
        recon_spin<MU, -1, 0, false>(qu, ql, t, k);
        su3_spin(W, h + 3, t);
        recon_spin<MU, -1, 1, false>(qu, ql, t, k);
    }
}

struct SArgs {
    Geom g;
    const int *blocks; // block ids of the swept colour
    int nblk;
    int nrhs;
    int rpg; // right-hand sides per workgroup (rhs_per_group)
    int nmr;
    int mode; // 0: psi = 0 everywhere; 1: psi_B = 0 on this colour; 2: general
    double m0[MAXRHS];
    const double *m0_dev; // per-rhs masses in device memory (overrides m0 when set)
    const long *eta_off;  // per-rhs element offsets of eta and psi (nullable)
    const long *psi_off;
    const int *active;    // right-hand sides with active[r] == 0 are skipped (nullable)
    int publish;          // write the face buffers for the next sweep
    int r12;              // links stored as SU(3): read two rows, rebuild the third
    int sig;              // the clover term is sigma . F: mirrored slots are not read
    int write_r;          // plain sweep: store the block residual for the next visit
    int fresh;            // plain FP64 sweep: form the block residual from psi (the faces are psi's)
    int psi_faces;        // plain FP64 sweep: publish the faces of psi, not of delta
};

// The block (grid x) and the right-hand sides [r0, r1) (grid y) of this
// workgroup.  False when none of them is active (uniform: nothing to do).
__device__ __forceinline__ bool sweep_part(const SArgs &a, int &b, int &r0, int &r1)
{
    b = a.blocks[xcd_remap(blockIdx.x, gridDim.x)];
    r0 = blockIdx.y * a.rpg;
    r1 = min(r0 + a.rpg, a.nrhs);
    if (!a.active) return true;
    bool any = false;
    for (int r = r0; r < r1; ++r) any |= a.active[r] != 0;
    return any;
}

// The MR coefficient of one right-hand side: the dot products <q, r> and
// <q, q> over the block (DPP sums within each wavefront, then a fixed-order
// combine of the four wavefronts through LDS), alpha = <q, r>/<q, q>; returns
// false when <q, q> vanishes (uniform over the workgroup).
template <typename LT, typename A>
__device__ __forceinline__ bool mr_alpha(LT &L, int lane, int wave, const cx<A> q[12], const cx<A> rr[12],
                                         cx<A> &alpha, bool mine = true)
{
    A qr_re = 0, qr_im = 0, qq = 0;
    if (mine) { // whether this wavefront's sites count
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            qr_re = fma(q[c].re, rr[c].re, qr_re);
            qr_re = fma(q[c].im, rr[c].im, qr_re);
            qr_im = fma(q[c].re, rr[c].im, qr_im);
            qr_im = fma(-q[c].im, rr[c].re, qr_im);
            qq = fma(q[c].re, q[c].re, qq);
            qq = fma(q[c].im, q[c].im, qq);
        }
    }
    qr_re = wave_sum(qr_re);
    qr_im = wave_sum(qr_im);
    qq = wave_sum(qq);
    if (lane == 63) { // where wave_sum leaves the total
        L.red[wave][0] = qr_re;
        L.red[wave][1] = qr_im;
        L.red[wave][2] = qq;
    }
    __syncthreads();
    qr_re = ((L.red[0][0] + L.red[1][0]) + L.red[2][0]) + L.red[3][0];
    qr_im = ((L.red[0][1] + L.red[1][1]) + L.red[2][1]) + L.red[3][1];
    qq = ((L.red[0][2] + L.red[1][2]) + L.red[2][2]) + L.red[3][2];
    if (qq == (A)0) return false;
    alpha = mk<A>(qr_re / qq, qr_im / qq);
    return true;
}

// SF is the storage type of the links and the clover term (S, or FP16 fields
// under FP32 spinors).
template <typename S, typename A, typename SF, int WAVES, bool WRAP, bool SIG>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(WAVES))) void k_sap_sweep(
    const vec2_t<S> *__restrict__ eta0, vec2_t<S> *__restrict__ psi0, const vec2_t<SF> *__restrict__ links,
    const vec2_t<SF> *__restrict__ clov, vec2_t<S> *__restrict__ faces, vec2_t<S> *__restrict__ resid, SArgs a)
{
    constexpr bool PL = PSI_LDS<S>;
    __shared__ SweepLds<S, A, PL> L;
    int b, rhs0, rhs1;
    if (!sweep_part(a, b, rhs0, rhs1)) return;
    const int s = threadIdx.x;
    const int lane = s & 63, wave = s >> 6;
    int bc[4];
    block_coords(a.g, b, bc);

    // register-resident links carry the hop factor -1/2
    cx<A> U[4][9];
    load_links4<A, true>(links + (long)b * 4 * 9 * BS + s, a.r12, (A)(-0.5), U);
    const vec2_t<SF> *cp = clov + (long)b * 36 * BS + s;
    constexpr bool HOLD = SIG && sizeof(A) == 4; // both clover halves in registers
    cx<A> cl[HOLD ? 36 : 18];
#pragma unroll
    for (int e = 0; e < (HOLD ? 36 : 18); ++e)
        if (clover_reads(SIG, e % 18)) cl[e] = ldc_stream<A>(cp + e * BS);

    for (int r = rhs0; r < rhs1; ++r) {
        // no barrier between right-hand sides: the t buffers and the partial
        // sums are rewritten only after the barriers of this one's first MR
        // step follow the last reads of the previous one's, the rest is each
        // thread's own
        if (a.active && !a.active[r]) continue; // uniform over the workgroup
        const A diag = (A)(4.0 + (a.m0_dev ? a.m0_dev[r] : a.m0[r]));
        const vec2_t<S> *__restrict__ eta = eta0 + (a.eta_off ? a.eta_off[r] : 0);
        vec2_t<S> *__restrict__ psi = psi0 + (a.psi_off ? a.psi_off[r] : 0);
        const long sp = ((long)b * a.nrhs + r) * 12 * BS + s; // (the carried residual has no slot offsets)
        // rho = R - (hops of the other colour's last update), R being this
        // block's residual after its previous visit (eta on the first)
        if (PL && a.mode == 2) {
#pragma unroll
            for (int c = 0; c < 12; ++c) L.psi[c][s] = psi[sp + c * BS];
        }
        // (FP64: where a.fresh is set, eta - (D psi)_B)
        const bool fresh = FRESH<S> && a.fresh;
        const vec2_t<S> *__restrict__ src = a.mode == 2 && !fresh ? resid : eta;
        vec2_t<S> er[12];
        cx<A> rr[12], q[12];
        const auto take_rho = [&]() {
#pragma unroll
            for (int c = 0; c < 12; ++c) er[c] = src[sp + c * BS];
            if (!PL && a.mode != 0) {
                vec2_t<S> f[6];
                blk_face_load<0, S, A>(a.g, b, bc, s, r, a.nrhs, faces, f);
                blk_face_add<0, S, A>(a.g, bc, s, f, U[0], q, q + 6);
                blk_face_load<1, S, A>(a.g, b, bc, s, r, a.nrhs, faces, f);
                blk_face_add<1, S, A>(a.g, bc, s, f, U[1], q, q + 6);
                blk_face_load<2, S, A>(a.g, b, bc, s, r, a.nrhs, faces, f);
                blk_face_add<2, S, A>(a.g, bc, s, f, U[2], q, q + 6);
                blk_face_load<3, S, A>(a.g, b, bc, s, r, a.nrhs, faces, f);
                blk_face_add<3, S, A>(a.g, bc, s, f, U[3], q, q + 6);
            }
            if (PL && a.mode != 0) face_consume<S, A>(a.g, b, bc, s, r, a.nrhs, faces, U, q);
#pragma unroll
            for (int c = 0; c < 12; ++c) rr[c] = ldc<A>(&er[c]) - q[c];
        };
        int it = 0;
        if (fresh) {
            // step -1 of the loop applies D_BB to psi
#pragma unroll
            for (int c = 0; c < 12; ++c) rr[c] = ldc<A>(psi + sp + c * BS);
            it = -1;
        } else {
#pragma unroll
            for (int c = 0; c < 12; ++c) q[c] = mk<A>(0, 0);
            take_rho();
        }
        // MR on D_BB: delta += alpha r, r -= alpha q
        for (; it < a.nmr; ++it) {
#pragma unroll
            for (int c = 0; c < 12; ++c) q[c] = mk<A>(0, 0);
            blk_t_post_spin<0>(L, U[3], s, rr, rr + 6);
            blk_t_post_spin<1>(L, U[3], s, rr, rr + 6);
            constexpr bool LATE = !HOLD && sizeof(SF) == 2;
            vec2_t<SF> c2late[LATE ? 18 : 1];
            if constexpr (HOLD) {
                clover_half_mac<A, SIG>(cl, diag, rr, q);
                clover_half_mac<A, SIG>(cl + 18, diag, rr + 6, q + 6);
            } else {
                const vec2_t<SF> *cp1 = cp + 18 * BS;
                // the address is the same at every MR step: hide that, or the
                // loads leave the loop and the half is held in registers
                asm volatile("" : "+v"(cp1));
                if constexpr (LATE) {
#pragma unroll
                    for (int e = 0; e < 18; ++e)
                        if (clover_reads(SIG, e)) c2late[e] = cp1[e * BS];
                    clover_half_mac<A, SIG>(cl, diag, rr, q);
                } else {
                    cx<A> c2[18];
#pragma unroll
                    for (int e = 0; e < 18; ++e)
                        if (clover_reads(SIG, e)) c2[e] = ldc<A>(cp1 + e * BS);
                    clover_half_mac<A, SIG>(cl, diag, rr, q);
                    clover_half_mac<A, SIG>(c2, diag, rr + 6, q + 6);
                }
            }
            blk_hop<0, WRAP>(a.g, b, bc, s, U[0], rr, rr + 6, q, q + 6);
            blk_hop<1, WRAP>(a.g, b, bc, s, U[1], rr, rr + 6, q, q + 6);
            blk_hop<2, WRAP>(a.g, b, bc, s, U[2], rr, rr + 6, q, q + 6);
            __syncthreads();
            blk_t_take<WRAP>(L, a.g, b, bc, s, U[3], q, q + 6);
            if constexpr (LATE) {
                cx<A> c2[18];
#pragma unroll
                for (int e = 0; e < 18; ++e)
                    if (clover_reads(SIG, e)) c2[e] = ldc<A>(&c2late[e]);
                clover_half_mac<A, SIG>(c2, diag, rr + 6, q + 6);
            }
            if (FRESH<S> && it < 0) { // uniform
                take_rho();
                __syncthreads(); // this step's reads of the t buffers end here
                continue;
            }
            cx<A> alpha;
            if (!mr_alpha(L, lane, wave, q, rr, alpha)) break;
#pragma unroll
            for (int c = 0; c < 12; ++c) {
                cx<A> d = mk<A>(0, 0);
                if (it > 0) d = L.del[c][s];
                cmac(d, alpha, rr[c]);
                L.del[c][s] = d;
                rr[c] = rr[c] - alpha * q[c];
            }
        }
        // psi_B += delta; the residual carried to the next visit; the faces
        // of delta for the other colour
        if (!PL && a.mode == 2) {
#pragma unroll
            for (int c = 0; c < 12; ++c) er[c] = psi[sp + c * BS];
        }
        if (a.write_r) {
#pragma unroll
            for (int c = 0; c < 12; ++c) stc(resid + sp + c * BS, rr[c]);
        }
#pragma unroll
        for (int c = 0; c < 12; ++c) rr[c] = it > 0 ? L.del[c][s] : mk<A>(0, 0);
        if (a.publish && !(FRESH<S> && a.psi_faces)) face_publish<S, A>(faces, b, a.nrhs, r, s, rr, U);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            if (a.mode == 2) rr[c] = rr[c] + ldc<A>(PL ? &L.psi[PL ? c : 0][s] : &er[c]);
            stc(psi + sp + c * BS, rr[c]);
        }
        if (FRESH<S> && a.publish && a.psi_faces) face_publish<S, A>(faces, b, a.nrhs, r, s, rr, U);
    }
}

} // namespace dd
