// Wilson-clover operator on the blocked layout.
//
//   (D psi)(x) = (4 + m0) psi(x) + C(x) psi(x)
//              - 1/2 sum_mu [ (1 - g_mu) U_mu(x) psi(x+mu) + (1 + g_mu) U_mu(x-mu)^+ psi(x-mu) ]
//
// Two forms.  Block-wise (k_dslash_block): one workgroup per Schwarz block and
// group of right-hand sides holds the block's links and clover term for all of
// them and hands the in-block hops across lanes.  Gather (k_dslash): one
// workgroup per block and right-hand side, one thread per site, each hop reads
// the neighbour's spinor and link.  block_wise() says which runs where.
// The hop uses the chiral-basis spin projection so each of the eight SU(3)
// products acts on two spins only.
// Bandwidth bound: per site the algorithmic traffic is links 72 + clover 72 +
// spinor in 24 + out 24 reals per right-hand side.  Workgroups are remapped
// so that each XCD sweeps a contiguous range of blocks (shared L2 for the
// neighbour faces); clover terms and outputs, used once, go through
// streaming loads/stores.
#include "block_ops.h"
#include "dd_device.h"
#include "dd_internal.h"

#include <type_traits>

namespace dd {

namespace {

struct DArgs {
    Geom g;
    int nrhs;
    int rpg; // block-wise form: right-hand sides per workgroup
    int block_id;
    double m0[MAXRHS];
    const double *m0_dev; // per-rhs masses in device memory (overrides m0 when set)
    const long *in_off;   // per-rhs element offset added to the input (nullable)
    const int *active;    // right-hand sides with active[r] == 0 are skipped (nullable)
    int r12;              // links stored as SU(3): read two rows, rebuild the third
    int sig;              // the clover term is sigma . F: mirrored slots are not read
};

// One hop of direction index k = 2 mu + (0: forward, 1: backward) onto acc.
template <int K, typename A>
__device__ __forceinline__ void hop_k(const cx<A> psi[12], const cx<A> U[9], A kk, cx<A> acc[12])
{
    cx<A> h[6], uh[6];
    if (K & 1) {
        proj_plus<K / 2>(psi, h);
        su3_mul_adj(U, h, uh);
        recon_plus<K / 2>(acc, uh, kk);
    } else {
        proj_minus<K / 2>(psi, h);
        su3_mul(U, h, uh);
        recon_minus<K / 2>(acc, uh, kk);
    }
}

// The gather form keeps the block's own input spinor in LDS: an in-block
// neighbour is read from there and only a neighbour across the block face
// comes from memory (those lanes alone).
template <int K, typename SI, typename A>
__device__ __forceinline__ void hop_stg(const vec2_t<SI> *__restrict__ g, const vec2_t<SI> *stg, int sn, bool inb,
                                        const cx<A> U[9], A kk, cx<A> acc[12])
{
    vec2_t<SI> raw[12];
    if (inb) {
#pragma unroll
        for (int c = 0; c < 12; ++c) raw[c] = stg[c * BS + sn];
    } else {
#pragma unroll
        for (int c = 0; c < 12; ++c) raw[c] = g[c * BS];
    }
    cx<A> psi[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) psi[c] = ldc<A>(&raw[c]);
    hop_k<K, A>(psi, U, kk, acc);
}

template <typename SI, typename A>
__device__ __forceinline__ void hop_stg_switch(int k, const vec2_t<SI> *__restrict__ g, const vec2_t<SI> *stg, int sn,
                                               bool inb, const cx<A> U[9], A kk, cx<A> acc[12])
{
    switch (k) {
    case 0: hop_stg<0, SI, A>(g, stg, sn, inb, U, kk, acc); break;
    case 1: hop_stg<1, SI, A>(g, stg, sn, inb, U, kk, acc); break;
    case 2: hop_stg<2, SI, A>(g, stg, sn, inb, U, kk, acc); break;
    case 3: hop_stg<3, SI, A>(g, stg, sn, inb, U, kk, acc); break;
    case 4: hop_stg<4, SI, A>(g, stg, sn, inb, U, kk, acc); break;
    case 5: hop_stg<5, SI, A>(g, stg, sn, inb, U, kk, acc); break;
    case 6: hop_stg<6, SI, A>(g, stg, sn, inb, U, kk, acc); break;
    default: hop_stg<7, SI, A>(g, stg, sn, inb, U, kk, acc); break;
    }
}

template <typename SF, typename A>
__device__ __forceinline__ void load_hop_link(const vec2_t<SF> *__restrict__ links, int b, int s, int k, int bn,
                                              int sn, bool r12, cx<A> U[9])
{
    const int mu = k >> 1;
    const int lb = (k & 1) ? bn : b, ls = (k & 1) ? sn : s;
    load_link<A>(links + ((long)lb * 4 + mu) * 9 * BS + ls, r12, U);
}

// The eight hops onto acc; in is this right-hand side's input, block stride
// bstr.  The loops over the directions are deliberately not unrolled: unrolled,
// the compiler hoists all hops' loads ahead of the arithmetic and spills.
template <typename SI, typename SF, typename A>
__device__ __forceinline__ void hops(const vec2_t<SI> *__restrict__ in, long bstr, const vec2_t<SF> *__restrict__ links,
                                     const DArgs &a, int b, const int bc[4], int s, const vec2_t<SI> *stg, cx<A> acc[12])
{
    if constexpr (sizeof(SI) == 4) {
        // FP32 input: both hops of a direction in one trip, so the link that
        // site x - mu reads for its forward hop is re-read for the backward hop
        // of site x at once (from L1) rather than a trip later (with FP64 input
        // the pair does not fit in registers, and FP16 input runs faster at
        // four waves per SIMD, where the pair spills)
#pragma unroll 1
        for (int mu = 0; mu < 4; ++mu) {
            int bf, sf, gf, bb, sb, gb;
            bool inf, inbk;
            neighbour_rt(a.g, b, bc, s, mu, +1, bf, sf, gf, inf);
            neighbour_rt(a.g, b, bc, s, mu, -1, bb, sb, gb, inbk);
            vec2_t<SI> pf[12], pb[12];
            cx<A> Uf[9], Ub[9];
            if (inf) {
#pragma unroll
                for (int c = 0; c < 12; ++c) pf[c] = stg[c * BS + sf];
            } else {
                const vec2_t<SI> *qf = in + bf * bstr + sf;
#pragma unroll
                for (int c = 0; c < 12; ++c) pf[c] = qf[c * BS];
            }
            load_hop_link<SF, A>(links, b, s, 2 * mu, bf, sf, a.r12, Uf);
            if (inbk) {
#pragma unroll
                for (int c = 0; c < 12; ++c) pb[c] = stg[c * BS + sb];
            } else {
                const vec2_t<SI> *qb = in + bb * bstr + sb;
#pragma unroll
                for (int c = 0; c < 12; ++c) pb[c] = qb[c * BS];
            }
            load_hop_link<SF, A>(links, b, s, 2 * mu + 1, bb, sb, a.r12, Ub);
            cx<A> psi[12];
#pragma unroll
            for (int c = 0; c < 12; ++c) psi[c] = ldc<A>(&pf[c]);
            const A kf = (A)(-0.5 * gf), kb = (A)(-0.5 * gb);
            switch (mu) {
            case 0: hop_k<0, A>(psi, Uf, kf, acc); break;
            case 1: hop_k<2, A>(psi, Uf, kf, acc); break;
            case 2: hop_k<4, A>(psi, Uf, kf, acc); break;
            default: hop_k<6, A>(psi, Uf, kf, acc); break;
            }
#pragma unroll
            for (int c = 0; c < 12; ++c) psi[c] = ldc<A>(&pb[c]);
            switch (mu) {
            case 0: hop_k<1, A>(psi, Ub, kb, acc); break;
            case 1: hop_k<3, A>(psi, Ub, kb, acc); break;
            case 2: hop_k<5, A>(psi, Ub, kb, acc); break;
            default: hop_k<7, A>(psi, Ub, kb, acc); break;
            }
        }
    } else {
        // the link of the next hop is loaded one trip ahead, so only the
        // spinor loads of a hop wait a full round trip
        int bn, sn, sign;
        bool inb;
        neighbour_rt(a.g, b, bc, s, 0, +1, bn, sn, sign, inb);
        cx<A> U[9];
        load_hop_link<SF, A>(links, b, s, 0, bn, sn, a.r12, U);
#pragma unroll 1
        for (int k = 0; k < 8; ++k) {
            const vec2_t<SI> *p = in + bn * bstr + sn;
            const A kk = (A)(-0.5 * sign);
            int bn2 = bn, sn2 = sn, sign2 = sign;
            bool inb2 = inb;
            cx<A> Un[9];
            if (k < 7) { // uniform
                const int k2 = k + 1;
                neighbour_rt(a.g, b, bc, s, k2 >> 1, (k2 & 1) ? -1 : 1, bn2, sn2, sign2, inb2);
                load_hop_link<SF, A>(links, b, s, k2, bn2, sn2, a.r12, Un);
            }
            hop_stg_switch<SI, A>(k, p, stg, sn, inb, U, kk, acc);
#pragma unroll
            for (int e = 0; e < 9; ++e) U[e] = Un[e];
            bn = bn2;
            sn = sn2;
            sign = sign2;
            inb = inb2;
        }
    }
}

// The hops inside block b alone (the block operator D_BB).
template <typename SI, typename SF, typename A>
__device__ __forceinline__ void hops_block(const vec2_t<SF> *__restrict__ links, const DArgs &a, int b, const int bc[4],
                                           int s, const vec2_t<SI> *stg, cx<A> acc[12])
{
#pragma unroll 1
    for (int k = 0; k < 8; ++k) {
        int bn, sn, sign;
        bool inb;
        neighbour_rt(a.g, b, bc, s, k >> 1, (k & 1) ? -1 : 1, bn, sn, sign, inb);
        if (!inb) continue;
        cx<A> U[9];
        load_hop_link<SF, A>(links, b, s, k, bn, sn, a.r12, U);
        hop_stg_switch<SI, A>(k, stg, stg, sn, true, U, (A)(-0.5 * sign), acc);
    }
}

// occupancy target per precision: enough waves per SIMD to keep HBM busy
// without letting the scheduler hoist all eight hops' loads at once
template <typename SI, typename A> struct DslashWaves {
    static constexpr int value = sizeof(A) == 8 ? 2 : (sizeof(SI) == 2 ? 4 : 3);
};

// Gather form: one 256-thread workgroup per (block, right-hand side); those of
// one block follow each other in the launch order, so the block's links and
// clover terms are re-read from L2.  Streaming clover loads (NTC) only with a
// single right-hand side.  SIG: 1 a mirrored clover term, 0 a full one, -1 as
// a.sig says.  (FP64 fields with several right-hand sides: lanes of a wavefront
// that shared each link among two or four right-hand sides took 573 us where
// this form takes 519, 24^3x48 and four, and 5240 where it takes 4800, 32^3x64
// and twelve: a wavefront then covers 16 or 32 sites, short of whole 128-byte
// lines, and its in-block neighbours come from memory.)
template <typename SI, typename SO, typename SF, typename A, bool BLOCKONLY, bool RESID, bool NTC, int SIG>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(DslashWaves<SI, A>::value))) void k_dslash(
    const vec2_t<SI> *__restrict__ in, vec2_t<SO> *__restrict__ out, const vec2_t<SF> *__restrict__ links,
    const vec2_t<SF> *__restrict__ clov, const vec2_t<SO> *__restrict__ resid, DArgs a)
{
    const int s = threadIdx.x;
    int b = a.block_id, r = 0;
    if (!BLOCKONLY) {
        const int wg = xcd_remap(blockIdx.x, gridDim.x);
        b = wg / a.nrhs;
        r = wg - b * a.nrhs;
        if (a.active && !a.active[r]) return; // uniform over the workgroup
    }
    int bc[4];
    block_coords(a.g, b, bc);
    cx<A> acc[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = mk<A>(0, 0);
    const A diag = (A)(4.0 + (a.m0_dev ? a.m0_dev[r] : a.m0[r]));
    const vec2_t<SI> *__restrict__ inr = in + (a.in_off ? a.in_off[r] : 0) + (long)r * 12 * BS;
    const long bstr = (long)a.nrhs * 12 * BS;
    __shared__ vec2_t<SI> stg[12 * BS];
    {
        const vec2_t<SI> *own = inr + b * bstr + s;
#pragma unroll
        for (int c = 0; c < 12; ++c) stg[c * BS + s] = own[c * BS];
        __syncthreads();
    }
    if constexpr (BLOCKONLY) hops_block<SI, SF, A>(links, a, b, bc, s, stg, acc);
    else hops<SI, SF, A>(inr, bstr, links, a, b, bc, s, stg, acc);
    // one chiral half at a time: halves the registers the clover needs
#pragma unroll 1
    for (int k = 0; k < 2; ++k) {
        cx<A> cl[18];
        const vec2_t<SF> *cp = clov + ((long)b * 36 + 18 * k) * BS + s;
        load_clover_half<A, NTC>(cp, SIG < 0 ? a.sig != 0 : SIG != 0, cl);
        cx<A> psi[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) psi[c] = ldc<A>(&stg[(6 * k + c) * BS + s]);
        if (k == 0) clover_half_mac(cl, diag, psi, acc);
        else clover_half_mac(cl, diag, psi, acc + 6);
    }
    const long sp = b * bstr + (long)r * 12 * BS + s;
    if (RESID) {
#pragma unroll
        for (int c = 0; c < 12; ++c) stc_stream(out + sp + c * BS, ldc_stream<A>(resid + sp + c * BS) - acc[c]);
    } else {
#pragma unroll
        for (int c = 0; c < 12; ++c) stc_stream(out + sp + c * BS, acc[c]);
    }
}

// Block-wise form: one workgroup per Schwarz block (and group of a.rpg
// right-hand sides) holds the site's links and clover term in registers for all
// of them and takes them one after the other; the in-block hops go across lanes
// (t through LDS), the hops that leave the block are computed two per thread
// (face_hop) and handed over through LDS.  A right-hand side then reads each
// spinor of the block once, a half more for the neighbours' faces, and no link
// or clover term; the links of the face hops wait in LDS.  Bound by the L2
// before: with every right-hand side (or three) fetching the links and clover
// terms of its hops anew, the 61 KB of face links a workgroup needs kept falling
// out of the L2 -- 11.0 GB fetched for the 3.3 GB that 32^3x64 with twelve
// right-hand sides needs in FP32, at a hit rate of 48%.  32^3x64 FP32: 2380 ->
// 1790 us with twelve, 327 -> 279 with one; 24^3x48 FP16 with five: 281 -> 205.
// Now bound by HBM and the memory latency of a right-hand side's faces, which
// two workgroups per CU cover for each other.
// WRAP: some direction has a single block.  R12: two rows a link; else a.r12
// says.  SIG: a mirrored clover term; else all of it is read, half 1 anew for
// each right-hand side (FP16 as stored, in registers).  RESID: out = resid - D in.
// LAST: the clover term, the largest of the nine, is added after the hops, as in
// the gather form and in the sums of FP64 and of FP32 with up to three
// right-hand sides since ever: started from, every hop rounds at its size (FP32
// 1.09e-7 against 9.7e-8, FP64 2.41e-16 against 2.20e-16).  FP32 with four and
// more has always started from it, and the setup's interpolation, twelve
// vectors at a time, magnifies a last bit.
// The links of a thread's two face hops: their first two rows and, with nine
// entries, the third of as many as there is room for (ROWS3; the other's is read
// again from the L2).  Nine entries, all read again for each right-hand side:
// 32^3x64 FP32 with twelve 2840 us, 4x24^2x48 122; in LDS 1932 and 85.
template <typename A, typename SF> struct DLds {
    cx<A> tf[6][BS]; // projected half spinors for the +t hops
    cx<A> tb[6][BS]; // U^+ times projected half spinors for the -t hops
    cx<A> fb[2][6][BS]; // transported half spinors of the face hops
    vec2_t<SF> fl[2][6][BS];
};
template <typename SF, bool R12> constexpr int ROWS3 = R12 ? 0 : sizeof(SF) == 2 ? 2 : sizeof(SF) == 4 ? 1 : 0;
template <typename A, typename SF, int N3> struct DLds3 : DLds<A, SF> {
    vec2_t<SF> f3[N3][3][BS];
};

template <typename SI, typename SO, typename SF, typename A, int WAVES, bool WRAP, bool R12, bool SIG, bool LAST, bool RESID>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(WAVES))) void k_dslash_block(
    const vec2_t<SI> *__restrict__ in, vec2_t<SO> *__restrict__ out, const vec2_t<SF> *__restrict__ links,
    const vec2_t<SF> *__restrict__ clov, const vec2_t<SO> *__restrict__ resid, DArgs a)
{
    constexpr int N3 = ROWS3<SF, R12>;
    __shared__ std::conditional_t<(N3 > 0), DLds3<A, SF, N3>, DLds<A, SF>> L;
    const bool r12 = R12 || a.r12;
    const int rend = min((int)(blockIdx.y + 1) * a.rpg, a.nrhs);
    if (a.active) {
        bool any = false;
        for (int r = blockIdx.y * a.rpg; r < rend; ++r) any |= a.active[r] != 0;
        if (!any) return; // uniform: nothing to do
    }
    const int b = xcd_remap(blockIdx.x, gridDim.x);
    const int s = threadIdx.x;
    int bc[4];
    block_coords(a.g, b, bc);
    const FaceHop h0 = face_hop(a.g, b, bc, s, 0), h1 = face_hop(a.g, b, bc, s, 1);
    const vec2_t<SF> *l0 = links + ((long)h0.lb * 4 + h0.mu) * 9 * BS + h0.ls;
    const vec2_t<SF> *l1 = links + ((long)h1.lb * 4 + h1.mu) * 9 * BS + h1.ls;
#pragma unroll
    for (int e = 0; e < 6; ++e) {
        L.fl[0][e][s] = l0[e * BS];
        L.fl[1][e][s] = l1[e * BS];
    }
    if (!r12) {
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            if constexpr (N3 > 0) L.f3[0][e][s] = l0[(6 + e) * BS];
            if constexpr (N3 > 1) L.f3[1][e][s] = l1[(6 + e) * BS];
        }
    }
    // register-resident links carry the hop factor -1/2
    cx<A> U[4][9];
    load_links4<A>(links + (long)b * 4 * 9 * BS + s, r12, (A)(-0.5), U);
    constexpr bool HOLD = SIG && sizeof(A) == 4; // both clover halves in registers
    constexpr bool RAW = !SIG && sizeof(SF) == 2; // half 1 as stored
    cx<A> cl[HOLD ? 36 : 18];
    vec2_t<SF> c2[HOLD ? 1 : 18];
    const vec2_t<SF> *cp = clov + (long)b * 36 * BS + s;
#pragma unroll
    for (int e = 0; e < (HOLD ? 36 : 18); ++e)
        if (clover_reads(SIG, e % 18)) cl[e] = ldc<A>(cp + e * BS);
    if constexpr (RAW) {
#pragma unroll
        for (int e = 0; e < 18; ++e) c2[e] = cp[(18 + e) * BS];
    }

    // FP16 data leave room for one face hop's spinor of the next right-hand side,
    // in flight during the present one (32^3x64 with two 310 -> 297 us, with twelve
    // 1456 -> 1393; with wrap tests it is slower, 4x24^2x48 with two 17.7 -> 18.8,
    // and next to a full clover term it spills)
    constexpr bool AHEAD = sizeof(SI) == 2 && SIG && !WRAP;
    vec2_t<SI> wn[AHEAD ? 12 : 1];
    const auto face0 = [&](int r) {
        const vec2_t<SI> *pp = in + (a.in_off ? a.in_off[r] : 0) + ((long)h0.bn * a.nrhs + r) * 12 * BS + h0.sn;
#pragma unroll
        for (int c = 0; c < 12; ++c) wn[c] = pp[c * BS];
    };
    if constexpr (AHEAD) face0(blockIdx.y * a.rpg);
    for (int r = blockIdx.y * a.rpg; r < rend; ++r) {
        if (a.active && !a.active[r]) { // uniform over the workgroup
            if constexpr (AHEAD) {
                if (r + 1 < rend) face0(r + 1);
            }
            continue;
        }
        const A diag = (A)(4.0 + (a.m0_dev ? a.m0_dev[r] : a.m0[r]));
        const vec2_t<SI> *__restrict__ inr = in + (a.in_off ? a.in_off[r] : 0);
        const long sp = ((long)b * a.nrhs + r) * 12 * BS + s;
        // in flight while the faces are computed
        vec2_t<SI> xr[12];
#pragma unroll
        for (int c = 0; c < 12; ++c) xr[c] = inr[sp + c * BS];
        // the previous right-hand side's reads of the LDS buffers end here
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const FaceHop &h = j == 0 ? h0 : h1;
            if (WRAP && h.inblk) continue; // uniform
            const vec2_t<SI> *pp = inr + ((long)h.bn * a.nrhs + r) * 12 * BS + h.sn;
            cx<A> W[9], w[12];
#pragma unroll
            for (int c = 0; c < 12; ++c) w[c] = AHEAD && j == 0 ? ldc<A>(&wn[AHEAD ? c : 0]) : ldc<A>(pp + c * BS);
#pragma unroll
            for (int e = 0; e < 6; ++e) W[e] = ldc<A>(&L.fl[j][e][s]);
            if (r12) {
                face_third_row(W);
            } else {
                const vec2_t<SF> *lj = (j == 0 ? l0 : l1) + 6 * BS;
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    if constexpr (N3 > 0) W[6 + e] = j < N3 ? ldc<A>(&L.f3[j % N3][e][s]) : ldc<A>(lj + e * BS);
                    else W[6 + e] = ldc<A>(lj + e * BS);
                }
            }
            face_hop_post(h, w, W, s, L.fb[j]);
        }
        if constexpr (AHEAD) {
            if (r + 1 < rend) face0(r + 1);
        }
        cx<A> x[12], q[12];
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            x[c] = ldc<A>(&xr[c]);
            q[c] = mk<A>(0, 0);
        }
        blk_t_post_spin<0>(L, U[3], s, x, x + 6);
        blk_t_post_spin<1>(L, U[3], s, x, x + 6);
        const auto load_half1 = [&]() {
            if constexpr (!HOLD && !RAW) {
                // the same for every right-hand side: hide that, or it is held
                // in registers
                int zero = 0;
                asm volatile("" : "+s"(zero));
#pragma unroll
                for (int e = 0; e < 18; ++e)
                    if (clover_reads(SIG, e)) c2[e] = cp[zero + (18 + e) * BS];
            }
        };
        const auto site_term = [&]() {
            clover_half_mac<A, SIG>(cl, diag, x, q);
            if constexpr (HOLD) {
                clover_half_mac<A, SIG>(cl + 18, diag, x + 6, q + 6);
            } else {
                cx<A> ch[18];
#pragma unroll
                for (int e = 0; e < 18; ++e)
                    if (clover_reads(SIG, e)) ch[e] = ldc<A>(&c2[e]);
                clover_half_mac<A, SIG>(ch, diag, x + 6, q + 6);
            }
        };
        if constexpr (!LAST) {
            load_half1();
            site_term();
        }
        blk_hop<0, WRAP>(a.g, b, bc, s, U[0], x, x + 6, q, q + 6);
        blk_hop<1, WRAP>(a.g, b, bc, s, U[1], x, x + 6, q, q + 6);
        blk_hop<2, WRAP>(a.g, b, bc, s, U[2], x, x + 6, q, q + 6);
        __syncthreads();
        if constexpr (LAST) load_half1();
        blk_t_take<WRAP>(L, a.g, b, bc, s, U[3], q, q + 6);
        face_gather(a.g, s, &L.fb[0][0][0], &L.fb[1][0][0], q);
        if constexpr (LAST) site_term();
        if (RESID) {
#pragma unroll
            for (int c = 0; c < 12; ++c) stc_stream(out + sp + c * BS, ldc_stream<A>(resid + sp + c * BS) - q[c]);
        } else {
#pragma unroll
            for (int c = 0; c < 12; ++c) stc_stream(out + sp + c * BS, q[c]);
        }
    }
}

DArgs make_args(const dd_ctx *ctx, const double *m0, int nrhs)
{
    DArgs a{};
    for (int i = 0; i < 4; ++i) {
        a.g.nb[i] = ctx->g.nb[i];
        a.g.bstride[i] = ctx->g.bstride[i];
        a.g.bcs[i] = ctx->g.bcs[i];
    }
    a.g.nblocks = ctx->g.nblocks;
    a.nrhs = nrhs;
    a.r12 = ctx->link_r12 ? 1 : 0;
    a.sig = ctx->clover_sigma ? 1 : 0;
    for (int r = 0; r < nrhs && r < MAXRHS && m0; ++r) a.m0[r] = m0[r];
    return a;
}

// Which form runs.  Block-wise where all its workgroups run at once (waves per
// CU), since latency is what counts there and the gather form's eight serial
// round trips lose: FP64 8^4 12.9 against 11.2 us, 16^4 22.4 against 18.8 (one
// workgroup per CU: a second round costs more than it gains, 4x16^3 with seven
// right-hand sides 20.7 against 23.6), FP16 16^4 12.8 against 8.9, 4x24^2x48
// 14.4 against 11.3.  Beyond that, several right-hand sides share the fields:
// FP32 at every count, FP16 (24^3x48: two 94 -> 92 us, five 281 -> 205), not FP64,
// where the exchange buffers leave one workgroup per CU, which streams worse
// than the gather form (24^3x48 with five: 707 us against 637).  One alone:
// block-wise in FP32 with a mirrored clover term (24^3x48 91.9 -> 90.4 us); with
// an explicit one, re-read late, the gather form stays ahead (95.3 against 92.0),
// as in FP16, where its four waves per SIMD stream better (32^3x64: 173 us
// against 193).
bool wraps(const Geom &g) { return g.nb[0] == 1 || g.nb[1] == 1 || g.nb[2] == 1 || g.nb[3] == 1; }
template <typename SF> bool block_wise(const dd_ctx *ctx, const DArgs &a, int waves)
{
    if ((long)ctx->g.nblocks * a.nrhs <= (long)ctx->ncu * waves) return true;
    return a.nrhs > 1 ? sizeof(SF) < 8 : sizeof(SF) == 4 && a.sig;
}

template <typename SI, typename SO, typename SF, typename A, bool RESID, bool NTC>
void launch_gather(dd_ctx *ctx, const DArgs &a, const void *in, void *out, int field_prec, const void *resid)
{
    // FP64 fields test the clover term's form at run time; FP16 fields gain by
    // not waiting for that (24^3x48: 59.1 -> 56.1 us, explicit 64.7 -> 57.4);
    // FP32 fields come here with an explicit one only
    constexpr int OTHER = sizeof(SF) == 8 ? -1 : 0;
    auto kernel = k_dslash<SI, SO, SF, A, false, RESID, NTC, OTHER>;
    if constexpr (sizeof(SF) == 2) {
        if (a.sig) kernel = k_dslash<SI, SO, SF, A, false, RESID, NTC, 1>;
    }
    kernel<<<ctx->g.nblocks * a.nrhs, BS, 0, ctx->stream>>>(
        static_cast<const vec2_t<SI> *>(in), static_cast<vec2_t<SO> *>(out),
        static_cast<const vec2_t<SF> *>(ctx->links[field_prec].p), static_cast<const vec2_t<SF> *>(ctx->clover[field_prec].p),
        static_cast<const vec2_t<SO> *>(resid), a);
}

template <typename SI, typename SO, typename SF, typename A, int WAVES, bool LAST, bool RESID>
void launch_block(dd_ctx *ctx, DArgs a, const void *in, void *out, int field_prec, const void *resid)
{
    a.rpg = rhs_per_group(ctx->g.nblocks, a.nrhs, ctx->ncu * WAVES);
    // two rows a link and a mirrored clover term, nine entries, or any
    auto pick = [&](auto wrap) {
        constexpr bool WRAP = decltype(wrap)::value;
        return !a.sig ? k_dslash_block<SI, SO, SF, A, WAVES, WRAP, false, false, LAST, RESID>
               : a.r12 ? k_dslash_block<SI, SO, SF, A, WAVES, WRAP, true, true, LAST, RESID>
                       : k_dslash_block<SI, SO, SF, A, WAVES, WRAP, false, true, LAST, RESID>;
    };
    auto kernel = wraps(a.g) ? pick(std::true_type{}) : pick(std::false_type{});
    kernel<<<dim3(ctx->g.nblocks, (a.nrhs + a.rpg - 1) / a.rpg), BS, 0, ctx->stream>>>(
        static_cast<const vec2_t<SI> *>(in), static_cast<vec2_t<SO> *>(out),
        static_cast<const vec2_t<SF> *>(ctx->links[field_prec].p), static_cast<const vec2_t<SF> *>(ctx->clover[field_prec].p),
        static_cast<const vec2_t<SO> *>(resid), a);
}

template <typename SI, typename SO, typename SF, typename A, bool RESID>
Status launch(dd_ctx *ctx, const DArgs &a, const void *in, void *out, int field_prec, const void *resid)
{
    const double V = (double)ctx->g.V, n = a.nrhs;
    // the method's data volume: links (72 reals per site) + clover (72) once,
    // input and output spinors per right-hand side; with gauge compression the
    // kernel reads 48 of the 72 link reals, which this figure does not count
    const double by = V * (144.0 * sizeof(SF) + 24.0 * n * (sizeof(SI) + sizeof(SO) * (RESID ? 2 : 1)));
    int cls = sizeof(SF) == 8 ? (sizeof(SI) == 8 ? K_DSLASH_F64 : K_DSLASH_F32IN_F64)
                              : (sizeof(SF) == 4 ? K_DSLASH_F32 : K_DSLASH_F16);
    ProfScope ps(ctx->prof, ctx->stream, cls, by, 1848.0 * V * n);
    // workgroups per CU that the LDS buffers leave room for
    constexpr int WAVES = sizeof(A) == 8 ? 1 : 2;
    if (block_wise<SF>(ctx, a, WAVES)) {
        if (sizeof(SF) == 8 || (sizeof(SF) == 4 && a.nrhs < 4)) launch_block<SI, SO, SF, A, WAVES, sizeof(SF) != 2, RESID>(ctx, a, in, out, field_prec, resid);
        else launch_block<SI, SO, SF, A, WAVES, sizeof(SF) == 8, RESID>(ctx, a, in, out, field_prec, resid);
    } else {
        if (sizeof(SF) < 8 || a.nrhs == 1) launch_gather<SI, SO, SF, A, RESID, true>(ctx, a, in, out, field_prec, resid);
        else launch_gather<SI, SO, SF, A, RESID, sizeof(SF) < 8>(ctx, a, in, out, field_prec, resid);
    }
    DD_HIP_TRY(hipGetLastError());
    return Status::ok();
}

} // namespace

Status launch_dslash(dd_ctx *ctx, const double *m0, int nrhs, const void *in, int in_prec, void *out, int out_prec,
                     int field_prec, const double *resid, const double *m0_dev, const long *in_off, const int *active)
{
    if (!in || !out || !ctx->links[field_prec].p || !ctx->clover[field_prec].p || (!m0 && !m0_dev))
        return Status{DD_INVALID_ARG, "operator: missing buffer"};
    DArgs a = make_args(ctx, m0, nrhs);
    a.m0_dev = m0_dev;
    a.in_off = in_off;
    a.active = active;
    bool rs = resid != nullptr;
    if (in_prec == DD_F64 && out_prec == DD_F64 && field_prec == DD_F64)
        return rs ? launch<double, double, double, double, true>(ctx, a, in, out, DD_F64, resid)
                  : launch<double, double, double, double, false>(ctx, a, in, out, DD_F64, resid);
    if (in_prec == DD_F32 && out_prec == DD_F64 && field_prec == DD_F64 && !rs)
        return launch<float, double, double, double, false>(ctx, a, in, out, DD_F64, nullptr);
    if (in_prec == DD_F32 && out_prec == DD_F32 && field_prec == DD_F32)
        return rs ? launch<float, float, float, float, true>(ctx, a, in, out, DD_F32, resid)
                  : launch<float, float, float, float, false>(ctx, a, in, out, DD_F32, nullptr);
    if (in_prec == DD_F16 && out_prec == DD_F16 && field_prec == DD_F16 && !rs)
        return launch<__half, __half, __half, float, false>(ctx, a, in, out, DD_F16, nullptr);
    return Status{DD_INVALID_ARG, "unsupported precision combination for the operator"};
}

Status launch_dslash_block(dd_ctx *ctx, double m0, int block_id, const void *in, void *out, int prec)
{
    DArgs a = make_args(ctx, &m0, 1);
    a.block_id = block_id;
    ProfScope ps(ctx->prof, ctx->stream, K_DSLASH_BLOCK, 256.0 * (144.0 + 48.0) * real_bytes(prec), 1848.0 * 256);
    if (prec == DD_F64)
        k_dslash<double, double, double, double, true, false, true, -1><<<1, BS, 0, ctx->stream>>>(
            static_cast<const double2 *>(in), static_cast<double2 *>(out), ctx->links[DD_F64].as<double2>(),
            ctx->clover[DD_F64].as<double2>(), nullptr, a);
    else if (prec == DD_F32)
        k_dslash<float, float, float, float, true, false, true, -1><<<1, BS, 0, ctx->stream>>>(
            static_cast<const float2 *>(in), static_cast<float2 *>(out), ctx->links[DD_F32].as<float2>(),
            ctx->clover[DD_F32].as<float2>(), nullptr, a);
    else
        k_dslash<__half, __half, __half, float, true, false, true, -1><<<1, BS, 0, ctx->stream>>>(
            static_cast<const __half2 *>(in), static_cast<__half2 *>(out), ctx->links[DD_F16].as<__half2>(),
            ctx->clover[DD_F16].as<__half2>(), nullptr, a);
    DD_HIP_TRY(hipGetLastError());
    return Status::ok();
}

} // namespace dd
