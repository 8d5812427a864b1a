// Block-local building blocks shared by the Schwarz sweeps and the operator
// kernel that works block by block: the hops inside a 4^4 block, the hops that
// leave it, and the sums over a wavefront.
//
// One 256-thread workgroup owns one block, one thread one site.  D_BB is
// applied direction by direction: each thread publishes the spin-projected
// half spinor of its site for the +mu hop of site x-mu, and U_mu(x)^+ times
// the projected half spinor for the -mu hop of site x+mu, across the lanes of
// a wavefront (one t-slice) for x, y and z and through LDS for t; so every
// link of the block is read once and no in-block spinor is re-read from
// memory.
#pragma once

#include "dd_device.h"

namespace dd {

// Direction-dispatched spin algebra for run-time loops over mu (a switch on a
// uniform value; each case is the compile-time specialisation).
template <typename A> __device__ __forceinline__ void proj_m(int mu, const cx<A> v[12], cx<A> h[6])
{
    switch (mu) {
    case 0: proj_minus<0>(v, h); break;
    case 1: proj_minus<1>(v, h); break;
    case 2: proj_minus<2>(v, h); break;
    default: proj_minus<3>(v, h); break;
    }
}
template <typename A> __device__ __forceinline__ void proj_p(int mu, const cx<A> v[12], cx<A> h[6])
{
    switch (mu) {
    case 0: proj_plus<0>(v, h); break;
    case 1: proj_plus<1>(v, h); break;
    case 2: proj_plus<2>(v, h); break;
    default: proj_plus<3>(v, h); break;
    }
}
template <typename A> __device__ __forceinline__ void recon_m(int mu, cx<A> q[12], const cx<A> t[6], A k)
{
    switch (mu) {
    case 0: recon_minus<0>(q, t, k); break;
    case 1: recon_minus<1>(q, t, k); break;
    case 2: recon_minus<2>(q, t, k); break;
    default: recon_minus<3>(q, t, k); break;
    }
}
template <typename A> __device__ __forceinline__ void recon_p(int mu, cx<A> q[12], const cx<A> t[6], A k)
{
    switch (mu) {
    case 0: recon_plus<0>(q, t, k); break;
    case 1: recon_plus<1>(q, t, k); break;
    case 2: recon_plus<2>(q, t, k); break;
    default: recon_plus<3>(q, t, k); break;
    }
}

// The complex value that lane (src4 / 4) of this wavefront holds in v
// (ds_bpermute: a cross-lane read, no LDS storage and no barrier).
template <typename A> __device__ __forceinline__ cx<A> lane_fetch(const cx<A> &v, int src4)
{
    if constexpr (sizeof(A) == 4) {
        return mk<A>(__int_as_float(__builtin_amdgcn_ds_bpermute(src4, __float_as_int(v.re))),
                     __int_as_float(__builtin_amdgcn_ds_bpermute(src4, __float_as_int(v.im))));
    } else {
        const long long r = __double_as_longlong(v.re), i = __double_as_longlong(v.im);
        const int r0 = __builtin_amdgcn_ds_bpermute(src4, (int)r), r1 = __builtin_amdgcn_ds_bpermute(src4, (int)(r >> 32));
        const int i0 = __builtin_amdgcn_ds_bpermute(src4, (int)i), i1 = __builtin_amdgcn_ds_bpermute(src4, (int)(i >> 32));
        return mk<A>(__longlong_as_double(((long long)r1 << 32) | (unsigned)r0),
                     __longlong_as_double(((long long)i1 << 32) | (unsigned)i0));
    }
}

// The x and y neighbours of a 4^4 block (site s = x + 4y + 16z + 64t on
// thread s) are lanes of the same quad (x) or 16-lane row (y): DPP moves
// reach them at VALU rate, rotating within the quad (x +- 1 mod 4) or the row
// (y +- 1 mod 4, i.e. lane +- 4 mod 16).  Lanes whose neighbour lies outside
// the block get their own block's wrapped site and never use it.  z crosses
// rows and keeps ds_bpermute.
template <int CTRL> __device__ __forceinline__ int dpp_mov(int v)
{
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, false);
}
template <int MU, int DIR, typename A> __device__ __forceinline__ cx<A> lane_hop(const cx<A> &v, int sn)
{
    if constexpr (MU >= 2) {
        return lane_fetch<A>(v, (sn & 63) << 2);
    } else {
        // quad_perm [1,2,3,0] / [3,0,1,2]: lane k reads lane k + 1 / k - 1 of
        // its quad; row_ror:12 / row_ror:4: lane i reads lane i + 4 / i - 4
        // of its row of 16
        constexpr int CTRL = MU == 0 ? (DIR > 0 ? 0x39 : 0x93) : (DIR > 0 ? 0x12C : 0x124);
        if constexpr (sizeof(A) == 4) {
            return mk<A>(__int_as_float(dpp_mov<CTRL>(__float_as_int(v.re))),
                         __int_as_float(dpp_mov<CTRL>(__float_as_int(v.im))));
        } else {
            const long long r = __double_as_longlong(v.re), i = __double_as_longlong(v.im);
            const int r0 = dpp_mov<CTRL>((int)r), r1 = dpp_mov<CTRL>((int)(r >> 32));
            const int i0 = dpp_mov<CTRL>((int)i), i1 = dpp_mov<CTRL>((int)(i >> 32));
            return mk<A>(__longlong_as_double(((long long)r1 << 32) | (unsigned)r0),
                         __longlong_as_double(((long long)i1 << 32) | (unsigned)i0));
        }
    }
}

// ---- one spin (SP = 0, 1) of the projections, SG = -1: (1 - g), +1: (1 + g)
// h = u_SP + SG (A l)_SP with A_k = -i sigma_k, A_t = 1
template <int MU, int SG, int SP, typename A>
__device__ __forceinline__ void proj_spin(const cx<A> u[6], const cx<A> l[6], cx<A> h[3])
{
    constexpr int SL = MU < 2 ? 1 - SP : SP; // the lower spin that A mixes in
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const cx<A> a = u[3 * SP + c], x = l[3 * SL + c];
        // (A l): x: -i l1, -i l0; y: -l1, l0; z: -i l0, i l1; t: l0, l1
        if (MU == 0) h[c] = SG > 0 ? a + tmi(x) : a + ti(x);
        if (MU == 1) h[c] = (SG > 0) == (SP == 0) ? a - x : a + x;
        if (MU == 2) h[c] = (SG > 0) == (SP == 0) ? a + tmi(x) : a + ti(x);
        if (MU == 3) h[c] = SG > 0 ? a + x : a - x;
    }
}
// (u, l) += k (t, SG A^+ t) for the spin SP of t (k = 1 when KONE)
template <int MU, int SG, int SP, bool KONE, typename A>
__device__ __forceinline__ void recon_spin(cx<A> u[6], cx<A> l[6], const cx<A> t[3], A k)
{
    constexpr int SL = MU < 2 ? 1 - SP : SP;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const cx<A> x = KONE ? t[c] : k * t[c];
        u[3 * SP + c] = u[3 * SP + c] + x;
        cx<A> &y = l[3 * SL + c];
        // A^+ t: x: i t1, i t0 on l0, l1; y: t1, -t0; z: i t0, -i t1; t: t0, t1
        if (MU == 0) y = y + (SG > 0 ? ti(x) : tmi(x));
        if (MU == 1) y = (SG > 0) == (SP == 1) ? y + x : y - x;
        if (MU == 2) y = y + ((SG > 0) == (SP == 0) ? ti(x) : tmi(x));
        if (MU == 3) y = SG > 0 ? y + x : y - x;
    }
}
// t = W h and t = W^+ h for one spin, in explicit multiply-adds (their order: see
// face_mul)
template <typename A> __device__ __forceinline__ void su3_spin(const cx<A> W[9], const cx<A> h[3], cx<A> t[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const cx<A> u = W[a * 3], x = h[0];
        cx<A> acc = mk<A>(fma(u.re, x.re, -(u.im * x.im)), fma(u.im, x.re, u.re * x.im));
        cmac(acc, W[a * 3 + 1], h[1]);
        cmac(acc, W[a * 3 + 2], h[2]);
        t[a] = acc;
    }
}
template <int MU, typename A> __device__ __forceinline__ void su3_spin_adj(const cx<A> W[9], const cx<A> h[3], cx<A> t[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const cx<A> u = W[a], x = h[0];
        cx<A> acc = mk<A>(MU % 2 == 0 ? fma(u.im, x.im, u.re * x.re) : fma(u.re, x.re, u.im * x.im),
                          fma(u.re, x.im, -(u.im * x.re)));
        cmacc(acc, W[3 + a], h[1]);
        cmacc(acc, W[6 + a], h[2]);
        t[a] = acc;
    }
}
// row_shl:4 (0x104: lane i reads lane i + 4 of its row) and row_shr:4 (0x114),
// zero from outside the row
template <int CTRL> __device__ __forceinline__ int shift_mov(int v)
{
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
template <int CTRL, typename A> __device__ __forceinline__ cx<A> row_shift(const cx<A> &v)
{
    if constexpr (sizeof(A) == 4) {
        return mk<A>(__int_as_float(shift_mov<CTRL>(__float_as_int(v.re))), __int_as_float(shift_mov<CTRL>(__float_as_int(v.im))));
    } else {
        const long long r = __double_as_longlong(v.re), i = __double_as_longlong(v.im);
        const int r0 = shift_mov<CTRL>((int)r), r1 = shift_mov<CTRL>((int)(r >> 32));
        const int i0 = shift_mov<CTRL>((int)i), i1 = shift_mov<CTRL>((int)(i >> 32));
        return mk<A>(__longlong_as_double(((long long)r1 << 32) | (unsigned)r0),
                     __longlong_as_double(((long long)i1 << 32) | (unsigned)i0));
    }
}

// ---- in-block hops of direction MU across the lanes of a wavefront.  With
// WRAP every hop is multiplied by its sign (one unless it wraps): a branch on
// whether the direction wraps saved those multiplications and made the code of
// an MR step twice as long, which cost more (4x16^3, FP32, eleven cycles of
// three steps: 501 -> 478 us; FP64 691 -> 658; 4x24^2x48 with twelve right-hand
// sides 2796 -> 2719; the operator 10.0 -> 9.5).
template <int MU, int SP, bool WRAP, typename A>
__device__ __forceinline__ void blk_hop_spin(const cx<A> W[9], const cx<A> u[6], const cx<A> l[6], cx<A> qu[6],
                                              cx<A> ql[6], bool inf, bool inb, int snf, int snb, A kf, A kb)
{
    cx<A> h[3], t[3];
    if constexpr (MU == 1 && !WRAP) {
        // y: a shift within the row of 16 lanes fills with zero where the
        // neighbour leaves the block, so every lane adds
        proj_spin<MU, -1, SP>(u, l, h);
#pragma unroll
        for (int c = 0; c < 3; ++c) t[c] = row_shift<0x104, A>(h[c]);
        su3_spin(W, t, h);
        recon_spin<MU, -1, SP, true>(qu, ql, h, kf);
        proj_spin<MU, +1, SP>(u, l, h);
        su3_spin_adj<MU>(W, h, t);
#pragma unroll
        for (int c = 0; c < 3; ++c) h[c] = row_shift<0x114, A>(t[c]);
        recon_spin<MU, +1, SP, true>(qu, ql, h, kb);
        return;
    }
    proj_spin<MU, -1, SP>(u, l, h);
#pragma unroll
    for (int c = 0; c < 3; ++c) t[c] = lane_hop<MU, +1, A>(h[c], snf);
    if (inf) {
        su3_spin(W, t, h);
        recon_spin<MU, -1, SP, !WRAP>(qu, ql, h, kf);
    }
    proj_spin<MU, +1, SP>(u, l, h);
    su3_spin_adj<MU>(W, h, t);
#pragma unroll
    for (int c = 0; c < 3; ++c) h[c] = lane_hop<MU, -1, A>(t[c], snb);
    if (inb) {
        recon_spin<MU, +1, SP, !WRAP>(qu, ql, h, kb);
    }
}
template <int MU, bool WRAP, typename A>
__device__ __forceinline__ void blk_hop(const Geom &g, int b, const int bc[4], int s, const cx<A> W[9],
                                         const cx<A> u[6], const cx<A> l[6], cx<A> qu[6], cx<A> ql[6])
{
    int bn, snf, snb, gf, gb;
    bool inf, inb;
    neighbour<MU, +1>(g, b, bc, s, bn, snf, gf, inf);
    neighbour<MU, -1>(g, b, bc, s, bn, snb, gb, inb);
    if (!WRAP) {
        inf = ((s >> (2 * MU)) & 3) < BEXT - 1;
        inb = ((s >> (2 * MU)) & 3) > 0;
    }
    blk_hop_spin<MU, 0, WRAP>(W, u, l, qu, ql, inf, inb, snf, snb, (A)gf, (A)gb);
    blk_hop_spin<MU, 1, WRAP>(W, u, l, qu, ql, inf, inb, snf, snb, (A)gf, (A)gb);
}

// ---- the t direction through LDS
template <int SP, typename LT, typename A>
__device__ __forceinline__ void blk_t_post_spin(LT &L, const cx<A> W[9], int s, const cx<A> u[6], const cx<A> l[6])
{
    cx<A> h[3], t[3];
    proj_spin<3, -1, SP>(u, l, h);
#pragma unroll
    for (int c = 0; c < 3; ++c) L.tf[3 * SP + c][s] = h[c];
    proj_spin<3, +1, SP>(u, l, h);
    su3_spin_adj<3>(W, h, t);
#pragma unroll
    for (int c = 0; c < 3; ++c) L.tb[3 * SP + c][s] = t[c];
}
template <int SP, bool WRAP, typename LT, typename A>
__device__ __forceinline__ void blk_t_take_spin(LT &L, const cx<A> W[9], cx<A> qu[6], cx<A> ql[6], bool inf,
                                                 bool inb, int snf, int snb, A kf, A kb)
{
    cx<A> h[3], t[3];
    if (inf) {
#pragma unroll
        for (int c = 0; c < 3; ++c) h[c] = L.tf[3 * SP + c][snf];
        su3_spin(W, h, t);
        recon_spin<3, -1, SP, !WRAP>(qu, ql, t, kf);
    }
    if (inb) {
#pragma unroll
        for (int c = 0; c < 3; ++c) h[c] = L.tb[3 * SP + c][snb];
        recon_spin<3, +1, SP, !WRAP>(qu, ql, h, kb);
    }
}

template <bool WRAP, typename LT, typename A>
__device__ __forceinline__ void blk_t_take(LT &L, const Geom &g, int b, const int bc[4], int s, const cx<A> W[9], cx<A> qu[6],
                                           cx<A> ql[6])
{
    int bn, snf, snb, gf, gb;
    bool inf, inb;
    neighbour<3, +1>(g, b, bc, s, bn, snf, gf, inf);
    neighbour<3, -1>(g, b, bc, s, bn, snb, gb, inb);
    if (!WRAP) {
        inf = s < 3 * 64;
        inb = s >= 64;
    }
    blk_t_take_spin<0, WRAP>(L, W, qu, ql, inf, inb, snf, snb, (A)gf, (A)gb);
    blk_t_take_spin<1, WRAP>(L, W, qu, ql, inf, inb, snf, snb, (A)gf, (A)gb);
}

// ---------------------------------------------------------------------------
// Face buffers of the Schwarz sweep.  A block that has just been solved
// publishes, for each of its boundary sites and a spinor p (its update delta
// in the plain sweep, its psi in the even-odd sweep and where the next visits of
// the plain one form their residual anew), the half spinor that
// the neighbouring block (of the other colour) needs for the hop into it:
//   face 2 mu     (sites with l_mu = 0): h = (1 - gamma_mu) p, projected,
//                 for the +mu hop of the block below, which applies its own
//                 link U_mu(x);
//   face 2 mu + 1 (sites with l_mu = 3): t = U~_mu(y)^+ (1 + gamma_mu) p,
//                 projected, with U~ = -U/2 the register-resident link, for
//                 the -mu hop of the block above.
// The consumer then reads six components per boundary hop, dense in a row of
// 64 face sites, instead of the neighbour's twelve (strided) and its link.
// Layout per block and right-hand side: [face 0..7][half-spinor comp. 0..5][64].
constexpr int FACE_ELEMS = 8 * 6 * 64; // = 12 * BS: one spinor's worth per block

// Position of site s in the face of direction mu (the other three
// coordinates, 2 bits each, in order).
__device__ __forceinline__ int face_index(int s, int mu)
{
    const int lo = s & ((1 << (2 * mu)) - 1);
    return lo | ((s >> (2 * mu + 2)) << (2 * mu));
}

// The hops that leave a block, computed cooperatively by the workgroup: the
// 8 faces x 64 sites of a 4^4 block are 512 hops, two per thread, with the
// face (and so mu and the direction) uniform over each wavefront: wavefront w
// takes face w (hop j = 0, mu = w/2) and face w + 4 (j = 1, mu = 2 + w/2),
// face 2 mu being the sites with l_mu = 0 (hop from x - mu) and face 2 mu + 1
// those with l_mu = 3.  Each hop's transported half spinor, times -1/2 and the
// boundary sign, goes to FB[j] at [component][face mod 4][64], i.e. at
// [component][thread]; after the caller's next barrier face_gather adds them
// to their sites.
struct FaceHop {
    int mu, dir;  // uniform over the wavefront
    bool inblk;   // the block spans the direction: the in-block exchange wraps (uniform)
    int bn, sn;   // the neighbour's block (uniform) and site
    int lb, ls;   // block and site whose link the hop takes
    int sign;
};
__device__ __forceinline__ FaceHop face_hop(const Geom &g, int b, const int bc[4], int tid, int j)
{
    FaceHop h;
    const int f = __builtin_amdgcn_readfirstlane(tid >> 6) + 4 * j, k = tid & 63;
    h.mu = f >> 1;
    h.dir = (f & 1) ? 1 : -1;
    // values, not addresses, are selected: an address into the argument block
    // or bc would put it in scratch memory
    const int n0 = g.nb[0], n1 = g.nb[1], n2 = g.nb[2], n3 = g.nb[3];
    const int s0 = g.bstride[0], s1 = g.bstride[1], s2 = g.bstride[2], s3 = g.bstride[3];
    const int p0 = g.bcs[0], p1 = g.bcs[1], p2 = g.bcs[2], p3 = g.bcs[3];
    const int c0 = bc[0], c1 = bc[1], c2 = bc[2], c3 = bc[3];
    const int mu = h.mu;
    const int nb = mu < 2 ? (mu == 0 ? n0 : n1) : (mu == 2 ? n2 : n3);
    const int st = mu < 2 ? (mu == 0 ? s0 : s1) : (mu == 2 ? s2 : s3);
    const int bs = mu < 2 ? (mu == 0 ? p0 : p1) : (mu == 2 ? p2 : p3);
    const int cm = mu < 2 ? (mu == 0 ? c0 : c1) : (mu == 2 ? c2 : c3);
    const int lo = k & ((1 << (2 * mu)) - 1), up = (k >> (2 * mu)) << (2 * mu + 2);
    const int x0 = lo | up, x3 = x0 | ((BEXT - 1) << (2 * mu)); // the face sites with l_mu = 0 and 3
    const int s = h.dir > 0 ? x3 : x0;
    h.sn = h.dir > 0 ? x0 : x3;
    h.inblk = nb == 1;
    const bool edge = h.dir > 0 ? cm + 1 == nb : cm == 0;
    h.bn = h.dir > 0 ? (edge ? b - (nb - 1) * st : b + st) : (edge ? b + (nb - 1) * st : b - st);
    h.sign = edge ? bs : 1;
    h.lb = h.dir > 0 ? b : h.bn;
    h.ls = h.dir > 0 ? s : h.sn;
    return h;
}
// The products of a face hop and the third row of its link, as explicit
// multiply-adds.  Which of two products a sum fuses is otherwise the compiler's
// choice and changes with the code around it, and the adaptive rounds of the
// two-level setup magnify a last bit of the FP32 residual (8^4, twelve vectors,
// two rounds: 1e-8 in the residual moves the interpolation by 6e-6).  Either
// choice is as good; the ones here, which differ by spin and by direction, are
// those that interpolations have been made with so far, and keep them what they
// were, bit for bit.  It costs no time.
template <typename A> __device__ __forceinline__ void face_mul(const cx<A> U[9], const cx<A> h[6], cx<A> out[6])
{
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const cx<A> u = U[a * 3], x = h[s * 3];
            cx<A> acc = mk<A>(fma(u.re, x.re, -(u.im * x.im)),
                              s == 0 ? fma(u.re, x.im, u.im * x.re) : fma(u.im, x.re, u.re * x.im));
            cmac(acc, U[a * 3 + 1], h[s * 3 + 1]);
            cmac(acc, U[a * 3 + 2], h[s * 3 + 2]);
            out[s * 3 + a] = acc;
        }
}
template <typename A> __device__ __forceinline__ void face_mul_adj(const cx<A> U[9], const cx<A> h[6], cx<A> out[6])
{
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const cx<A> u = U[a], x = h[s * 3];
            cx<A> acc = mk<A>(s == 0 ? fma(u.im, x.im, u.re * x.re) : fma(u.re, x.re, u.im * x.im),
                              fma(u.re, x.im, -(u.im * x.re)));
            cmacc(acc, U[3 + a], h[s * 3 + 1]);
            cmacc(acc, U[6 + a], h[s * 3 + 2]);
            out[s * 3 + a] = acc;
        }
}
// conj(a b - c d)
template <typename A> __device__ __forceinline__ cx<A> face_minor(cx<A> a, cx<A> b, cx<A> c, cx<A> d)
{
    return mk<A>(fma(a.re, b.re, -(a.im * b.im)) - fma(c.re, d.re, -(c.im * d.im)),
                 fma(c.im, d.re, c.re * d.im) - fma(a.im, b.re, a.re * b.im));
}
template <typename A> __device__ __forceinline__ void face_third_row(cx<A> U[9])
{
    U[6] = face_minor(U[1], U[5], U[2], U[4]);
    U[7] = face_minor(U[2], U[3], U[0], U[5]);
    U[8] = face_minor(U[0], U[4], U[1], U[3]);
}
// One such hop of the spinor p with the link W (as stored) to fb[component].
template <typename A>
__device__ __forceinline__ void face_hop_post(const FaceHop &f, const cx<A> p[12], const cx<A> W[9], int tid,
                                              cx<A> (*fb)[BS])
{
    cx<A> h[6], t[6];
    if (f.dir > 0) {
        proj_m(f.mu, p, h);
        face_mul(W, h, t);
    } else {
        proj_p(f.mu, p, h);
        face_mul_adj(W, h, t);
    }
    const A kk = (A)(-0.5f * f.sign);
#pragma unroll
    for (int c = 0; c < 6; ++c) fb[c][tid] = kk * t[c];
}

// q += the face hops of site s from the buffers FB0, FB1 that face_hop_post wrote.
template <int MU, typename A>
__device__ __forceinline__ void face_gather_dir(const Geom &g, int s, const cx<A> *FB0, const cx<A> *FB1,
                                                cx<A> q[12])
{
    if (g.nb[MU] == 1) return;
    const int l = (s >> (2 * MU)) & 3;
    if (l != 0 && l != BEXT - 1) return;
    const int f = 2 * MU + (l == 0 ? 0 : 1);
    const cx<A> *fb = (f < 4 ? FB0 : FB1) + (f & 3) * 64 + face_index(s, MU);
    cx<A> t[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) t[c] = fb[c * BS];
    if (l == 0) recon_plus1<MU>(q, t);
    else recon_minus1<MU>(q, t);
}
template <typename A>
__device__ __forceinline__ void face_gather(const Geom &g, int s, const cx<A> *FB0, const cx<A> *FB1, cx<A> q[12])
{
    face_gather_dir<0, A>(g, s, FB0, FB1, q);
    face_gather_dir<1, A>(g, s, FB0, FB1, q);
    face_gather_dir<2, A>(g, s, FB0, FB1, q);
    face_gather_dir<3, A>(g, s, FB0, FB1, q);
}

template <typename S, typename A>
__device__ __forceinline__ void face_publish(vec2_t<S> *__restrict__ F, int b, int nrhs, int r, int s,
                                             const cx<A> p[12], const cx<A> Ur[4][9])
{
    vec2_t<S> *base = F + ((long)b * nrhs + r) * FACE_ELEMS;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        const int l = (s >> (2 * mu)) & 3;
        cx<A> h[6], t[6];
        if (l == 0) {
            proj_m(mu, p, h);
            vec2_t<S> *fp = base + (2 * mu) * 6 * 64 + face_index(s, mu);
#pragma unroll
            for (int e = 0; e < 6; ++e) stc(fp + e * 64, h[e]);
        } else if (l == BEXT - 1) {
            proj_p(mu, p, h);
            su3_mul_adj(Ur[mu], h, t);
            vec2_t<S> *fp = base + (2 * mu + 1) * 6 * 64 + face_index(s, mu);
#pragma unroll
            for (int e = 0; e < 6; ++e) stc(fp + e * 64, t[e]);
        }
    }
}

// The boundary hops of site s from the faces the neighbouring blocks
// published, accumulated into q (one direction per trip: the register
// budget of the sweep has no room for more face data in flight).
template <typename S, typename A>
__device__ __forceinline__ void face_consume(const Geom &g, int b, const int bc[4], int s, int r, int nrhs,
                                             const vec2_t<S> *__restrict__ F, const cx<A> Ur[4][9], cx<A> q[12])
{
#pragma unroll 1
    for (int mu = 0; mu < 4; ++mu) {
        const int l = (s >> (2 * mu)) & 3;
        if (l != 0 && l != BEXT - 1) continue;
        const int dir = l == 0 ? -1 : 1;
        int bn, sn, sign;
        bool inb;
        neighbour_rt(g, b, bc, s, mu, dir, bn, sn, sign, inb);
        if (inb) continue;
        // the +mu face of the block below, or the -mu face of the block above
        const vec2_t<S> *fp =
            F + ((long)bn * nrhs + r) * FACE_ELEMS + (2 * mu + (dir < 0 ? 1 : 0)) * 6 * 64 + face_index(s, mu);
        cx<A> h[6], t[6], U[9];
#pragma unroll
        for (int e = 0; e < 6; ++e) h[e] = ldc<A>(fp + e * 64);
        // U~ and the published t carry -1/2: only the boundary sign remains
        if (dir > 0) {
            // explicit branches: a switch would become a dynamic register index
            if (mu == 0) { for (int e = 0; e < 9; ++e) U[e] = Ur[0][e]; }
            else if (mu == 1) { for (int e = 0; e < 9; ++e) U[e] = Ur[1][e]; }
            else if (mu == 2) { for (int e = 0; e < 9; ++e) U[e] = Ur[2][e]; }
            else { for (int e = 0; e < 9; ++e) U[e] = Ur[3][e]; }
            su3_mul(U, h, t);
            recon_m(mu, q, t, (A)sign);
        } else {
            recon_p(mu, q, h, (A)sign);
        }
    }
}

// One DPP step of the wavefront sum: v + (v moved by ctrl), with rows outside
// row_mask (and invalid source lanes) adding zero.
template <int CTRL, int ROWS> __device__ __forceinline__ float dpp_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, true));
}
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_add(double v)
{
    const long long x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), CTRL, ROWS, 0xf, true);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Sum over the 64 lanes of a wavefront in a fixed order, with cross-lane DPP
// moves (no LDS round trips): pairs, quads, half rows and rows of 16, then
// row 1 += row 0 and row 3 += row 2 (row_bcast:15), then rows 2-3 += the
// first half (row_bcast:31).  The total is valid in lane 63 only.
template <typename A> __device__ __forceinline__ A wave_sum(A v)
{
    v = dpp_add<0xB1, 0xf>(v);  // quad_perm [1,0,3,2]
    v = dpp_add<0x4E, 0xf>(v);  // quad_perm [2,3,0,1]
    v = dpp_add<0x141, 0xf>(v); // row_half_mirror
    v = dpp_add<0x140, 0xf>(v); // row_mirror
    v = dpp_add<0x142, 0xa>(v); // row_bcast:15
    v = dpp_add<0x143, 0xc>(v); // row_bcast:31
    return v;
}


} // namespace dd
