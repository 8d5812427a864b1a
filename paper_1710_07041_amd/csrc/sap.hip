// Red-black Schwarz alternating procedure (SAP) with block-local minimal
// residual (MR) solves -- the "MR inversion within a domain" and the "entire
// Schwarz method" whose per-core rates the paper reports (Sec. 3.1, Tables 1
// and 2); the algorithm is Luescher's multiplicative SAP (Comput. Phys.
// Commun. 156 (2004) 209) with Saad's MR iteration on each block.
//
// One launch sweeps every block of one colour.  One 256-thread workgroup owns
// one 4^4 block, one thread one site, and keeps everything the MR loop needs
// on chip (k_sap_sweep, sap_sweep.h):
//   * the site's four forward links (pre-multiplied by the hop factor -1/2)
//     and its clover term live in registers for the whole sweep and every
//     right-hand side (of a clover term that does not mirror itself, and in
//     FP64, half 1 is re-read at each block application and stays in L2); the
//     MR accumulator lives in LDS;
//   * D_BB is applied direction by direction: each thread provides the
//     spin-projected half spinor of its site for the +mu hop of site x-mu and
//     U_mu(x)^+ times the projected half spinor for the -mu hop of site x+mu,
//     across lanes of its wavefront for x, y, z (a wavefront is one t-slice)
//     and through LDS for t, so no spinor leaves the chip inside the MR loop;
//   * the two block dot products per MR step reduce with DPP sums within each
//     wavefront and a fixed-order combine of the four wavefronts
//     (deterministic).
// eta and psi go through the caches (they are re-read by the next sweep and
// by the operator that follows the smoother, and fit in the 256 MB
// last-level cache in FP32); links and clover, read once per sweep, stream.
// The block residual rho_B = eta_B - (D psi)_B is carried from visit to visit
// rather than recomputed.  Luescher's formulation of the procedure: after its
// MR steps a block stores its MR residual R_B, and the next visit forms
// rho_B = R_B - D_{B,dB} delta_dB, where delta_dB is the update that the
// neighbouring blocks of the other colour made in between (on the first
// visit R_B = eta_B).  The hops of delta arrive through face buffers that the
// other colour published at the end of its solves (block_ops.h: six dense
// components per boundary hop).  FP64 forms the residual anew from psi every
// eighth cycle, from faces of psi (FRESH, sap_sweep.h).
// Blocks of one colour share no site and read only the other colour's data,
// so a sweep needs no synchronisation between workgroups.
//
// k_sap_sweep_eo is the same sweep with the even-odd preconditioned block
// solve (MR on the even-site Schur complement, odd sites reconstructed);
// see the comment above it.
#include "block_ops.h"
#include "dd_device.h"
#include "dd_internal.h"
#include "sap_sweep.h"

namespace dd {

namespace {

// ---------------------------------------------------------------------------
// Even-odd preconditioned block solve (site parity p = (x+y+z+t) mod 2).  On
// block B, with A = (4 + m0) + C site-local and H the in-block hops,
//   S = A_ee - H_eo A_oo^-1 H_oe on the even sites,
//   y_o = A_oo^-1 rho_o,  r_e = rho_e - H_eo y_o,  nMR MR steps on S: with
//   w_o = A_oo^-1 H_oe r_e, q_e = A_ee r_e - H_eo w_o: delta_e += alpha r_e,
//   r_e -= alpha q_e, and delta_o = y_o - sum alpha w_o, which is
//   A_oo^-1 (rho_o - H_oe delta_e) without another exchange and solve.
// Each visit forms the block residual anew from the stored psi, so that what
// rounding psi left is taken out again by the next visit (a residual carried
// from visit to visit, one exchange less, let the rounding add up: FP32 at 8^4
// 1.87e-7 after twelve cycles and 2.19e-7 after 32, where this stays at 1.5e-7;
// 3.67 against 3.78 ms a call at 24^3x48).  It takes one exchange: with
// z_o = psi_o + y_o,
//   rho_o = eta_o - (hops from outside) - A_oo psi_o - H_oe psi_e,
//   r_e = eta_e - (hops from outside) - A_ee psi_e - H_eo z_o.
// Threads 0-127 (waves 0-1) own the even sites, threads 128-255 (waves 2-3)
// the odd ones, so every parity branch is uniform over a wavefront.  A hop
// exchange between the parities is pipelined: at stage k the publishing
// waves post direction k while the consuming waves take direction k-1 from
// the other LDS buffer.  A_oo^-1 is applied through the Cholesky factor of
// each chiral half (the halves are Hermitian positive definite: the clover
// term is small against 4 + m0).
// What bounds it: a chain of 2 + 2 nMR exchanges of five stages and four
// barriers each, with half the wavefronts idle in the first and last stage of
// each; so what counts are few exchanges and a second workgroup per CU to fill
// them (FP32 arithmetic).  24^3x48, twelve cycles, against a form that took
// 4 + 2 nMR (the odd sites from an exchange and a solve of their own) and ran
// one workgroup per CU: FP32 6.56 -> 3.78 ms a call, FP16 6.28 -> 3.49, FP64
// (one workgroup per CU still; 46 registers spilled) 11.9 -> 9.66.
// ---------------------------------------------------------------------------

// Site of thread t: the pair {2k, 2k+1} (k = t mod 128) holds one even and
// one odd site; which is which follows from (ly + lz + lt) mod 2.
__device__ __forceinline__ int eo_site(int t)
{
    const int k = t & 127, odd = t >> 7;
    const int bit = (((k >> 1) & 3) + ((k >> 3) & 3) + ((k >> 5) & 3)) & 1;
    return 2 * k + (bit ^ odd);
}

// Slot of the upper entry (j, i), j < i, of a packed Hermitian 6x6 half.
__host__ __device__ constexpr int hslot(int j, int i) { return 3 + j * 5 - j * (j - 1) / 2 + (i - j - 1); }

// In place: the packed half c, plus diag on the diagonal, becomes its
// Cholesky factor M = R^+ R (R upper triangular, real positive diagonal):
// slots 0-2 receive 1/R_jj in pairs, the slot of (j, i) receives R_ji.
template <typename A> __device__ __forceinline__ void chol_half(cx<A> c[18], A diag)
{
    A d[6] = {c[0].re + diag, c[0].im + diag, c[1].re + diag, c[1].im + diag, c[2].re + diag, c[2].im + diag};
    A inv[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        A t = d[j];
#pragma unroll
        for (int k = 0; k < j; ++k) {
            const cx<A> u = c[hslot(k, j)];
            t -= u.re * u.re + u.im * u.im;
        }
        inv[j] = (A)1 / sqrt(t);
#pragma unroll
        for (int i = j + 1; i < 6; ++i) {
            cx<A> acc = c[hslot(j, i)];
#pragma unroll
            for (int k = 0; k < j; ++k) {
                // acc -= conj(R_kj) R_ki
                const cx<A> a = c[hslot(k, j)], b2 = c[hslot(k, i)];
                acc.re -= a.re * b2.re + a.im * b2.im;
                acc.im -= a.re * b2.im - a.im * b2.re;
            }
            c[hslot(j, i)] = inv[j] * acc;
        }
    }
    c[0] = mk<A>(inv[0], inv[1]);
    c[1] = mk<A>(inv[2], inv[3]);
    c[2] = mk<A>(inv[4], inv[5]);
}

// x = M^-1 x in place from the factor written by chol_half: R^+ y = x, then
// R x = y.
template <typename A> __device__ __forceinline__ void chol_solve(const cx<A> f[18], cx<A> x[6])
{
    const A inv[6] = {f[0].re, f[0].im, f[1].re, f[1].im, f[2].re, f[2].im};
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        cx<A> acc = x[i];
#pragma unroll
        for (int k = 0; k < i; ++k) {
            // acc -= conj(R_ki) y_k
            const cx<A> a = f[hslot(k, i)];
            acc.re -= a.re * x[k].re + a.im * x[k].im;
            acc.im -= a.re * x[k].im - a.im * x[k].re;
        }
        x[i] = inv[i] * acc;
    }
#pragma unroll
    for (int i = 5; i >= 0; --i) {
        cx<A> acc = x[i];
#pragma unroll
        for (int k = i + 1; k < 6; ++k) acc = acc - f[hslot(i, k)] * x[k];
        x[i] = inv[i] * acc;
    }
}

// LDS of the even-odd sweep.  One parity posts at a time: the exchange buffers
// are indexed by the ordinal k = s / 2 of the posting site.
template <typename A> struct EoLds {
    cx<A> hf[2][6][BS / 2];
    cx<A> hb[2][6][BS / 2];
    cx<A> del[12][BS / 2]; // delta_e (by even ordinal)
    cx<A> f1[18][BS];      // chiral half 1 by thread: clover (even), Cholesky factor of A_oo (odd)
    A red[4][4];
};

// Post direction MU of v (this thread's site s) into buffer X.
template <int MU, typename A>
__device__ __forceinline__ void eo_publish(EoLds<A> &L, int X, int s, const cx<A> U[9], const cx<A> v[12])
{
    cx<A> h[6], t[6];
    const int k = s >> 1;
    proj_minus<MU>(v, h);
#pragma unroll
    for (int c = 0; c < 6; ++c) L.hf[X][c][k] = h[c];
    proj_plus<MU>(v, h);
    su3_mul_adj(U, h, t);
#pragma unroll
    for (int c = 0; c < 6; ++c) L.hb[X][c][k] = t[c];
}

// Take direction MU from buffer X: q += the two in-block hops of site s.
template <int MU, bool WRAP, typename A>
__device__ __forceinline__ void eo_consume(EoLds<A> &L, int X, const Geom &g, int b, const int bc[4], int s,
                                           const cx<A> U[9], cx<A> q[12])
{
    const bool wraps = WRAP && g.nb[MU] == 1; // uniform
    cx<A> h[6], t[6];
    int bn, sn, sign;
    bool inb;
    neighbour<MU, +1>(g, b, bc, s, bn, sn, sign, inb);
    if (!WRAP) inb = ((s >> (2 * MU)) & 3) < BEXT - 1;
    if (inb) {
#pragma unroll
        for (int c = 0; c < 6; ++c) h[c] = L.hf[X][c][sn >> 1];
        su3_mul(U, h, t);
        if (wraps) recon_minus<MU>(q, t, (A)sign);
        else recon_minus1<MU>(q, t);
    }
    neighbour<MU, -1>(g, b, bc, s, bn, sn, sign, inb);
    if (!WRAP) inb = ((s >> (2 * MU)) & 3) > 0;
    if (inb) {
#pragma unroll
        for (int c = 0; c < 6; ++c) t[c] = L.hb[X][c][sn >> 1];
        if (wraps) recon_plus<MU>(q, t, (A)sign);
        else recon_plus1<MU>(q, t);
    }
}

// q += H v across the parities: the waves with pub set post v, the others
// accumulate the hops into q.  Stage k posts direction k and takes direction
// k - 1 (the two LDS buffers alternate), one barrier per stage.  Buffer reuse
// is safe across consecutive calls: a buffer is rewritten only after a
// barrier that follows its last read.
template <bool WRAP, typename A>
__device__ __forceinline__ void eo_exchange(EoLds<A> &L, const Geom &g, int b, const int bc[4], int s,
                                            const cx<A> Ur[4][9], bool pub, const cx<A> v[12], cx<A> q[12])
{
    if (pub) eo_publish<0, A>(L, 0, s, Ur[0], v);
    __syncthreads();
    if (pub) eo_publish<1, A>(L, 1, s, Ur[1], v);
    else eo_consume<0, WRAP, A>(L, 0, g, b, bc, s, Ur[0], q);
    __syncthreads();
    if (pub) eo_publish<2, A>(L, 0, s, Ur[2], v);
    else eo_consume<1, WRAP, A>(L, 1, g, b, bc, s, Ur[1], q);
    __syncthreads();
    if (pub) eo_publish<3, A>(L, 1, s, Ur[3], v);
    else eo_consume<2, WRAP, A>(L, 0, g, b, bc, s, Ur[2], q);
    __syncthreads();
    if (!pub) eo_consume<3, WRAP, A>(L, 1, g, b, bc, s, Ur[3], q);
}

template <typename S, typename A, int WAVES, bool WRAP, bool SIG>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(WAVES))) void k_sap_sweep_eo(
    const vec2_t<S> *__restrict__ eta0, vec2_t<S> *__restrict__ psi0, const vec2_t<S> *__restrict__ links,
    const vec2_t<S> *__restrict__ clov, vec2_t<S> *__restrict__ faces, SArgs a)
{
    // FP32 at two workgroups per CU: no room for eta meanwhile, it is read again
    constexpr bool AGAIN = WAVES == 2 && sizeof(S) == 4;
    __shared__ EoLds<A> E;
    int b, rhs0, rhs1;
    if (!sweep_part(a, b, rhs0, rhs1)) return;
    const int tid = threadIdx.x, s = eo_site(tid), k = tid & (BS / 2 - 1);
    const bool odd = __builtin_amdgcn_readfirstlane(tid >> 7) != 0;
    const int lane = tid & 63, wave = tid >> 6;
    int bc[4];
    block_coords(a.g, b, bc);

    // register-resident links carry the hop factor -1/2
    cx<A> U[4][9];
    load_links4<A, true>(links + (long)b * 4 * 9 * BS + s, a.r12, (A)(-0.5), U);

    // no barrier between right-hand sides: every buffer is rewritten only
    // after a barrier that follows its last read (eo_exchange), or is each
    // thread's own
    for (int r = rhs0; r < rhs1; ++r) {
        if (a.active && !a.active[r]) continue; // uniform over the workgroup
        const A diag = (A)(4.0 + (a.m0_dev ? a.m0_dev[r] : a.m0[r]));
        const vec2_t<S> *__restrict__ eta = eta0 + (a.eta_off ? a.eta_off[r] : 0);
        vec2_t<S> *__restrict__ psi = psi0 + (a.psi_off ? a.psi_off[r] : 0);
        const long sp = ((long)b * a.nrhs + r) * 12 * BS + s;
        // the clover term's addresses are the same for every right-hand side:
        // hide that, or they leave the loop and spill
        int zero = 0;
        asm volatile("" : "+s"(zero));
        const vec2_t<S> *cp = clov + (long)b * 36 * BS + s + zero;

        // q = A psi of the site; the site's clover term (odd sites: the
        // Cholesky factors of A_oo) stays, half 0 in registers, half 1 in LDS
        cx<A> rr[12], q[12], cl[18];
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            q[c] = mk<A>(0, 0);
            rr[c] = a.mode == 2 ? ldc<A>(psi + sp + c * BS) : mk<A>(0, 0);
        }
        load_clover_half<A>(cp + 18 * BS, SIG, cl);
        if (a.mode == 2) clover_half_mac<A>(cl, diag, rr + 6, q + 6);
        if (odd) chol_half<A>(cl, diag);
#pragma unroll
        for (int e = 0; e < 18; ++e) E.f1[e][tid] = cl[e];
        load_clover_half<A>(cp, SIG, cl);
        if (a.mode == 2) clover_half_mac<A>(cl, diag, rr, q);
        if (odd) chol_half<A>(cl, diag);
        // odd: q = A_oo psi_o + H_oe psi_e
        if (a.mode == 2) eo_exchange<WRAP>(E, a.g, b, bc, s, U, !odd, rr, q);

        vec2_t<S> er[12];
#pragma unroll
        for (int c = 0; c < 12; ++c) er[c] = eta[sp + c * BS];
        if (a.mode != 0) face_consume<S, A>(a.g, b, bc, s, r, a.nrhs, faces, U, q);
        if (odd) {
            // rr = y_o, from here on delta_o; q = z_o
#pragma unroll
            for (int c = 0; c < 12; ++c) rr[c] = ldc<A>(&er[c]) - q[c];
            cx<A> f[18];
#pragma unroll
            for (int e = 0; e < 18; ++e) f[e] = E.f1[e][tid];
            chol_solve<A>(cl, rr);
            chol_solve<A>(f, rr + 6);
#pragma unroll
            for (int c = 0; c < 12; ++c) q[c] = a.mode == 2 ? rr[c] + ldc<A>(psi + sp + c * BS) : rr[c];
        }
        // even: rr = r_e
        if constexpr (AGAIN) asm volatile("" : "+s"(zero));
        eo_exchange<WRAP>(E, a.g, b, bc, s, U, odd, q, q);
        if (!odd) {
            if constexpr (AGAIN) {
#pragma unroll
                for (int c = 0; c < 12; ++c) er[c] = eta[sp + zero + c * BS];
            }
#pragma unroll
            for (int c = 0; c < 12; ++c) rr[c] = ldc<A>(&er[c]) - q[c];
        }

        int it = 0;
        for (; it < a.nmr; ++it) {
            // odd: q = H_oe r_e
#pragma unroll
            for (int c = 0; c < 12; ++c) q[c] = mk<A>(0, 0);
            eo_exchange<WRAP>(E, a.g, b, bc, s, U, !odd, rr, q);
            cx<A> f[18];
#pragma unroll
            for (int e = 0; e < 18; ++e) f[e] = E.f1[e][tid];
            if (odd) {
                // q = -w_o
                chol_solve<A>(cl, q);
                chol_solve<A>(f, q + 6);
#pragma unroll
                for (int c = 0; c < 12; ++c) q[c] = mk<A>(-q[c].re, -q[c].im);
            } else {
                // q = A_ee r_e
                clover_half_mac<A>(cl, diag, rr, q);
                clover_half_mac<A>(f, diag, rr + 6, q + 6);
            }
            // even: q = A_ee r_e - H_eo w_o = S r_e
            eo_exchange<WRAP>(E, a.g, b, bc, s, U, odd, q, q);
            cx<A> alpha;
            if (!mr_alpha(E, lane, wave, q, rr, alpha, !odd)) break;
            if (odd) {
#pragma unroll
                for (int c = 0; c < 12; ++c) cmac(rr[c], alpha, q[c]);
            } else {
#pragma unroll
                for (int c = 0; c < 12; ++c) {
                    cx<A> d = mk<A>(0, 0);
                    if (it > 0) d = E.del[c][k];
                    cmac(d, alpha, rr[c]);
                    E.del[c][k] = d;
                    rr[c] = rr[c] - alpha * q[c];
                }
            }
        }

        // psi_B += delta and, for the other colour, its faces as stored
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            cx<A> v = rr[c];
            if (!odd) v = it > 0 ? E.del[c][k] : mk<A>(0, 0);
            if (a.mode == 2) v = v + ldc<A>(psi + sp + c * BS);
            vec2_t<S> st;
            stc(&st, v);
            psi[sp + c * BS] = st;
            rr[c] = ldc<A>(&st);
        }
        if (a.publish) face_publish<S, A>(faces, b, a.nrhs, r, s, rr, U);
    }
}

// Algorithmic traffic of one colour sweep: links + clover once (72 reals per
// site each, also when compressed: the method's volume), eta or the carried
// residual, psi (read only when nonzero), psi written and, in the plain form,
// the residual carried to the next visit.
double sweep_bytes(const SArgs &a, size_t field_bytes, size_t spinor_bytes, bool carry)
{
    return 256.0 * a.nblk *
           (144.0 * field_bytes + a.nrhs * (double)spinor_bytes *
                                      (48.0 + (a.mode == 2 ? 24.0 : 0.0) + (carry && a.write_r ? 24.0 : 0.0)));
}

// WAVES wavefronts per SIMD: that many four-wavefront workgroups per CU.
template <typename S, typename A, typename SF, int WAVES>
Status sweep(dd_ctx *ctx, SArgs a, int prec, const void *eta, void *psi, void *faces, void *resid, bool quiet)
{
    const int fprec = sizeof(SF) == 8 ? DD_F64 : (sizeof(SF) == 4 ? DD_F32 : DD_F16);
    const int cls = prec == DD_F64 ? K_SAP_F64 : prec == DD_F32 ? K_SAP_F32 : K_SAP_F16;
    ProfScope ps(ctx->prof, ctx->stream, cls, sweep_bytes(a, sizeof(SF), sizeof(S), true),
                 256.0 * a.nblk * a.nrhs * (a.nmr * 2184.0 + (a.fresh ? 1848.0 : 0.0)), !quiet);
    a.rpg = rhs_per_group(a.nblk, a.nrhs, ctx->ncu * WAVES);
    // a direction that one block spans wraps inside it
    const bool wrap = a.g.nb[0] == 1 || a.g.nb[1] == 1 || a.g.nb[2] == 1 || a.g.nb[3] == 1;
    auto kernel = wrap ? (a.sig ? k_sap_sweep<S, A, SF, WAVES, true, true> : k_sap_sweep<S, A, SF, WAVES, true, false>)
                       : (a.sig ? k_sap_sweep<S, A, SF, WAVES, false, true> : k_sap_sweep<S, A, SF, WAVES, false, false>);
    kernel<<<dim3(a.nblk, (a.nrhs + a.rpg - 1) / a.rpg), BS, 0, ctx->stream>>>(
        static_cast<const vec2_t<S> *>(eta), static_cast<vec2_t<S> *>(psi),
        static_cast<const vec2_t<SF> *>(ctx->links[fprec].p), static_cast<const vec2_t<SF> *>(ctx->clover[fprec].p),
        static_cast<vec2_t<S> *>(faces), static_cast<vec2_t<S> *>(resid), a);
    DD_HIP_TRY(hipGetLastError());
    return Status::ok();
}

template <typename S, typename A, int WAVES>
Status sweep_eo(dd_ctx *ctx, SArgs a, int prec, const void *eta, void *psi, void *faces, bool quiet)
{
    // the block residual costs one operator application when psi_B != 0; the
    // right-hand side and the odd reconstruction one in-block hop application
    // per block solve
    const double fl = 256.0 * a.nblk * a.nrhs * (a.nmr * 2184.0 + (a.mode == 2 ? 1848.0 : 0.0) + 1848.0);
    const int cls = prec == DD_F64 ? K_SAP_EO_F64 : prec == DD_F32 ? K_SAP_EO_F32 : K_SAP_EO_F16;
    ProfScope ps(ctx->prof, ctx->stream, cls, sweep_bytes(a, sizeof(S), sizeof(S), false), fl, !quiet);
    a.rpg = rhs_per_group(a.nblk, a.nrhs, ctx->ncu * WAVES);
    const bool wrap = a.g.nb[0] == 1 || a.g.nb[1] == 1 || a.g.nb[2] == 1 || a.g.nb[3] == 1;
    // the form with wrap tests spills at two workgroups per CU: where there is
    // at most one, its wavefronts have all registers (4x8x16x16, FP16, one
    // right-hand side: 1089 -> 1043 us a call of twelve cycles)
    const bool lone = (long)a.nblk * ((a.nrhs + a.rpg - 1) / a.rpg) <= ctx->ncu;
    auto kernel = !wrap ? (a.sig ? k_sap_sweep_eo<S, A, WAVES, false, true> : k_sap_sweep_eo<S, A, WAVES, false, false>)
                  : lone ? (a.sig ? k_sap_sweep_eo<S, A, 1, true, true> : k_sap_sweep_eo<S, A, 1, true, false>)
                         : (a.sig ? k_sap_sweep_eo<S, A, WAVES, true, true> : k_sap_sweep_eo<S, A, WAVES, true, false>);
    kernel<<<dim3(a.nblk, (a.nrhs + a.rpg - 1) / a.rpg), BS, 0, ctx->stream>>>(
        static_cast<const vec2_t<S> *>(eta), static_cast<vec2_t<S> *>(psi),
        static_cast<const vec2_t<S> *>(ctx->links[prec].p), static_cast<const vec2_t<S> *>(ctx->clover[prec].p),
        static_cast<vec2_t<S> *>(faces), a);
    DD_HIP_TRY(hipGetLastError());
    return Status::ok();
}

} // namespace

size_t sap_scratch_bytes(const GeomHost &g, int prec, int nrhs)
{
    // face buffers (FACE_ELEMS = 12 * BS per block and rhs) and the carried
    // block residual: one spinor each
    return 2 * spinor_bytes(g, prec, nrhs);
}

Status reserve_sap_scratch(dd_ctx *ctx, int prec, int nrhs)
{
    const size_t need = sap_scratch_bytes(ctx->g, prec, nrhs);
    if (ctx->sap_scratch.p && ctx->sap_scratch.bytes >= need) return Status::ok();
    return ctx->sap_scratch.alloc(need);
}

Status run_sap(dd_ctx *ctx, const double *m0, int nrhs, const void *eta, void *psi, int ncy, int nmr, int prec,
               const SapSlots *slots, bool eo)
{
    if (!eta || !psi || !ctx->links[prec].p || !ctx->clover[prec].p || (!m0 && !(slots && slots->m0_dev)))
        return Status{DD_INVALID_ARG, "SAP: missing buffer"};
    // FP16 links and clover under the plain FP32 sweep (the even-odd sweep
    // keeps its own precision's fields)
    const bool half_fields = prec == DD_F32 && !eo && ctx->sap_half_fields;
    if (half_fields && (!ctx->links[DD_F16].p || !ctx->clover[DD_F16].p))
        return Status{DD_INVALID_ARG, "SAP: missing FP16 fields"};
    if (ncy == 0) {
        if (slots) return Status{DD_INVALID_ARG, "SAP: zero cycles with per-slot offsets"};
        DD_HIP_TRY(hipMemsetAsync(psi, 0, spinor_bytes(ctx->g, prec, nrhs), ctx->stream));
        return Status::ok();
    }
    SArgs a{};
    for (int k = 0; k < 4; ++k) {
        a.g.nb[k] = ctx->g.nb[k];
        a.g.bstride[k] = ctx->g.bstride[k];
        a.g.bcs[k] = ctx->g.bcs[k];
    }
    a.g.nblocks = ctx->g.nblocks;
    a.nrhs = nrhs;
    a.nmr = nmr;
    a.r12 = ctx->link_r12 ? 1 : 0;
    a.sig = ctx->clover_sigma ? 1 : 0;
    for (int r = 0; r < nrhs && m0; ++r) a.m0[r] = m0[r];
    if (slots) {
        a.m0_dev = slots->m0_dev;
        a.eta_off = slots->eta_off;
        a.psi_off = slots->psi_off;
        a.active = slots->active;
    }
    // face buffers and carried residual: the caller's scratch, else the context's
    void *scratch = slots ? slots->scratch : nullptr;
    if (!scratch) {
        DD_TRY(reserve_sap_scratch(ctx, prec, nrhs));
        scratch = ctx->sap_scratch.p;
    }
    if (!scratch) return Status{DD_INVALID_ARG, "SAP: no scratch buffer"};
    void *faces = scratch;
    void *resid = static_cast<char *>(scratch) + spinor_bytes(ctx->g, prec, nrhs);
    const bool quiet = slots && slots->quiet;
    TraceRange tr(eo ? "sap_eo" : "sap");
    // the visits of cycle cy form their residual anew: the faces they read are psi's
    const auto fresh = [&](int cy) { return prec == DD_F64 && !eo && cy > 0 && cy % FRESH_EVERY == 0; };
    for (int cy = 0; cy < ncy; ++cy)
        for (int col = 0; col < 2; ++col) {
            if (ctx->ncolour[col] == 0) continue;
            a.blocks = ctx->colour_blocks[col].as<int>();
            a.nblk = ctx->ncolour[col];
            a.mode = (cy == 0 && col == 0) ? 0 : (cy == 0 ? 1 : 2);
            a.publish = !(cy == ncy - 1 && col == 1);
            a.write_r = cy < ncy - 1 && !fresh(cy + 1);
            a.fresh = fresh(cy);
            a.psi_faces = fresh(col == 0 ? cy : cy + 1);
            if (eo) {
                DD_TRY((prec == DD_F64   ? sweep_eo<double, double, 1>(ctx, a, prec, eta, psi, faces, quiet)
                        : prec == DD_F32 ? sweep_eo<float, float, 2>(ctx, a, prec, eta, psi, faces, quiet)
                                         : sweep_eo<__half, float, 2>(ctx, a, prec, eta, psi, faces, quiet)));
            } else {
                DD_TRY((prec == DD_F64   ? sweep<double, double, double, 1>(ctx, a, prec, eta, psi, faces, resid, quiet)
                        : prec == DD_F16 ? sweep<__half, float, __half, 2>(ctx, a, prec, eta, psi, faces, resid, quiet)
                        : half_fields    ? sweep<float, float, __half, 2>(ctx, a, prec, eta, psi, faces, resid, quiet)
                                         : sweep<float, float, float, 2>(ctx, a, prec, eta, psi, faces, resid, quiet)));
            }
        }
    return Status::ok();
}

} // namespace dd
