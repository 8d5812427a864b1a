// Two-level coarse correction of DD-alpha-AMG on the GPU: the multigrid
// level the paper's solver puts above the Schwarz smoother (Sec. 1 names the
// method, Sec. 2.1 the smoother as its fine grid, Sec. 5 its coarse grid).
// The method is the published one (Frommer, Kahl, Krieg, Leder, Rottmann,
// SIAM J. Sci. Comput. 36 (2014) A1581):
//   * aggregates: each 4^4 Schwarz block split into its two chiral halves
//     (spins 0-1, spins 2-3), so the interpolation commutes with gamma_5;
//   * interpolation P: N test vectors restricted to every aggregate and
//     orthonormalised there by Gram-Schmidt in their order (P^+ P = 1);
//   * test vectors: inverse iteration with the Schwarz smoother from N
//     starting vectors, optionally refined by rounds of the two-grid method;
//   * coarse operator D_c = P^+ D P: a nearest-neighbour stencil on the
//     lattice of blocks with 2N unknowns per block, nine dense 2N x 2N
//     matrices per block (the block itself and its eight neighbours), built
//     at m0 = 0 -- because P^+ P = 1 the mass enters as + m0 at apply time,
//     so one coarse operator serves every mass;
//   * coarse solve: k steps of GMRES from zero (the least-residual vector of
//     the Krylov space), run entirely on the device for every right-hand
//     side at once (no host round trip, so the preconditioner can be
//     captured in a graph);
//   * two-grid preconditioner: psi_0 = P x_c with x_c the coarse solve of
//     D_c x_c = P^+ eta, then psi = psi_0 + SAP_nu(eta - D psi_0).
//
// Layouts (complex numbers as (re, im) pairs):
//   P      [block][chiral half c][vector i][component 0..5][site 0..255],
//          component = (spin - 2c) * 3 + colour; FP64 master, FP32 copy;
//   D_c    [block][d][column k'][row k], d = 0 the block itself, 1 + 2 mu
//          the +mu neighbour, 2 + 2 mu the -mu neighbour; row/column index
//          k = c * N + i; FP64 master, FP16 copy read by the coarse solve
//          (the coarse system is solved only approximately, and its nine
//          blocks per row are the largest array the solve streams);
//   coarse vectors [slot][block][k], FP64.
// Everything a block or a coarse site reduces is summed in a fixed order
// (DPP within a wavefront, then the wavefronts in order), so results are
// deterministic.
#include <algorithm>
#include <cmath>

#include "block_ops.h"
#include "dd_device.h"
#include "dd_internal.h"

namespace dd {

namespace {

constexpr int NMAX = 16;  // test vectors
constexpr int CK = 32;    // largest coarse GMRES step count
constexpr int CTPB = 256; // threads per coarse workgroup
constexpr int CG = 256;   // workgroups of the coarse reductions (grid-stride; one partial sum each)

// ---------------------------------------------------------------------------
// block reductions: the wavefront sum of each value lands in lane 63, the
// four wavefronts are added in order through LDS
// ---------------------------------------------------------------------------
struct Red {
    double v[4][2 * NMAX][2];
};

__device__ __forceinline__ void wave_put(Red &R, int lane, int wave, int slot, double re, double im)
{
    re = wave_sum(re);
    im = wave_sum(im);
    if (lane == 63) {
        R.v[wave][slot][0] = re;
        R.v[wave][slot][1] = im;
    }
}

__device__ __forceinline__ cx<double> wave_get(const Red &R, int slot)
{
    return mk<double>(((R.v[0][slot][0] + R.v[1][slot][0]) + R.v[2][slot][0]) + R.v[3][slot][0],
                      ((R.v[0][slot][1] + R.v[1][slot][1]) + R.v[2][slot][1]) + R.v[3][slot][1]);
}

__device__ __forceinline__ long pidx(int b, int c, int i, int N, int comp, int s)
{
    return ((((long)b * 2 + c) * N + i) * 6 + comp) * BS + s;
}

// ---------------------------------------------------------------------------
// interpolation: Gram-Schmidt of the test vectors on every aggregate
// ---------------------------------------------------------------------------
// tv: N test vectors in the blocked FP64 layout with N right-hand sides.
__global__ __launch_bounds__(BS) void k_amg_gs(const double2 *__restrict__ tv, double2 *__restrict__ Pd,
                                               float2 *__restrict__ Pf, int N)
{
    __shared__ Red R;
    const int b = blockIdx.x, c = blockIdx.y, s = threadIdx.x, lane = s & 63, wave = s >> 6;
    for (int i = 0; i < N; ++i) {
        cx<double> w[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) w[k] = ldc<double>(tv + (((long)b * N + i) * 12 + 6 * c + k) * BS + s);
        for (int j = 0; j < i; ++j) {
            cx<double> q[6];
            double re = 0, im = 0;
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                q[k] = ldc<double>(Pd + pidx(b, c, j, N, k, s));
                re += q[k].re * w[k].re + q[k].im * w[k].im;
                im += q[k].re * w[k].im - q[k].im * w[k].re;
            }
            wave_put(R, lane, wave, 0, re, im);
            __syncthreads();
            const cx<double> h = wave_get(R, 0);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 6; ++k) w[k] = w[k] - h * q[k];
        }
        double n2 = 0;
#pragma unroll
        for (int k = 0; k < 6; ++k) n2 += w[k].re * w[k].re + w[k].im * w[k].im;
        wave_put(R, lane, wave, 0, n2, 0.0);
        __syncthreads();
        // a piece that vanishes on the aggregate (dependent vectors) gives a
        // zero column instead of NaN
        const double nn = wave_get(R, 0).re;
        const double inv = nn > 0 ? 1.0 / sqrt(nn) : 0.0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const cx<double> p = inv * w[k];
            stc(Pd + pidx(b, c, i, N, k, s), p);
            stc(Pf + pidx(b, c, i, N, k, s), p);
        }
    }
}

// ---------------------------------------------------------------------------
// coarse operator: D_c[b][d][k'][k] = <P_{b,k}, (D P_{nbr_d(b),k'})|_b> at m0 = 0
// ---------------------------------------------------------------------------
struct AGeom {
    Geom g;
    int N;
    int r12;
};

// one hop into site s of block b from (bn, sn): forward (dir > 0) applies
// -1/2 (1 - g_mu) U_mu(x), backward -1/2 (1 + g_mu) U_mu(x - mu)^+, both
// times the boundary sign
__device__ __forceinline__ void hop_into(const double2 *__restrict__ links, bool r12, int b, int s, int bn, int sn,
                                         int mu, int dir, int sign, const cx<double> p[12], cx<double> q[12])
{
    cx<double> U[9], h[6], t[6];
    const double kk = sign > 0 ? -0.5 : 0.5;
    if (dir > 0) {
        load_link<double>(links + ((long)b * 4 + mu) * 9 * BS + s, r12, U);
        proj_m(mu, p, h);
        su3_mul(U, h, t);
        recon_m(mu, q, t, kk);
    } else {
        load_link<double>(links + ((long)bn * 4 + mu) * 9 * BS + sn, r12, U);
        proj_p(mu, p, h);
        su3_mul_adj(U, h, t);
        recon_p(mu, q, t, kk);
    }
}

__device__ __forceinline__ void load_col(const double2 *__restrict__ Pd, int b, int kp, int N, int s, cx<double> p[12])
{
    const int c = kp / N, i = kp % N;
#pragma unroll
    for (int k = 0; k < 12; ++k) p[k] = mk<double>(0, 0);
    // explicit halves: a run-time index into p would put it in scratch memory
    if (c == 0) {
#pragma unroll
        for (int k = 0; k < 6; ++k) p[k] = ldc<double>(Pd + pidx(b, 0, i, N, k, s));
    } else {
#pragma unroll
        for (int k = 0; k < 6; ++k) p[6 + k] = ldc<double>(Pd + pidx(b, 1, i, N, k, s));
    }
}

__global__ __launch_bounds__(BS) void k_amg_build(const double2 *__restrict__ Pd, const double2 *__restrict__ links,
                                                  const double2 *__restrict__ clov, double2 *__restrict__ Ad,
                                                  __half2 *__restrict__ Ah, AGeom a)
{
    __shared__ Red R;
    const int b = blockIdx.x, d = blockIdx.y, s = threadIdx.x, lane = s & 63, wave = s >> 6;
    const int N = a.N, N2 = 2 * N;
    int bc[4];
    block_coords(a.g, b, bc);
    const int mu = d == 0 ? 0 : (d - 1) >> 1, dir = (d - 1) & 1 ? -1 : 1;
    // the source block of this matrix
    int src = b;
    if (d > 0) {
        if (a.g.nb[mu] == 1) {
            // all hops of this direction stay in the block: counted in d = 0
            for (int e = s; e < N2 * N2; e += BS) {
                Ad[((long)b * 9 + d) * N2 * N2 + e] = make_double2(0, 0);
                Ah[((long)b * 9 + d) * N2 * N2 + e] = __floats2half2_rn(0.f, 0.f);
            }
            return;
        }
        const int up = bc[mu] + 1 == a.g.nb[mu] ? -(a.g.nb[mu] - 1) : 1;
        const int dn = bc[mu] == 0 ? a.g.nb[mu] - 1 : -1;
        src = b + (dir > 0 ? up : dn) * a.g.bstride[mu];
    }
    // this site's P rows for the dot products are re-read per column (L2)
    for (int kp = 0; kp < N2; ++kp) {
        cx<double> q[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) q[k] = mk<double>(0, 0);
        if (d == 0) {
            cx<double> p[12];
            load_col(Pd, b, kp, N, s, p);
            // (4 + C(x)) p(x): the mass is added at apply time
#pragma unroll 1
            for (int h = 0; h < 2; ++h) {
                cx<double> cl[18];
#pragma unroll
                for (int e = 0; e < 18; ++e) cl[e] = ldc<double>(clov + ((long)b * 36 + 18 * h + e) * BS + s);
                clover_half_mac<double>(cl, 4.0, p + 6 * h, q + 6 * h);
            }
            // hops whose neighbour lies in the block (with the boundary sign
            // when the block spans the whole direction)
#pragma unroll 1
            for (int m = 0; m < 4; ++m)
#pragma unroll 1
                for (int dr = -1; dr <= 1; dr += 2) {
                    int bn, sn, sign;
                    bool inb;
                    neighbour_rt(a.g, b, bc, s, m, dr, bn, sn, sign, inb);
                    if (!inb) continue;
                    cx<double> pn[12];
                    load_col(Pd, b, kp, N, sn, pn);
                    hop_into(links, a.r12, b, s, bn, sn, m, dr, sign, pn, q);
                }
        } else {
            int bn, sn, sign;
            bool inb;
            neighbour_rt(a.g, b, bc, s, mu, dir, bn, sn, sign, inb);
            if (!inb && bn == src) {
                cx<double> pn[12];
                load_col(Pd, src, kp, N, sn, pn);
                hop_into(links, a.r12, b, s, bn, sn, mu, dir, sign, pn, q);
            }
        }
        // entries (k, kp) for every row k = c * N + i
#pragma unroll
        for (int c = 0; c < 2; ++c)
            for (int i = 0; i < N; ++i) {
                double re = 0, im = 0;
#pragma unroll
                for (int e = 0; e < 6; ++e) {
                    const cx<double> pk = ldc<double>(Pd + pidx(b, c, i, N, e, s));
                    const cx<double> qe = q[6 * c + e];
                    re += pk.re * qe.re + pk.im * qe.im;
                    im += pk.re * qe.im - pk.im * qe.re;
                }
                wave_put(R, lane, wave, c * N + i, re, im);
            }
        __syncthreads();
        if (s < N2) {
            const cx<double> v = wave_get(R, s);
            const long o = (((long)b * 9 + d) * N2 + kp) * N2 + s;
            stc(Ad + o, v);
            stc(Ah + o, v);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// restriction x_c = P^+ eta and prolongation psi = P x_c (W slots; a slot's
// fine data at base + off[r] in the blocked layout with W right-hand sides)
// ---------------------------------------------------------------------------
// FP64 data are restricted and prolongated with the FP64 interpolation in
// FP64 arithmetic, FP32 data with the FP32 copy in FP32 arithmetic.
//
// Bound by reading P (N spinors a block, 764 MB in FP32 at 24^3x48 and N = 12).
// A thread takes two sites of one chiral half, neighbours in FP32 so that P comes
// in 16-byte loads, and RR right-hand sides, which share them; FP32 takes two
// vectors at a time and FP64, short of registers, one (two workgroups per CU with
// RR = 2 instead of one), the next in flight meanwhile.  The groups of a block's
// right-hand sides follow each other on one XCD and share its L2 (transfer_part).
// Restriction / prolongation in us, P read for each right-hand side anew, then in
// groups at a grid's length from each other, now: 24^3x48 FP32 with three
// 416 / 511, 160 / 175, 161 / 175, with five 703 / 852, 300 / 370, 287 / 257;
// FP64 with three 849 / 1018, 591 / 697, 340 / 378, with five 1396 / 1679,
// 886 / 1048, 434 / 446; 16^4 FP64 with three 49 / 42, 62 / 65, 41 / 40; 8^4 FP32
// with twelve 22 / 19, 26 / 22, 19 / 18.  One right-hand side: 24^3x48 FP32 159 /
// 182, now 140 / 160; 16^3x32 37 / 36, now 39 / 37.
template <typename S> using PT = vec2_t<S>;
template <typename S> struct alignas(16) Pair {
    vec2_t<S> e[2];
};
// the two sites of thread h (0..127) of a chiral half
template <typename S> __device__ __forceinline__ int pair_site(int h, int k) { return sizeof(S) == 4 ? 2 * h + k : h + (BS / 2) * k; }
// right-hand sides that share a read of P, as many as registers hold (a group
// past the last repeats the last one's reads: 24^3x48 FP32, three 161 us, four 168)
template <typename S> constexpr int rr_max() { return sizeof(S) == 4 ? 4 : 2; }
// vectors taken at a time
template <typename S> constexpr int PU = sizeof(S) == 4 ? 2 : 1;

// six components of a vector at the thread's two sites
template <typename S, bool NT> __device__ __forceinline__ void load_p(const PT<S> *__restrict__ p, int h, Pair<S> q[6])
{
#pragma unroll
    for (int x = 0; x < 6; ++x) {
        if constexpr (sizeof(S) == 4 && !NT) {
            q[x] = *reinterpret_cast<const Pair<S> *>(p + x * BS + 2 * h);
        } else {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const PT<S> *e = p + x * BS + pair_site<S>(h, k);
                q[x].e[k] = NT ? ld_stream(e) : *e;
            }
        }
    }
}

// The block and the group of right-hand sides of this workgroup.  The groups of
// a block follow each other on one XCD (workgroups go to the XCDs in turn), so
// the block's P comes from its L2 for all but the first.  False past the last
// block (the launch rounds them up to whole turns).
constexpr int NXCD = 8;
__device__ __forceinline__ bool transfer_part(int nblocks, int ngroups, int &b, int &grp)
{
    const int t = blockIdx.x / NXCD;
    grp = t % ngroups;
    b = t / ngroups * NXCD + blockIdx.x % NXCD;
    return b < nblocks;
}

template <typename S, int RR, bool NT>
__global__ __launch_bounds__(BS) void k_amg_restrict(const vec2_t<S> *__restrict__ in, const PT<S> *__restrict__ P,
                                                     double2 *__restrict__ xc, const int *__restrict__ active, int N,
                                                     int nblocks, int W)
{
    __shared__ double part[4][RR][NMAX][2];
    int b, grp;
    if (!transfer_part(nblocks, (W + RR - 1) / RR, b, grp)) return;
    const int r0 = grp * RR, s = threadIdx.x, lane = s & 63;
    const int wave = __builtin_amdgcn_readfirstlane(s >> 6), c = wave >> 1, h = s & 127;
    bool on = false;
#pragma unroll
    for (int rr = 0; rr < RR; ++rr) on |= r0 + rr < W && (!active || active[r0 + rr]);
    if (!on) return; // uniform
    const PT<S> *p = P + pidx(b, c, 0, N, 0, 0);
    constexpr int U = PU<S>;
    Pair<S> q[U][6], qn[U][6];
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u < N) load_p<S, NT>(p + u * 6 * BS, h, q[u]);
    cx<S> v[RR][6][2];
#pragma unroll
    for (int rr = 0; rr < RR; ++rr) {
        // a slot past the last repeats the last; its sums are not stored
        const vec2_t<S> *e = in + ((long)b * W + min(r0 + rr, W - 1)) * 12 * BS + 6 * c * BS;
#pragma unroll
        for (int x = 0; x < 6; ++x)
#pragma unroll
            for (int k = 0; k < 2; ++k) v[rr][x][k] = ldc<S>(e + x * BS + pair_site<S>(h, k));
    }
#pragma unroll 1
    for (int i = 0; i < N; i += U) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + U + u < N) load_p<S, NT>(p + (long)(i + U + u) * 6 * BS, h, qn[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i + u < N) {
#pragma unroll
                for (int rr = 0; rr < RR; ++rr) {
                    S re[2] = {0, 0}, im[2] = {0, 0}; // a site's sum in S, all further in FP64
#pragma unroll
                    for (int x = 0; x < 6; ++x)
#pragma unroll
                        for (int k = 0; k < 2; ++k) {
                            const cx<S> a = ldc<S>(&q[u][x].e[k]), f = v[rr][x][k];
                            re[k] = fma(a.re, f.re, fma(a.im, f.im, re[k]));
                            im[k] = fma(a.re, f.im, fma(-a.im, f.re, im[k]));
                        }
                    const double tre = wave_sum((double)re[0] + (double)re[1]), tim = wave_sum((double)im[0] + (double)im[1]);
                    if (lane == 63) {
                        part[wave][rr][i + u][0] = tre;
                        part[wave][rr][i + u][1] = tim;
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int x = 0; x < 6; ++x) q[u][x] = qn[u][x];
    }
    __syncthreads();
    if (s < 2 * N * RR) {
        const int rr = s / (2 * N), k = s - rr * 2 * N, cc = k / N, i = k - cc * N, r = r0 + rr;
        if (r < W && (!active || active[r]))
            stc(xc + ((long)r * nblocks + b) * 2 * N + k,
                mk<double>(part[2 * cc][rr][i][0] + part[2 * cc + 1][rr][i][0],
                           part[2 * cc][rr][i][1] + part[2 * cc + 1][rr][i][1]));
    }
}

template <typename S, int RR, bool NT>
__global__ __launch_bounds__(BS) void k_amg_prolong(const double2 *__restrict__ xc, const PT<S> *__restrict__ P,
                                                    vec2_t<S> *__restrict__ out, const long *__restrict__ off,
                                                    const int *__restrict__ active, int N, int nblocks, int W)
{
    __shared__ cx<S> xs[RR][2 * NMAX];
    int b, grp;
    if (!transfer_part(nblocks, (W + RR - 1) / RR, b, grp)) return;
    const int r0 = grp * RR, s = threadIdx.x;
    const int c = __builtin_amdgcn_readfirstlane(s >> 7), h = s & 127;
    bool on = false;
#pragma unroll
    for (int rr = 0; rr < RR; ++rr) on |= r0 + rr < W && (!active || active[r0 + rr]);
    if (!on) return; // uniform
    const PT<S> *p = P + pidx(b, c, 0, N, 0, 0);
    constexpr int U = PU<S>;
    Pair<S> q[U][6], qn[U][6];
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u < N) load_p<S, NT>(p + u * 6 * BS, h, q[u]);
    if (s < 2 * N * RR) {
        const int rr = s / (2 * N), k = s - rr * 2 * N;
        xs[rr][k] = ldc<S>(xc + ((long)min(r0 + rr, W - 1) * nblocks + b) * 2 * N + k);
    }
    __syncthreads();
    cx<S> acc[RR][6][2];
#pragma unroll
    for (int rr = 0; rr < RR; ++rr)
#pragma unroll
        for (int x = 0; x < 6; ++x) acc[rr][x][0] = acc[rr][x][1] = mk<S>(0, 0);
#pragma unroll 1
    for (int i = 0; i < N; i += U) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + U + u < N) load_p<S, NT>(p + (long)(i + U + u) * 6 * BS, h, qn[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i + u < N) {
#pragma unroll
                for (int rr = 0; rr < RR; ++rr) {
                    const cx<S> xi = xs[rr][c * N + i + u];
#pragma unroll
                    for (int x = 0; x < 6; ++x)
#pragma unroll
                        for (int k = 0; k < 2; ++k) cmac(acc[rr][x][k], ldc<S>(&q[u][x].e[k]), xi);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int x = 0; x < 6; ++x) q[u][x] = qn[u][x];
    }
#pragma unroll
    for (int rr = 0; rr < RR; ++rr) {
        const int r = r0 + rr;
        if (r >= W || (active && !active[r])) continue; // uniform
        vec2_t<S> *o = out + (off ? off[r] : 0) + ((long)b * W + r) * 12 * BS + 6 * c * BS;
#pragma unroll
        for (int x = 0; x < 6; ++x)
#pragma unroll
            for (int k = 0; k < 2; ++k) stc(o + x * BS + pair_site<S>(h, k), acc[rr][x][k]);
    }
}

// An FP32 P that outgrows the 256 MB cache in front of HBM is read past it
// (24^3x48, 764 MB: restriction 168 -> 146 us, prolongation 160 -> 149).  A
// smaller one stays cached from call to call, and FP64, two loads for a pair,
// lost by it (24^3x48: 310 -> 346 and 320 -> 357 us).
template <typename S> bool p_streams(int nb, int N)
{
    return sizeof(S) == 4 && (size_t)nb * N * 12 * BS * sizeof(vec2_t<S>) > (256u << 20);
}

template <typename S, int RR>
void restrict_rr(int nb, int W, hipStream_t st, const void *in, const DevBuf &P, void *xc, const int *active, int N)
{
    (p_streams<S>(nb, N) ? k_amg_restrict<S, RR, sizeof(S) == 4> : k_amg_restrict<S, RR, false>)<<<(nb + NXCD - 1) / NXCD * NXCD * ((W + RR - 1) / RR), BS, 0, st>>>(
        static_cast<const vec2_t<S> *>(in), static_cast<const vec2_t<S> *>(P.p), static_cast<double2 *>(xc), active, N, nb, W);
}
template <typename S, int RR>
void prolong_rr(int nb, int W, hipStream_t st, const void *xc, const DevBuf &P, void *out, const long *off, const int *active,
                int N)
{
    (p_streams<S>(nb, N) ? k_amg_prolong<S, RR, sizeof(S) == 4> : k_amg_prolong<S, RR, false>)<<<(nb + NXCD - 1) / NXCD * NXCD * ((W + RR - 1) / RR), BS, 0, st>>>(
        static_cast<const double2 *>(xc), static_cast<const vec2_t<S> *>(P.p), static_cast<vec2_t<S> *>(out), off, active, N,
        nb, W);
}
// Right-hand sides per workgroup: as few as keep the workgroups to two per CU
// (waiting for each other's sums costs a lone workgroup more than the reads that
// it shares), else as many as registers hold.
template <typename S> int rr_of(const dd_ctx *ctx, int W)
{
    for (int rr = 1; rr < rr_max<S>(); rr *= 2)
        if (W <= rr || (long)ctx->g.nblocks * ((W + rr - 1) / rr) <= 2L * ctx->ncu) return rr;
    return rr_max<S>();
}

// x_c = P^+ in and out = P x_c
template <typename S>
void amg_restrict(const dd_ctx *ctx, int W, const void *in, const DevBuf &P, void *xc, const int *active, int N)
{
    const int nb = ctx->g.nblocks;
    hipStream_t st = ctx->stream;
    const int rr = rr_of<S>(ctx, W);
    if (rr == 1) restrict_rr<S, 1>(nb, W, st, in, P, xc, active, N);
    else if (rr == 2) restrict_rr<S, 2>(nb, W, st, in, P, xc, active, N);
    else restrict_rr<S, rr_max<S>()>(nb, W, st, in, P, xc, active, N);
}
template <typename S>
void amg_prolong(const dd_ctx *ctx, int W, const void *xc, const DevBuf &P, void *out, const long *off, const int *active, int N)
{
    const int nb = ctx->g.nblocks;
    hipStream_t st = ctx->stream;
    const int rr = rr_of<S>(ctx, W);
    if (rr == 1) prolong_rr<S, 1>(nb, W, st, xc, P, out, off, active, N);
    else if (rr == 2) prolong_rr<S, 2>(nb, W, st, xc, P, out, off, active, N);
    else prolong_rr<S, rr_max<S>()>(nb, W, st, xc, P, out, off, active, N);
}

// ---------------------------------------------------------------------------
// coarse vectors: y = (D_c + m0) x, and the device-side GMRES
// ---------------------------------------------------------------------------
struct CArgs {
    Geom g;
    int N;
    int nblocks;
    int W;
    const double *m0_dev;
    const int *active;
};

// neighbour block of b in direction d (1 + 2 mu: +mu, 2 + 2 mu: -mu)
__device__ __forceinline__ int cnbr(const Geom &g, int b, const int bc[4], int d)
{
    const int mu = (d - 1) >> 1;
    if ((d - 1) & 1) return bc[mu] == 0 ? b + (g.nb[mu] - 1) * g.bstride[mu] : b - g.bstride[mu];
    return bc[mu] + 1 == g.nb[mu] ? b - (g.nb[mu] - 1) * g.bstride[mu] : b + g.bstride[mu];
}


// Per-slot state of the device GMRES (k <= CK steps).
struct GState {
    double2 H[(CK + 1) * CK]; // rotated Hessenberg (row i, column j at i * CK + j)
    double2 g[CK + 1];
    double2 sn[CK];
    double cs[CK];
    int ncol;   // columns built so far
    // the first step not to take: one past the step at which the Krylov space
    // closed.  Step j tests it against j, so what that step sets while others
    // are still to read it changes no test of the step itself.
    int stop;
};

// The totals of values 0..count-1 over the CG group partials
// (part[(r * nvals + v) * CG + group]), computed by the whole workgroup --
// wavefront w takes values w, w + 4, ...; each lane adds CG / 64 partials,
// then a fixed-order DPP sum -- into out[] (shared).  Every workgroup gets
// the same totals.  Ends with a barrier.
__device__ __forceinline__ void group_totals(const double2 *__restrict__ part, int r, int nvals, int count,
                                             double2 *out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int v = wave; v < count; v += CTPB / 64) {
        double re = 0, im = 0;
        double2 x[CG / 64];
#pragma unroll
        for (int q = 0; q < CG / 64; ++q) x[q] = part[((long)r * nvals + v) * CG + q * 64 + lane];
#pragma unroll
        for (int q = 0; q < CG / 64; ++q) {
            re += x[q].x;
            im += x[q].y;
        }
        re = wave_sum(re);
        im = wave_sum(im);
        if (lane == 63) out[v] = make_double2(re, im);
    }
    __syncthreads();
}

// The partial dots <v_i, w>, i <= j, of this workgroup's rows of w, four
// vectors at a time (their loads and sums overlap).
__device__ __forceinline__ void group_dots(Red &R, const double2 *__restrict__ Vr, const double2 *w, long nrow, int j,
                                           double2 *__restrict__ part, int r, int nvals)
{
    const int s = threadIdx.x, lane = s & 63, wave = s >> 6;
    for (int i0 = 0; i0 <= j; i0 += 4) {
        double re[4] = {0, 0, 0, 0}, im[4] = {0, 0, 0, 0};
        for (long t = (long)blockIdx.x * CTPB + s; t < nrow; t += (long)gridDim.x * CTPB) {
            const double2 x = w[t];
            double2 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = Vr[(long)min(i0 + u, j) * nrow + t];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                re[u] += v[u].x * x.x + v[u].y * x.y;
                im[u] += v[u].x * x.y - v[u].y * x.x;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            re[u] = wave_sum(re[u]);
            im[u] = wave_sum(im[u]);
        }
        if (lane == 63) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (i0 + u <= j) {
                    R.v[wave][i0 + u][0] = re[u];
                    R.v[wave][i0 + u][1] = im[u];
                }
            }
        }
    }
    __syncthreads();
    if (s <= j) stc(part + ((long)r * nvals + s) * CG + blockIdx.x, wave_get(R, s));
}

// |b|^2 partials (stage 0 of the solve)
__global__ __launch_bounds__(CTPB) void k_cg_norm(const double2 *__restrict__ bvec, double2 *__restrict__ part, CArgs a)
{
    __shared__ Red R;
    const int r = blockIdx.y, s = threadIdx.x;
    if (a.active && !a.active[r]) return;
    const long nrow = (long)a.nblocks * 2 * a.N;
    double n2 = 0;
    for (long t = (long)blockIdx.x * CTPB + s; t < nrow; t += (long)gridDim.x * CTPB) {
        const double2 v = bvec[(long)r * nrow + t];
        n2 += v.x * v.x + v.y * v.y;
    }
    wave_put(R, s & 63, s >> 6, 0, n2, 0.0);
    __syncthreads();
    if (s == 0) stc(part + ((long)r * CG + blockIdx.x), wave_get(R, 0));
}

// v_0 = b / |b|, state reset
__global__ __launch_bounds__(CTPB) void k_cg_init(const double2 *__restrict__ bvec, double2 *__restrict__ V,
                                                  const double2 *__restrict__ part, GState *__restrict__ st, CArgs a,
                                                  int kmax)
{
    const int r = blockIdx.y, s = threadIdx.x;
    if (a.active && !a.active[r]) return;
    const long nrow = (long)a.nblocks * 2 * a.N;
    __shared__ double2 tot[1];
    group_totals(part, r, 1, 1, tot);
    const double nb = sqrt(tot[0].x);
    const double inv = nb > 0 ? 1.0 / nb : 0.0;
    for (long t = (long)blockIdx.x * CTPB + s; t < nrow; t += (long)gridDim.x * CTPB) {
        const double2 v = bvec[(long)r * nrow + t];
        V[((long)r * (kmax + 1)) * nrow + t] = make_double2(v.x * inv, v.y * inv);
    }
    if (blockIdx.x == 0) {
        GState &S = st[r];
        for (int e = s; e < (CK + 1) * CK; e += CTPB) S.H[e] = make_double2(0, 0);
        for (int e = s; e <= CK; e += CTPB) S.g[e] = make_double2(0, 0);
        __syncthreads();
        if (s == 0) {
            S.ncol = 0;
            S.stop = nb > 0 ? CK : 0;
            S.g[0] = make_double2(nb, 0);
        }
    }
}

// Givens rotation in the convention of LAPACK's zlartg: [c s; -conj(s) c]
// [f; g] = [r; 0] with c real >= 0
__device__ __forceinline__ void givens(cx<double> f, cx<double> g, double &c, cx<double> &sn, cx<double> &rr)
{
    const double af = sqrt(f.re * f.re + f.im * f.im), ag = sqrt(g.re * g.re + g.im * g.im);
    if (ag == 0.0) {
        c = 1.0;
        sn = mk<double>(0, 0);
        rr = f;
    } else if (af == 0.0) {
        c = 0.0;
        sn = (1.0 / ag) * conjx(g);
        rr = mk<double>(ag, 0);
    } else {
        const double nrm = sqrt(af * af + ag * ag);
        const cx<double> ph = (1.0 / af) * f;
        c = af / nrm;
        sn = (1.0 / nrm) * (ph * conjx(g));
        rr = nrm * ph;
    }
}

// One Arnoldi step is three kernels after the operator: the dots of w with the
// basis; a first Gram-Schmidt pass, with the dots and the norm of what it
// leaves; a second pass, which also normalises.  The norm after the second
// pass is |w|^2 - sum |h|^2 with the norm after the first and the second pass's
// h, so the vector needs no kernel of its own to be normalised: the basis is
// orthonormal, and those h are the rounding of the first pass, a few eps
// |D v_j|.  Where w itself is no longer than that (1e-14 |D v_j|) the space has
// closed and the vector is not used; else they take little off |w|^2.  (Against
// |b| the test depended on the right-hand side's scale: a tiny one went on with
// vectors that were all rounding and not of length one, a huge one stopped at
// once.)  Bound by the launches (4.5 us each) and a chain of a few memory round
// trips.  Four kernels, partial sums read across lines and one vector's dot
// after another took 32.5 us a step at 24^3x48 (N = 12, sixteen steps) where
// this takes 23, and 28 us at 16^4 where this takes 19; the preconditioner
// 2.83 -> 2.68 and 0.99 -> 0.87 ms.
__global__ __launch_bounds__(CTPB) void k_cg_dots(const double2 *__restrict__ V, const double2 *__restrict__ w,
                                                  double2 *__restrict__ part, const GState *__restrict__ st, CArgs a,
                                                  int kmax, int j)
{
    __shared__ Red R;
    const int r = blockIdx.y;
    if ((a.active && !a.active[r]) || st[r].stop <= j) return;
    const long nrow = (long)a.nblocks * 2 * a.N;
    group_dots(R, V + (long)r * (kmax + 1) * nrow, w + (long)r * nrow, nrow, j, part, r, kmax + 1);
}

// First pass: w -= sum_i h_i v_i (i <= j), h_i the totals of part; the partial
// dots of the new w (partB) and of |w|^2 (partN; group 0's imaginary part, else
// zero, is sum |h_i|^2, so that the total is |w|^2 + i (|D v_j|^2 - |w|^2)).
__global__ __launch_bounds__(CTPB) void k_cg_orth(const double2 *__restrict__ V, double2 *__restrict__ w,
                                                  const double2 *__restrict__ part, double2 *__restrict__ partB,
                                                  double2 *__restrict__ partN, const GState *__restrict__ st, CArgs a,
                                                  int kmax, int j)
{
    __shared__ Red R, Rn;
    __shared__ double2 h[CK + 1];
    const int r = blockIdx.y, s = threadIdx.x;
    if ((a.active && !a.active[r]) || st[r].stop <= j) return;
    const long nrow = (long)a.nblocks * 2 * a.N;
    group_totals(part, r, kmax + 1, j + 1, h);
    const double2 *Vr = V + (long)r * (kmax + 1) * nrow;
    double2 *wr = w + (long)r * nrow;
    double n2 = 0;
    for (long t = (long)blockIdx.x * CTPB + s; t < nrow; t += (long)gridDim.x * CTPB) {
        cx<double> x = ldc<double>(wr + t);
#pragma unroll 4
        for (int i = 0; i <= j; ++i) x = x - ldc<double>(&h[i]) * ldc<double>(Vr + (long)i * nrow + t);
        stc(wr + t, x);
        n2 += x.re * x.re + x.im * x.im;
    }
    double hh = 0;
    if (blockIdx.x == 0 && s == 0)
        for (int i = 0; i <= j; ++i) hh += h[i].x * h[i].x + h[i].y * h[i].y;
    wave_put(Rn, s & 63, s >> 6, 0, n2, hh);
    // the rows of this thread were written by this thread: no barrier needed
    group_dots(R, Vr, wr, nrow, j, partB, r, kmax + 1);
    if (s == 0) stc(partN + ((long)r * CG + blockIdx.x), wave_get(Rn, 0));
}

// Second pass, h the totals of partB: v_{j+1} = (w - sum_i h_i v_i) / beta;
// group 0 sets column j of H, the totals of both passes, and rotates it; a
// space that closed (beta tiny against |D v_j|) stops growing.
__global__ __launch_bounds__(CTPB) void k_cg_next(double2 *__restrict__ V, const double2 *__restrict__ w,
                                                  const double2 *__restrict__ partA, const double2 *__restrict__ partB,
                                                  const double2 *__restrict__ partN, GState *__restrict__ st, CArgs a,
                                                  int kmax, int j)
{
    __shared__ double2 h[CK + 1], h1[CK + 1], tot[1];
    const int r = blockIdx.y, s = threadIdx.x;
    if ((a.active && !a.active[r]) || st[r].stop <= j) return;
    const long nrow = (long)a.nblocks * 2 * a.N;
    group_totals(partN, r, 1, 1, tot);
    group_totals(partB, r, kmax + 1, j + 1, h);
    double n2 = tot[0].x;
    for (int i = 0; i <= j; ++i) n2 -= h[i].x * h[i].x + h[i].y * h[i].y;
    const double beta = n2 > 0 ? sqrt(n2) : n2 == n2 ? 0.0 : n2; // (a NaN stays one)
    const bool closes = !(beta > 1e-14 * sqrt(tot[0].x + tot[0].y));
    if (!closes && j + 1 <= kmax) {
        const double inv = 1.0 / beta;
        double2 *Vr = V + (long)r * (kmax + 1) * nrow;
        for (long t = (long)blockIdx.x * CTPB + s; t < nrow; t += (long)gridDim.x * CTPB) {
            cx<double> x = ldc<double>(w + (long)r * nrow + t);
#pragma unroll 4
            for (int i = 0; i <= j; ++i) x = x - ldc<double>(&h[i]) * ldc<double>(Vr + (long)i * nrow + t);
            stc(Vr + (long)(j + 1) * nrow + t, inv * x);
        }
    }
    if (blockIdx.x == 0) { // uniform
        group_totals(partA, r, kmax + 1, j + 1, h1);
        GState &S = st[r];
        if (s <= j) {
            h[s].x += h1[s].x;
            h[s].y += h1[s].y;
        }
        // the earlier rotations, all at hand before the chain
        __shared__ double2 sn_[CK];
        __shared__ double cs_[CK];
        if (s < j) {
            sn_[s] = S.sn[s];
            cs_[s] = S.cs[s];
        }
        __syncthreads();
        if (s == 0) {
            // apply the earlier rotations to column j, then form rotation j
            cx<double> x0 = ldc<double>(&h[0]);
            for (int i = 0; i < j; ++i) {
                const cx<double> x1 = ldc<double>(&h[i + 1]), sn = ldc<double>(&sn_[i]);
                stc(&S.H[i * CK + j], cs_[i] * x0 + sn * x1);
                x0 = cs_[i] * x1 - conjx(sn) * x0;
            }
            double c;
            cx<double> sn, rr;
            givens(x0, mk<double>(closes ? 0.0 : beta, 0), c, sn, rr);
            S.cs[j] = c;
            stc(&S.sn[j], sn);
            stc(&S.H[j * CK + j], rr);
            const cx<double> gj = ldc<double>(&S.g[j]);
            stc(&S.g[j], c * gj);
            stc(&S.g[j + 1], mk<double>(0, 0) - conjx(sn) * gj);
            S.ncol = j + 1;
            if (closes) S.stop = j + 1;
        }
    }
}

// y_r = (D_c + m0_r) x_r for the slots (slot r reads x + r * xs and writes
// y + r * ys; [nblocks][2N] each), the FP16 copy of D_c with FP64 vectors and
// accumulation.  A workgroup takes CS coarse sites, a thread one row of one of a
// site's nine 2N x 2N blocks, read column by column, so the 2N threads of a
// block read consecutive entries; the source vectors wait in LDS, and the nine
// partial sums of a row are added in order through LDS.
// Bound by latency on small lattices and by the 576-entry blocks coming from
// the cache on large ones.  One thread per row, all nine blocks in turn and the
// source entries loaded by every lane, took 16.4 us a launch at 24^3x48 (N = 12)
// where this takes 12, and 15.9 us at 16^4 where this takes 6.2; the whole
// preconditioner 2.91 -> 2.84 ms, 1.16 -> 1.00 ms (8^4: 1.05 -> 0.95).
template <int N2> constexpr int CS = 256 / (9 * N2) > 0 ? 256 / (9 * N2) : 1; // sites per workgroup
template <int N2> constexpr int CT = (9 * N2 * CS<N2> + 63) / 64 * 64;        // threads
// N2 = 2N is a compile-time constant so that the loads of a block row are
// issued together (a run-time loop waits on each pair of loads in turn)
template <int N2>
__global__ __launch_bounds__(CT<N2>) void k_coarse_apply(const __half2 *__restrict__ Ah, const double2 *__restrict__ x,
                                                         long xs, double2 *__restrict__ y, long ys,
                                                         const GState *__restrict__ st, CArgs a, int j)
{
    __shared__ double2 X[CS<N2> * 9][N2]; // source vectors, then the partial sums
    const int r = blockIdx.y, t = threadIdx.x;
    if ((a.active && !a.active[r]) || (st && st[r].stop <= j)) return;
    const int sd = t / N2, k = t - sd * N2; // block (site, direction) of the workgroup, row
    const int site = sd / 9, d = sd - 9 * site;
    const int b = blockIdx.x * CS<N2> + site;
    const bool on = site < CS<N2> && b < a.nblocks;
    const double2 *xr = x + (long)r * xs;
    cx<double> acc = mk<double>(0, 0);
    __half2 A[N2];
    if (on) {
        const __half2 *Ac = Ah + ((long)b * 9 + d) * N2 * N2 + k;
#pragma unroll
        for (int kp = 0; kp < N2; ++kp) A[kp] = Ac[kp * N2];
        int bc[4];
        block_coords(a.g, b, bc);
        const int src = d == 0 ? b : cnbr(a.g, b, bc, d);
        X[sd][k] = xr[(long)src * N2 + k];
    }
    __syncthreads();
    if (on) {
        if (d == 0) acc = a.m0_dev[r] * ldc<double>(&X[sd][k]);
#pragma unroll
        for (int kp = 0; kp < N2; ++kp) cmac(acc, ldc<double>(&A[kp]), ldc<double>(&X[sd][kp]));
    }
    __syncthreads();
    if (on) stc(&X[sd][k], acc);
    __syncthreads();
    if (on && d == 0) {
#pragma unroll
        for (int e = 1; e < 9; ++e) acc = acc + ldc<double>(&X[sd + e][k]);
        stc(y + (long)r * ys + (long)b * N2 + k, acc);
    }
}

void coarse_apply(const dd_ctx *ctx, int W, const __half2 *Ah, const double2 *x, long xs, double2 *y, long ys,
                  const GState *S, const CArgs &a, int j)
{
    switch (a.N) {
#define DD_CA(n) case n: k_coarse_apply<2 * n><<<dim3((a.nblocks + CS<2 * n> - 1) / CS<2 * n>, W), CT<2 * n>, 0, ctx->stream>>>(Ah, x, xs, y, ys, S, a, j); break;
        DD_CA(1) DD_CA(2) DD_CA(3) DD_CA(4) DD_CA(5) DD_CA(6) DD_CA(7) DD_CA(8)
        DD_CA(9) DD_CA(10) DD_CA(11) DD_CA(12) DD_CA(13) DD_CA(14) DD_CA(15) DD_CA(16)
#undef DD_CA
    default: break;
    }
}

// y = R^-1 g over the columns built, then x = V y (one slot per grid row)
__global__ __launch_bounds__(CTPB) void k_cg_finish(const double2 *__restrict__ V, double2 *__restrict__ x,
                                                    const GState *__restrict__ st, CArgs a, int kmax)
{
    __shared__ double2 y[CK], H[CK * CK];
    const int r = blockIdx.y, s = threadIdx.x;
    if (a.active && !a.active[r]) return;
    const GState &S = st[r];
    const int n = S.ncol;
    for (int e = s; e < n * CK; e += CTPB) H[e] = S.H[e];
    if (s < n) y[s] = S.g[s];
    __syncthreads();
    if (s == 0) { // the chain works in LDS (on global memory it took 5 us more)
        for (int i = n - 1; i >= 0; --i) {
            cx<double> acc = ldc<double>(&y[i]);
            for (int k = i + 1; k < n; ++k) acc = acc - ldc<double>(&H[i * CK + k]) * ldc<double>(&y[k]);
            const cx<double> d = ldc<double>(&H[i * CK + i]);
            const double dd = d.re * d.re + d.im * d.im;
            // a zero pivot only if the coarse operator is singular on the space
            const cx<double> q = dd > 0 ? (1.0 / dd) * (acc * conjx(d)) : mk<double>(0, 0);
            stc(&y[i], q);
        }
    }
    __syncthreads();
    const long nrow = (long)a.nblocks * 2 * a.N;
    const double2 *Vr = V + (long)r * (kmax + 1) * nrow;
    for (long t = (long)blockIdx.x * CTPB + s; t < nrow; t += (long)gridDim.x * CTPB) {
        cx<double> acc = mk<double>(0, 0);
#pragma unroll 4
        for (int i = 0; i < n; ++i) cmac(acc, ldc<double>(&y[i]), ldc<double>(Vr + (long)i * nrow + t));
        stc(x + (long)r * nrow + t, acc);
    }
}

// z (slot offsets) = a + b for the W slots
template <typename S>
__global__ __launch_bounds__(BS) void k_amg_sum(const vec2_t<S> *__restrict__ p, const vec2_t<S> *__restrict__ q,
                                                vec2_t<S> *__restrict__ z, const long *__restrict__ zoff,
                                                const int *__restrict__ active, int nblocks, int W)
{
    const int r = blockIdx.y, s = threadIdx.x;
    if (active && !active[r]) return;
    for (int b = blockIdx.x; b < nblocks; b += gridDim.x) {
        const long base = ((long)b * W + r) * 12 * BS + s;
        for (int c = 0; c < 12; ++c)
            stc(z + (zoff ? zoff[r] : 0) + base + c * BS,
                ldc<double>(p + base + c * BS) + ldc<double>(q + base + c * BS));
    }
}

// contiguous copy of W slots from base + off[r]
template <typename S>
__global__ __launch_bounds__(BS) void k_amg_gather(const vec2_t<S> *__restrict__ in, const long *__restrict__ off,
                                                   vec2_t<S> *__restrict__ out, const int *__restrict__ active,
                                                   int nblocks, int W)
{
    const int r = blockIdx.y, s = threadIdx.x;
    if (active && !active[r]) return;
    for (int b = blockIdx.x; b < nblocks; b += gridDim.x) {
        const long base = ((long)b * W + r) * 12 * BS + s;
        for (int c = 0; c < 12; ++c) out[base + c * BS] = in[(off ? off[r] : 0) + base + c * BS];
    }
}

// test-vector normalisation: per vector |v|^2 partials, then v /= |v|
template <typename S>
__global__ __launch_bounds__(BS) void k_tv_norm(const vec2_t<S> *__restrict__ v, double2 *__restrict__ part, int nblocks,
                                                int W)
{
    __shared__ Red R;
    const int r = blockIdx.y, s = threadIdx.x;
    double n2 = 0;
    for (int b = blockIdx.x; b < nblocks; b += gridDim.x) {
        const long base = ((long)b * W + r) * 12 * BS + s;
        for (int c = 0; c < 12; ++c) {
            const cx<double> x = ldc<double>(v + base + c * BS);
            n2 += x.re * x.re + x.im * x.im;
        }
    }
    wave_put(R, s & 63, s >> 6, 0, n2, 0.0);
    __syncthreads();
    if (s == 0) stc(part + (long)r * CG + blockIdx.x, wave_get(R, 0));
}

template <typename S>
__global__ __launch_bounds__(BS) void k_tv_scale(const vec2_t<S> *__restrict__ v, vec2_t<S> *__restrict__ out,
                                                 const double2 *__restrict__ part, int nblocks, int W)
{
    const int r = blockIdx.y, s = threadIdx.x;
    __shared__ double2 tot[1];
    group_totals(part, r, 1, 1, tot);
    const double inv = 1.0 / sqrt(tot[0].x);
    for (int b = blockIdx.x; b < nblocks; b += gridDim.x) {
        const long base = ((long)b * W + r) * 12 * BS + s;
        for (int c = 0; c < 12; ++c) stc(out + base + c * BS, inv * ldc<double>(v + base + c * BS));
    }
}

// FP32 blocked spinors -> FP64 (same layout)
__global__ __launch_bounds__(BS) void k_f32_to_f64(const float2 *__restrict__ in, double2 *__restrict__ out, long n)
{
    for (long i = (long)blockIdx.x * BS + threadIdx.x; i < n; i += (long)gridDim.x * BS) {
        const float2 v = in[i];
        out[i] = make_double2(v.x, v.y);
    }
}

unsigned grid_for(long n) { return (unsigned)std::min<long>((n + BS - 1) / BS, 8192); }

} // namespace

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
struct AmgWork {
    int W = 0, prec = -1, kmax = 0, N = 0;
    DevBuf xb, xx, V, w, partA, partB, partN, st; // coarse
    DevBuf et, ps, rr, dl, sapscr, m0;           // fine (smoother precision), masses
};

struct AmgData {
    int N = 0;
    dd_amg_params p{};
    DevBuf Pd, Pf, Ad, Ah; // P FP64 / FP32; D_c FP64 / FP16 (the copy the coarse solve reads)
    AmgWork work; // standalone calls and the setup's adaptive rounds
};

void AmgDeleter::operator()(AmgData *a) const { delete a; }

namespace {

CArgs cargs(const dd_ctx *ctx, int W, const double *m0_dev, const int *active)
{
    CArgs a{};
    for (int k = 0; k < 4; ++k) {
        a.g.nb[k] = ctx->g.nb[k];
        a.g.bstride[k] = ctx->g.bstride[k];
        a.g.bcs[k] = ctx->g.bcs[k];
    }
    a.g.nblocks = ctx->g.nblocks;
    a.N = ctx->amg->N;
    a.nblocks = ctx->g.nblocks;
    a.W = W;
    a.m0_dev = m0_dev;
    a.active = active;
    return a;
}

size_t ncoarse(const dd_ctx *ctx) { return (size_t)ctx->g.nblocks * 2 * ctx->amg->N; }

} // namespace

Status amg_reserve(dd_ctx *ctx, AmgWork &wk, int W, int prec, int kmax)
{
    kmax = std::max(kmax, ctx->amg->p.coarse_k);
    if (wk.W == W && wk.prec == prec && wk.kmax == kmax && wk.N == ctx->amg->N) return Status::ok();
    const size_t nc = ncoarse(ctx), cv = nc * 16 * W;
    DD_TRY(wk.xb.alloc(cv));
    DD_TRY(wk.xx.alloc(cv));
    DD_TRY(wk.V.alloc(cv * (kmax + 1)));
    DD_TRY(wk.w.alloc(cv));
    DD_TRY(wk.partA.alloc((size_t)W * CG * (kmax + 1) * 16));
    DD_TRY(wk.partB.alloc((size_t)W * CG * (kmax + 1) * 16));
    DD_TRY(wk.partN.alloc((size_t)W * CG * 16));
    DD_TRY(wk.st.alloc((size_t)W * sizeof(GState)));
    const size_t sb = spinor_bytes(ctx->g, prec, W);
    DD_TRY(wk.et.alloc(sb));
    DD_TRY(wk.ps.alloc(sb));
    DD_TRY(wk.rr.alloc(sb));
    DD_TRY(wk.dl.alloc(sb));
    DD_TRY(wk.sapscr.alloc(sap_scratch_bytes(ctx->g, prec, W)));
    DD_TRY(wk.m0.alloc((size_t)W * sizeof(double)));
    wk.W = W;
    wk.prec = prec;
    wk.kmax = kmax;
    wk.N = ctx->amg->N;
    return Status::ok();
}

AmgWork *amg_work_new() { return new AmgWork(); }
void AmgWorkDeleter::operator()(AmgWork *w) const { delete w; }

// k-step GMRES from zero on (D_c + m0_r) x_r = b_r for the W slots (b in
// wk.xb, x to wk.xx); device only.
Status coarse_gmres(dd_ctx *ctx, AmgWork &wk, int W, int k, const double *m0_dev, const int *active)
{
    AmgData &A = *ctx->amg;
    const CArgs a = cargs(ctx, W, m0_dev, active);
    const int kmax = wk.kmax;
    const dim3 grid(CG, W);
    hipStream_t st = ctx->stream;
    const long nrow = (long)ncoarse(ctx);
    double2 *V = wk.V.as<double2>(), *w = wk.w.as<double2>();
    GState *S = wk.st.as<GState>();
    k_cg_norm<<<grid, CTPB, 0, st>>>(wk.xb.as<double2>(), wk.partN.as<double2>(), a);
    k_cg_init<<<grid, CTPB, 0, st>>>(wk.xb.as<double2>(), V, wk.partN.as<double2>(), S, a, kmax);
    for (int j = 0; j < k; ++j) {
        // w = (D_c + m0) v_j
        coarse_apply(ctx, W, A.Ah.as<__half2>(), V + (long)j * nrow, (long)(kmax + 1) * nrow, w, nrow, S, a, j);
        k_cg_dots<<<grid, CTPB, 0, st>>>(V, w, wk.partA.as<double2>(), S, a, kmax, j);
        k_cg_orth<<<grid, CTPB, 0, st>>>(V, w, wk.partA.as<double2>(), wk.partB.as<double2>(), wk.partN.as<double2>(), S, a, kmax, j);
        k_cg_next<<<grid, CTPB, 0, st>>>(V, w, wk.partA.as<double2>(), wk.partB.as<double2>(), wk.partN.as<double2>(), S, a, kmax, j);
    }
    k_cg_finish<<<grid, CTPB, 0, st>>>(V, wk.xx.as<double2>(), S, a, kmax);
    DD_HIP_TRY(hipGetLastError());
    return Status::ok();
}

// The two-grid preconditioner for W slots: z = P x_c + SAP_nu(eta - D P x_c),
// x_c the coarse solve of D_c x_c = P^+ eta.  eta (z): slot r at base +
// off[r] in the blocked layout with W right-hand sides, precision prec.
Status run_two_grid(dd_ctx *ctx, AmgWork &wk, int W, const void *eta, const long *eta_off, int prec, void *z,
                    const long *z_off, const double *m0_dev, const int *active)
{
    AmgData &A = *ctx->amg;
    const int N = A.N, nb = ctx->g.nblocks;
    hipStream_t st = ctx->stream;
    const dim3 sg(std::min(nb, 1024), W);
    const void *e = eta;
    if (eta_off) {
        if (prec == DD_F64)
            k_amg_gather<double><<<sg, BS, 0, st>>>(static_cast<const double2 *>(eta), eta_off, wk.et.as<double2>(), active, nb, W);
        else
            k_amg_gather<float><<<sg, BS, 0, st>>>(static_cast<const float2 *>(eta), eta_off, wk.et.as<float2>(), active, nb, W);
        e = wk.et.p;
    }
    {
        ProfScope ps(ctx->prof, st, K_AMG_RESTRICT, (double)spinor_bytes(ctx->g, prec, W) * (1 + N), 0.0);
        if (prec == DD_F64)
            amg_restrict<double>(ctx, W, e, A.Pd, wk.xb.p, active, N);
        else
            amg_restrict<float>(ctx, W, e, A.Pf, wk.xb.p, active, N);
    }
    {
        ProfScope ps(ctx->prof, st, K_AMG_COARSE, 0.0, 0.0);
        DD_TRY(coarse_gmres(ctx, wk, W, A.p.coarse_k, m0_dev, active));
    }
    // psi_0 = P x_c: straight into z when no post-smoothing follows
    const bool post = A.p.post_ncy > 0;
    {
        ProfScope ps(ctx->prof, st, K_AMG_PROLONG, (double)spinor_bytes(ctx->g, prec, W) * (1 + N), 0.0);
        void *psi = post ? wk.ps.p : z;
        const long *off = post ? nullptr : z_off;
        if (prec == DD_F64) amg_prolong<double>(ctx, W, wk.xx.p, A.Pd, psi, off, active, N);
        else amg_prolong<float>(ctx, W, wk.xx.p, A.Pf, psi, off, active, N);
    }
    DD_HIP_TRY(hipGetLastError());
    if (!post) return Status::ok();
    // r = eta - D psi_0, delta = SAP(r), z = psi_0 + delta
    DD_TRY(launch_dslash(ctx, nullptr, W, wk.ps.p, prec, wk.rr.p, prec, prec, static_cast<const double *>(e), m0_dev,
                         nullptr, active));
    SapSlots ss;
    ss.m0_dev = m0_dev;
    ss.active = active;
    ss.scratch = wk.sapscr.p;
    DD_TRY(run_sap(ctx, nullptr, W, wk.rr.p, wk.dl.p, A.p.post_ncy, A.p.post_nmr, prec, &ss, false));
    if (prec == DD_F64)
        k_amg_sum<double><<<sg, BS, 0, st>>>(wk.ps.as<double2>(), wk.dl.as<double2>(), static_cast<double2 *>(z), z_off,
                                             active, nb, W);
    else
        k_amg_sum<float><<<sg, BS, 0, st>>>(wk.ps.as<float2>(), wk.dl.as<float2>(), static_cast<float2 *>(z), z_off,
                                            active, nb, W);
    DD_HIP_TRY(hipGetLastError());
    return Status::ok();
}

namespace {

Status build_P_Dc(dd_ctx *ctx, const double2 *tv64)
{
    AmgData &A = *ctx->amg;
    const int N = A.N, nb = ctx->g.nblocks;
    k_amg_gs<<<dim3(nb, 2), BS, 0, ctx->stream>>>(tv64, A.Pd.as<double2>(), A.Pf.as<float2>(), N);
    DD_HIP_TRY(hipGetLastError());
    AGeom ag{};
    for (int k = 0; k < 4; ++k) {
        ag.g.nb[k] = ctx->g.nb[k];
        ag.g.bstride[k] = ctx->g.bstride[k];
        ag.g.bcs[k] = ctx->g.bcs[k];
    }
    ag.g.nblocks = nb;
    ag.N = N;
    ag.r12 = ctx->link_r12 ? 1 : 0;
    k_amg_build<<<dim3(nb, 9), BS, 0, ctx->stream>>>(A.Pd.as<double2>(), ctx->links[DD_F64].as<double2>(),
                                                     ctx->clover[DD_F64].as<double2>(), A.Ad.as<double2>(),
                                                     A.Ah.as<__half2>(), ag);
    DD_HIP_TRY(hipGetLastError());
    return Status::ok();
}

template <typename S> Status normalise(dd_ctx *ctx, const void *in, void *out, DevBuf &part, int N)
{
    const int nb = ctx->g.nblocks;
    const dim3 g(CG, N);
    k_tv_norm<S><<<g, BS, 0, ctx->stream>>>(static_cast<const vec2_t<S> *>(in), part.as<double2>(), nb, N);
    k_tv_scale<S><<<g, BS, 0, ctx->stream>>>(static_cast<const vec2_t<S> *>(in), static_cast<vec2_t<S> *>(out),
                                              part.as<double2>(), nb, N);
    DD_HIP_TRY(hipGetLastError());
    return Status::ok();
}

} // namespace

Status amg_setup(dd_ctx *ctx, double m0, const double *v0, const dd_amg_params &p)
{
    if (p.nvec < 1 || p.nvec > NMAX || p.setup_iters < 0 || p.setup_ncy < 1 || p.setup_nmr < 1 || p.adapt < 0 ||
        p.coarse_k < 1 || p.coarse_k > CK || p.post_ncy < 0 || p.post_nmr < 0 ||
        (p.setup_prec != DD_F64 && p.setup_prec != DD_F32))
        return Status{DD_INVALID_ARG, "dd_amg_setup: bad parameters (1 <= nvec <= 16, 1 <= coarse_k <= 32, "
                                      "setup_prec FP64 or FP32, ...)"};
    bool bad = false;
    DD_TRY(any_nonfinite(ctx, v0, (size_t)ctx->g.V * 24 * p.nvec, bad));
    if (bad) return Status{DD_NAN, "dd_amg_setup: starting vectors hold NaN or Inf"};
    ctx->amg.reset(new AmgData());
    AmgData &A = *ctx->amg;
    A.N = p.nvec;
    A.p = p;
    const int N = A.N, sp = p.setup_prec;
    const size_t pbytes = (size_t)ctx->g.nblocks * 2 * N * 6 * BS;
    DD_TRY(A.Pd.alloc(pbytes * 16));
    DD_TRY(A.Pf.alloc(pbytes * 8));
    const size_t abytes = (size_t)ctx->g.nblocks * 9 * 4 * N * N;
    DD_TRY(A.Ad.alloc(abytes * 16));
    DD_TRY(A.Ah.alloc(abytes * 4));
    DevBuf ta, tb, t64, part;
    DD_TRY(ta.alloc(spinor_bytes(ctx->g, sp, N)));
    DD_TRY(tb.alloc(spinor_bytes(ctx->g, sp, N)));
    DD_TRY(part.alloc((size_t)N * CG * 16));
    DD_TRY(pack_spinor(ctx, v0, ta.p, sp, N));
    std::vector<double> m0s(N, m0);
    // inverse iteration with the Schwarz smoother: v <- SAP(v) / |SAP(v)|
    for (int it = 0; it < p.setup_iters; ++it) {
        DD_TRY(run_sap(ctx, m0s.data(), N, ta.p, tb.p, p.setup_ncy, p.setup_nmr, sp));
        DD_TRY(sp == DD_F64 ? normalise<double>(ctx, tb.p, ta.p, part, N) : normalise<float>(ctx, tb.p, ta.p, part, N));
    }
    auto build = [&]() -> Status {
        const double2 *tv = ta.as<double2>();
        if (sp == DD_F32) {
            DD_TRY(t64.alloc(spinor_bytes(ctx->g, DD_F64, N)));
            const long n = (long)ctx->g.V * 12 * N;
            k_f32_to_f64<<<grid_for(n), BS, 0, ctx->stream>>>(ta.as<float2>(), t64.as<double2>(), n);
            DD_HIP_TRY(hipGetLastError());
            tv = t64.as<double2>();
        }
        return build_P_Dc(ctx, tv);
    };
    DD_TRY(build());
    // adaptive rounds: the current two-grid method in place of the smoother
    if (p.adapt > 0) {
        DD_TRY(amg_reserve(ctx, A.work, N, sp, 0));
        DD_HIP_TRY(hipMemcpyAsync(A.work.m0.p, m0s.data(), N * sizeof(double), hipMemcpyHostToDevice, ctx->stream));
        for (int r = 0; r < p.adapt; ++r) {
            DD_TRY(run_two_grid(ctx, A.work, N, ta.p, nullptr, sp, tb.p, nullptr, A.work.m0.as<double>(), nullptr));
            DD_TRY(sp == DD_F64 ? normalise<double>(ctx, tb.p, ta.p, part, N) : normalise<float>(ctx, tb.p, ta.p, part, N));
            DD_TRY(build());
        }
    }
    DD_HIP_TRY(hipStreamSynchronize(ctx->stream));
    return Status::ok();
}

size_t amg_coarse_size(const dd_ctx *ctx) { return ctx->amg ? ncoarse(ctx) : 0; }

Status amg_export(dd_ctx *ctx, double *P_host, double *A_host)
{
    AmgData &A = *ctx->amg;
    if (P_host) DD_HIP_TRY(hipMemcpy(P_host, A.Pd.p, A.Pd.bytes, hipMemcpyDeviceToHost));
    if (A_host) DD_HIP_TRY(hipMemcpy(A_host, A.Ad.p, A.Ad.bytes, hipMemcpyDeviceToHost));
    return Status::ok();
}

Status amg_standalone(dd_ctx *ctx, int op, const double *m0, int nrhs, const void *in, void *out, int prec, int k)
{
    AmgData &A = *ctx->amg;
    AmgWork &wk = A.work;
    if (op == 3 && (k < 1 || k > CK)) return Status{DD_INVALID_ARG, "dd_amg_coarse_solve: 1 <= k <= 32"};
    DD_TRY(amg_reserve(ctx, wk, nrhs, prec, op == 3 ? k : 0));
    std::vector<double> masses(nrhs, 0.0);
    if (m0) masses.assign(m0, m0 + nrhs);
    DD_HIP_TRY(hipMemcpyAsync(wk.m0.p, masses.data(), nrhs * sizeof(double), hipMemcpyHostToDevice, ctx->stream));
    DD_HIP_TRY(hipStreamSynchronize(ctx->stream)); // masses is a host temporary
    const int N = A.N;
    const size_t cv = ncoarse(ctx) * 16 * nrhs;
    const CArgs a = cargs(ctx, nrhs, wk.m0.as<double>(), nullptr);
    switch (op) {
    case 0: // restrict: out (coarse) = P^+ in
        if (prec == DD_F64)
            amg_restrict<double>(ctx, nrhs, in, A.Pd, out, nullptr, N);
        else
            amg_restrict<float>(ctx, nrhs, in, A.Pf, out, nullptr, N);
        break;
    case 1: // prolong: out (fine) = P in
        if (prec == DD_F64)
            amg_prolong<double>(ctx, nrhs, in, A.Pd, out, nullptr, nullptr, N);
        else
            amg_prolong<float>(ctx, nrhs, in, A.Pf, out, nullptr, nullptr, N);
        break;
    case 2: // coarse apply
        coarse_apply(ctx, nrhs, A.Ah.as<__half2>(), static_cast<const double2 *>(in), (long)ncoarse(ctx),
                     static_cast<double2 *>(out), (long)ncoarse(ctx), nullptr, a, 0);
        break;
    case 3: // coarse solve with k steps
        DD_HIP_TRY(hipMemcpyAsync(wk.xb.p, in, cv, hipMemcpyDeviceToDevice, ctx->stream));
        DD_TRY(coarse_gmres(ctx, wk, nrhs, k, wk.m0.as<double>(), nullptr));
        DD_HIP_TRY(hipMemcpyAsync(out, wk.xx.p, cv, hipMemcpyDeviceToDevice, ctx->stream));
        break;
    default: // two-grid preconditioner
        DD_TRY(run_two_grid(ctx, wk, nrhs, in, nullptr, prec, out, nullptr, wk.m0.as<double>(), nullptr));
        break;
    }
    DD_HIP_TRY(hipGetLastError());
    return Status::ok();
}

} // namespace dd
