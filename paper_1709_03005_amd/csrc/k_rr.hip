// Rayleigh-Ritz eigenproblem of the Davidson solver (Sec. 3.2 lists
// Davidson among the diagonalisers): G (m x m, symmetric, m <= 96) ->
// ascending theta and orthonormal eigenvectors Y (column e at Y[q*ldy + e]),
// FP64, one workgroup, all of it in LDS.
//
// k_rr_eig, the main path:
//   1. G is scaled by a power of two and reduced to tridiagonal form
//      T = Q^T G Q by Householder reflectors (kept below the subdiagonal);
//   2. every eigenvalue of T: isolated by Sturm counts from the
//      leading-minor recurrence (rescaled by powers of two) at many shifts
//      at once, one thread per shift, then Laguerre's method, and
//      multisection for what it leaves;
//   3. one eigenvector of T per thread from the twisted factorisation of
//      T - lambda I at the twist index of smallest |gamma|;
//   4. modified Gram-Schmidt (two passes) inside clusters of eigenvalues
//      closer than 1e-3 ||T||, then the reflectors applied to the vectors;
//   5. one Newton-Schulz step Y <- Y (3I - Y^T Y) / 2 on FP64 MFMA, which
//      takes the orthogonality defect from ~1e-13 to rounding level.
// A failed check (a non-finite value, a twisted residual above 1e-10 ||T||,
// a cluster vector that loses 99% of its norm to the projections, or a
// defect above 1e-8 before the Newton-Schulz step, as with exactly
// repeated eigenvalues) reruns the problem by cyclic Jacobi in the same
// launch and counts the event. k_jacobi_eig is the Jacobi path alone.
#include <cfloat>

#include "ccham_internal.h"

namespace cch {

constexpr int RR_MAX = 96, RR_LD = RR_MAX + 1, RR_NT = 512, RR_NW = RR_NT / 64;
typedef double rr_dx4 __attribute__((ext_vector_type(4)));

constexpr int RR_SL = 4;     // row slices of the Householder products (x 2 column halves = 8 waves)
constexpr int RR_G = 512;    // shifts of the first multisection pass

struct RRShared {
    double A[RR_MAX][RR_LD];
    double Z[RR_MAX][RR_LD];
    double d[RR_MAX], e[RR_MAX], lam[RR_MAX], tau[RR_MAX], hinv[RR_MAX];
    double sc[6][RR_MAX];        // per-phase scratch vectors
    alignas(16) double de[RR_MAX][2];   // d_i and e_{i-1}^2 (at least 2^-120), for the counts
    double red[2][32];           // alternating reduction buffers
    union {
        int cnt[RR_NT];                  // Sturm counts; Jacobi pairing tables
        double dbl[RR_NT / 2];           // 16 x 16 Gram matrix of a reflector block
    } u;
    unsigned long long open_mask[2];   // eigenvalues still bracketed (multisection)
    int flag, nrot;
};
static_assert(sizeof(RRShared) <= 160 * 1024, "LDS budget");

__device__ __forceinline__ double rr_wave_sum(double v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ double rr_wave_max(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Block reductions with one barrier: consecutive calls must alternate the
// buffer, so that a buffer is written again only after a later barrier.
__device__ __forceinline__ double rr_block_sum(double v, double *red)
{
    v = rr_wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += red[w];
    return s;
}

__device__ __forceinline__ double rr_block_max(double v, double *red)
{
    v = rr_wave_max(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = red[0];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) s = fmax(s, red[w]);
    return s;
}

// a value every lane holds alike (read from LDS), as a wave-uniform scalar
__device__ __forceinline__ double rr_uni(double v)
{
    RrI2 a = __builtin_bit_cast(RrI2, v);
    a.x = __builtin_amdgcn_readfirstlane(a.x);
    a.y = __builtin_amdgcn_readfirstlane(a.y);
    return __builtin_bit_cast(double, a);
}

// ---------------------------------------------------------------------------
// Cyclic Jacobi, parallel (round-robin tournament) ordering: m/2 disjoint
// rotations per round, m-1 rounds per sweep; a rotation is skipped when
// |a_pq| <= 1e-16 sqrt(|a_pp a_qq|), and the sweeps stop after one with no
// rotation. Reads G itself (unscaled) and writes theta and Y.
// ---------------------------------------------------------------------------
__device__ void rr_jacobi(RRShared &sh, const double *__restrict__ G, int ldg, int m, double *__restrict__ theta,
                          double *__restrict__ Y, int ldy, int max_sweeps)
{
    double(*A)[RR_LD] = sh.A;
    double(*Z)[RR_LD] = sh.Z;
    double *cs = sh.sc[3], *sn = sh.sc[4];
    int *pp = sh.u.cnt, *qq = sh.u.cnt + RR_MAX / 2, *perm = sh.u.cnt + RR_MAX;
    const int me = (m + 1) & ~1;     // even size (a padded index is inert)
    const int half = me / 2;
    const int nthr = blockDim.x;
    __syncthreads();
    for (int t = threadIdx.x; t < me * me; t += nthr) {
        const int i = t / me, j = t % me;
        A[i][j] = (i < m && j < m) ? 0.5 * (G[(int64_t)i * ldg + j] + G[(int64_t)j * ldg + i]) : 0.0;
        Z[i][j] = (i == j) ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int sweep = 0; sweep < max_sweeps; ++sweep) {
        if (threadIdx.x == 0) sh.nrot = 0;
        __syncthreads();
        for (int round = 0; round < me - 1; ++round) {
            if (threadIdx.x < half) {
                const int k = threadIdx.x;
                const int s0 = k, s1 = me - 1 - k;
                int p = s0 == 0 ? 0 : 1 + (s0 - 1 + round) % (me - 1);
                int q = 1 + (s1 - 1 + round) % (me - 1);
                if (p > q) {
                    const int t = p;
                    p = q;
                    q = t;
                }
                pp[k] = p;
                qq[k] = q;
                const double apq = A[p][q];
                double c = 1.0, s = 0.0;
                if (fabs(apq) > 1e-16 * sqrt(fabs(A[p][p] * A[q][q])) && fabs(apq) > 1e-300) {
                    sh.nrot = 1;
                    const double tau = (A[q][q] - A[p][p]) / (2.0 * apq);
                    const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
                    c = 1.0 / sqrt(1.0 + t * t);
                    s = t * c;
                }
                cs[k] = c;
                sn[k] = s;
            }
            __syncthreads();
            // A <- J^T A J on 2x2 blocks (row pair k, column pair l), Z <- Z J
            const int nblk = half * half;
            for (int t = threadIdx.x; t < nblk + half * me; t += nthr) {
                if (t < nblk) {
                    const int k = t / half, l = t % half;
                    const int p = pp[k], q = qq[k], r = pp[l], u = qq[l];
                    const double ck = cs[k], sk = sn[k], cl = cs[l], sl = sn[l];
                    const double apr = A[p][r], apu = A[p][u], aqr = A[q][r], aqu = A[q][u];
                    const double bpr = ck * apr - sk * aqr, bpu = ck * apu - sk * aqu;
                    const double bqr = sk * apr + ck * aqr, bqu = sk * apu + ck * aqu;
                    A[p][r] = cl * bpr - sl * bpu;
                    A[p][u] = sl * bpr + cl * bpu;
                    A[q][r] = cl * bqr - sl * bqu;
                    A[q][u] = sl * bqr + cl * bqu;
                } else {
                    const int e = t - nblk;
                    const int l = e / me, i = e % me;
                    const int r = pp[l], u = qq[l];
                    const double cl = cs[l], sl = sn[l];
                    const double zr = Z[i][r], zu = Z[i][u];
                    Z[i][r] = cl * zr - sl * zu;
                    Z[i][u] = sl * zr + cl * zu;
                }
            }
            __syncthreads();
        }
        if (sh.nrot == 0) break;
        __syncthreads();
    }
    // ascending order (stable), written out
    if (threadIdx.x == 0) {
        for (int i = 0; i < m; ++i) perm[i] = i;
        for (int i = 1; i < m; ++i) {
            const int v = perm[i];
            int j = i - 1;
            while (j >= 0 && A[perm[j]][perm[j]] > A[v][v]) {
                perm[j + 1] = perm[j];
                --j;
            }
            perm[j + 1] = v;
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < m; e += nthr) theta[e] = A[perm[e]][perm[e]];
    for (int t = threadIdx.x; t < m * m; t += nthr) {
        const int q = t / m, e = t % m;
        Y[(int64_t)q * ldy + e] = Z[q][perm[e]];
    }
}

__global__ __launch_bounds__(RR_NT) void k_jacobi_eig(const double *__restrict__ G, int ldg, int m,
                                                      double *__restrict__ theta, double *__restrict__ Y, int ldy,
                                                      int max_sweeps)
{
    __shared__ RRShared sh;
    rr_jacobi(sh, G, ldg, m, theta, Y, ldy, max_sweeps);
}

// Householder reduction of A (n x n, in LDS) to T: d, e, and the reflectors
// H_k = I - tau v v^T with v_{k+1} = 1 and v_r = x_r hinv[k] below, x = row k of
// the trailing matrix, which row k of A keeps. One workgroup of 8 waves: waves
// 1-7 hold the matrix in registers, thread (ty, tx) of 14 x 32 the rows
// ty + 14 i and columns tx + 32 j, and wave 0 does what is done once per step,
// an entry or two a lane. The rows' products with x are taken before its
// reflector is known (v = e_{k+1} + hinv x below), so a step is one pass over the
// rows, update and product together, during which wave 0 forms the next sigma,
// tau and hinv, and then wave 0's sums, p, w and next x between two barriers.
// Bound by that chain (the vector units issue an instruction of a wave in four
// cycles: what every wave does alike costs as much as the rows themselves).
// Measured: 87 us at n = 80 and 31 at n = 40, where the matrix in LDS, the
// vector work in every wave and two barriers a step took 143 and 48.
constexpr int RR_TY = 14, RR_TX = 32;
constexpr int RR_RI = (RR_MAX + RR_TY - 1) / RR_TY, RR_CJ = RR_MAX / RR_TX;
static_assert(RR_TY * RR_TX == RR_NT - 64, "waves 1-7");

struct RRVec {   // entries of v, w and the next x below its second
    double v, w, x, pad;
};

// element i (wave-uniform, < 128) of a vector over the lanes, without a branch
__device__ __forceinline__ double rr_pick(double lo, double hi, int i)
{
    const double a = rr_rl(lo, i & 63), b = rr_rl(hi, i & 63);
    return i < 64 ? a : b;
}

// v + its value 32 lanes away, in every lane
__device__ __forceinline__ double rr_halves(double v)
{
    const RrI2 a = __builtin_bit_cast(RrI2, v);
    const auto x = __builtin_amdgcn_permlane32_swap(a.x, a.x, false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(a.y, a.y, false, false);
    return __builtin_bit_cast(double, RrI2{(int)x[0], (int)y[0]}) + __builtin_bit_cast(double, RrI2{(int)x[1], (int)y[1]});
}

// NI, CJ: row and column groups with entries (n <= RR_TY NI, n <= RR_TX CJ)
template <int NI, int CJ>
__device__ __forceinline__ void rr_house(RRShared &sh, int n, int tid, int wv)
{
    double(*A)[RR_LD] = sh.A;
    double(*P)[RR_LD] = sh.Z;                                    // the waves' partial sums, then row k + 1
    RRVec *vec = reinterpret_cast<RRVec *>(&sh.Z[RR_NW + 2][0]);   // 128 entries (an even row: 16-byte aligned)
    const int lane = tid & 63;
    const bool two = lane + 64 < RR_MAX;   // lanes with a second entry
    const int c1 = two ? lane + 64 : RR_MAX;   // (column RR_MAX is padding)
    double x0 = 0.0, x1 = 0.0;
    if (wv == 0) {
        x0 = lane >= 1 ? A[0][lane] : 0.0;
        x1 = two ? A[0][c1] : 0.0;
        if (lane == 0) sh.d[0] = A[0][0];
        vec[lane] = RRVec{0.0, 0.0, lane >= 2 ? x0 : 0.0, 0.0};
        vec[lane + 64] = RRVec{0.0, 0.0, x1, 0.0};
        for (int k = 0; k + 2 < n; ++k) {
            __syncthreads();
            // sigma, beta, tau, hinv of x = row k right of the diagonal: sqrt and the
            // two quotients from the refined hardware estimates (about one ulp each)
            const double m0 = lane >= k + 2 ? x0 : 0.0, m1 = lane + 64 >= k + 2 ? x1 : 0.0;
            const double sig = rr_uni(rr_wsum(m0 * m0 + m1 * m1));
            const double alpha = rr_pick(x0, x1, k + 1);
            const double h = fma(alpha, alpha, sig);
            const double bt = -copysign(h * rr_rsqrt(h), alpha);
            // (a sigma whose squares have lost bits to underflow gives no orthogonal
            // reflector: entries below 2^-500 of the largest one count as zero)
            const bool none = sig < 0x1p-1000;
            const double tau = none ? 0.0 : fma(-alpha, rr_recip(bt), 1.0);   // (beta - alpha) / beta
            const double inv = none ? 0.0 : rr_recip(alpha - bt);
            if (lane == 0) {
                sh.tau[k] = tau;
                sh.e[k] = none ? alpha : bt;
                sh.hinv[k] = inv;
            }
            A[k][lane] = x0;
            A[k][c1] = x1;
            const double v0 = lane == k + 1 ? 1.0 : m0 * inv, v1 = lane + 64 == k + 1 ? 1.0 : m1 * inv;
            const double t0 = lane >= k + 1 ? tau : 0.0, t1 = two && lane + 64 >= k + 1 ? tau : 0.0;
            __syncthreads();
            double q0 = 0.0, q1 = 0.0;
#pragma unroll
            for (int q = 0; q < RR_NW - 1; ++q) {
                q0 += P[q][lane];
                if (CJ > 2) q1 += P[q][c1];
            }
            const double y0 = P[RR_NW - 1][lane], y1 = CJ > 2 ? P[RR_NW - 1][c1] : 0.0;
            const double p0 = t0 * fma(inv, q0, y0);
            const double p1 = CJ > 2 && two ? t1 * fma(inv, q1, y1) : 0.0;
            const double K = 0.5 * tau * rr_wsum(CJ > 2 ? p0 * v0 + p1 * v1 : p0 * v0);
            const double w0 = p0 - K * v0, w1 = p1 - K * v1;
            // row k + 1 of the next matrix
            const double wk = CJ > 2 ? rr_pick(w0, w1, k + 1) : rr_rl(w0, k + 1);
            x0 = y0 - (w0 + wk * v0);
            x1 = CJ > 2 && two ? y1 - (w1 + wk * v1) : 0.0;
            vec[lane] = RRVec{v0, w0, lane >= k + 3 ? x0 : 0.0, 0.0};
            vec[lane + 64] = RRVec{v1, w1, lane + 64 >= k + 3 ? x1 : 0.0, 0.0};
            if (lane == ((k + 1) & 63)) sh.d[k + 1] = k + 1 < 64 ? x0 : x1;
            x0 = lane >= k + 2 ? x0 : 0.0;
            x1 = lane + 64 >= k + 2 ? x1 : 0.0;
        }
        __syncthreads();
        __syncthreads();
        // x is row n - 2; the last row's diagonal
        if (n >= 2 && lane == ((n - 1) & 63)) {
            sh.e[n - 2] = n - 1 < 64 ? x0 : x1;
            sh.d[n - 1] = P[RR_NW - 1][n - 1];
        }
    } else {
        const int ty = (tid - 64) / RR_TX, tx = tid % RR_TX;
        double a[NI][CJ];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int r = min(ty + RR_TY * i, RR_MAX - 1);
#pragma unroll
            for (int j = 0; j < CJ; ++j) a[i][j] = ty + RR_TY * i < RR_MAX ? A[r][tx + RR_TX * j] : 0.0;
        }
        for (int k = 0; k + 1 < max(n, 2); ++k) {
            __syncthreads();
            // the rows' update, their products with x = row k; row k + 1 to wave 0
            double vc[CJ], wc[CJ], s[CJ];
#pragma unroll
            for (int j = 0; j < CJ; ++j) {
                vc[j] = vec[tx + RR_TX * j].v;
                wc[j] = vec[tx + RR_TX * j].w;
                s[j] = 0.0;
            }
            const int g = (k + 1) / RR_TY;   // the group of row k + 1; those before it are done
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                if (i < g) continue;
                const RRVec u = vec[ty + RR_TY * i];
#pragma unroll
                for (int j = 0; j < CJ; ++j) {
                    a[i][j] -= u.v * wc[j] + u.w * vc[j];
                    s[j] = fma(a[i][j], u.x, s[j]);
                }
                if (__builtin_expect(i == g, 0) && ty + RR_TY * i == k + 1)
#pragma unroll
                    for (int j = 0; j < CJ; ++j) P[RR_NW - 1][tx + RR_TX * j] = a[i][j];
            }
#pragma unroll
            for (int j = 0; j < CJ; ++j) s[j] = rr_halves(s[j]);
            if ((tid & 63) < RR_TX)
#pragma unroll
                for (int j = 0; j < CJ; ++j) P[wv - 1][tx + RR_TX * j] = s[j];
            __syncthreads();
        }
    }
    __syncthreads();
}

// Sturm count: eigenvalues of T below x, from the signs of the leading
// principal minors of T - xI (p_{i+1} = (d_i - x) p_i - e_{i-1}^2 p_{i-1}); an
// exact zero minor counts as a sign change, and with e^2 > 0 the next one is
// not zero and no change. One multiply-add per step on the chain; the signs are
// beside it. d and e^2 come by broadcast reads of LDS, which run ahead (by lane
// reads of a register, 20 cycles each on the chain of a step, the counts took
// five times as long). The pair (p_i, p_{i-1}) is rescaled by 2^-+500 every
// fourth step: T is scaled to entries below 2 and e^2 >= 2^-120, so four steps
// can neither overflow nor underflow from [2^-500, 2^500].
__device__ __forceinline__ double rr_range(double mx)   // the factor of a rescaling
{
    return mx > 0x1p+500 ? 0x1p-500 : (mx < 0x1p-500 ? 0x1p+500 : 1.0);
}

// calls f(d_i, e_{i-1}^2) for i = 1 .. n - 1 and g() after every four
template <class F, class G>
__device__ __forceinline__ void rr_chain(const double (*de)[2], int n, F f, G g)
{
    typedef double d2 __attribute__((ext_vector_type(2)));
    int i = 1;
    for (; i + 4 <= n; i += 4) {
        d2 u[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) u[k] = *reinterpret_cast<const d2 *>(de[i + k]);
#pragma unroll
        for (int k = 0; k < 4; ++k) f(u[k].x, u[k].y);
        g();
    }
    for (; i < n; ++i) f(de[i][0], de[i][1]);
    g();
}

// step(i, load(i)) for i from i0 to i1 (excluded) by dir, eight loads ahead of
// their steps (the steps store to LDS, which holds later loads back)
struct RRTrip {
    double a, b, c;
};
template <class L, class S>
__device__ __forceinline__ void rr_ahead(int i0, int i1, int dir, L load, S step)
{
    int i = i0;
    for (; (i1 - i) * dir >= 8; i += 8 * dir) {
        RRTrip t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = load(i + u * dir);
#pragma unroll
        for (int u = 0; u < 8; ++u) step(i + u * dir, t[u]);
    }
    for (; (i1 - i) * dir > 0; i += dir) step(i, load(i));
}

__device__ __forceinline__ int rr_sturm(const double (*de)[2], int n, double x)
{
    double pp = 1.0, p = de[0][0] - x;
    bool neg = !(p > 0.0);
    int c = neg;
    rr_chain(de, n,
             [&](double di, double qi) {
                 const double q = fma(di - x, p, -(qi * pp));
                 const bool ng = q < 0.0 || (q == 0.0 && !neg);
                 c += ng != neg;
                 neg = ng;
                 pp = p;
                 p = q;
             },
             [&]() {
                 const double f = rr_range(fmax(fabs(p), fabs(pp)));
                 p *= f;
                 pp *= f;
             });
    return c;
}

__global__ __launch_bounds__(RR_NT) void k_rr_eig(const double *__restrict__ G, int ldg, int m,
                                                  double *__restrict__ theta, double *__restrict__ Y, int ldy,
                                                  int32_t *__restrict__ nfallback)
{
    __shared__ RRShared sh;
    double(*A)[RR_LD] = sh.A;
    double(*Z)[RR_LD] = sh.Z;
    const int tid = threadIdx.x, lane = tid & 63;
    // the wave index as a scalar: loops over row slices are then uniform, so
    // readlane takes its index from an SGPR and the loops can be pipelined
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = m;
    int rp = 0;
    auto bmax = [&](double v) {
        const double r = rr_block_max(v, sh.red[rp]);
        rp ^= 1;
        return r;
    };

    // ---- load, symmetrise, scale by a power of two --------------------------
    if (tid == 0) sh.flag = 0;
    double amax = 0.0;
    for (int t = tid; t < RR_MAX * RR_MAX; t += RR_NT) {
        const int i = t / RR_MAX, j = t % RR_MAX;
        double v = 0.0;
        if (i < n && j < n) v = 0.5 * (G[(int64_t)i * ldg + j] + G[(int64_t)j * ldg + i]);
        A[i][j] = v;
        Z[i][j] = 0.0;
        amax = fmax(amax, fabs(v));
    }
    amax = bmax(amax);
    if (amax == 0.0) {
        for (int e = tid; e < n; e += RR_NT) theta[e] = 0.0;
        for (int t = tid; t < n * n; t += RR_NT) Y[(int64_t)(t / n) * ldy + t % n] = (t / n == t % n) ? 1.0 : 0.0;
        return;
    }
    bool bad = !isfinite(amax);
    const double scale = bad ? 1.0 : ldexp(1.0, -ilogb(amax));
    for (int t = tid; t < n * RR_MAX; t += RR_NT) {
        const int i = t / RR_MAX, j = t % RR_MAX;
        A[i][j] *= scale;
    }
    __syncthreads();

    if (!bad) {
        // ---- Householder reduction to tridiagonal form ------------------------
        if (n <= 2 * RR_TX) rr_house<5, 2>(sh, n, tid, wv);
        else rr_house<RR_RI, RR_CJ>(sh, n, tid, wv);
        for (int t = tid; t < RR_MAX * RR_MAX; t += RR_NT) Z[t / RR_MAX][t % RR_MAX] = 0.0;
        // negligible couplings split T into independent blocks (a count takes them
        // as 2^-60, far below the rounding of a T with a largest entry near 1)
        double *e2 = sh.sc[2];
        for (int i = tid; i + 1 < n; i += RR_NT) {
            double ei = sh.e[i];
            if (fabs(ei) <= DBL_EPSILON * (fabs(sh.d[i]) + fabs(sh.d[i + 1]))) ei = 0.0;
            sh.e[i] = ei;
            e2[i] = ei * ei;   // (twisted factorisations)
        }
        __syncthreads();
        for (int i = tid; i < n; i += RR_NT) {
            sh.de[i][0] = sh.d[i];
            sh.de[i][1] = i > 0 ? fmax(e2[i - 1], 0x1p-120) : 0.0;
        }

        // ---- eigenvalues by multisection ---------------------------------------
        double glo = INFINITY, ghi = -INFINITY;
        for (int i = tid; i < n; i += RR_NT) {
            const double r = (i > 0 ? fabs(sh.e[i - 1]) : 0.0) + (i + 1 < n ? fabs(sh.e[i]) : 0.0);
            glo = fmin(glo, sh.d[i] - r);
            ghi = fmax(ghi, sh.d[i] + r);
        }
        double gl = -bmax(-glo);
        double gu = bmax(ghi);
        const double tnorm = fmax(fabs(gl), fabs(gu));
        gl -= 2.0 * n * DBL_EPSILON * tnorm + 2.0 * DBL_MIN;
        gu += 2.0 * n * DBL_EPSILON * tnorm + 2.0 * DBL_MIN;
        const double tolabs = 2.0 * DBL_EPSILON * tnorm;
        double *lo = sh.sc[0], *hi = sh.sc[1];
        int *cnt = sh.u.cnt;
        if (tid < RR_G) {   // RR_G shifts over the Gershgorin interval (whole waves)
            const double fr = (double)(tid + 1) / (double)(RR_G + 1);
            cnt[tid] = rr_sturm(sh.de, n, fma(gu - gl, fr, gl));
        }
        __syncthreads();
        if (tid < n) {
            // a transition cnt[a] <= j < cnt[b] (virtual ends gl, gu) by bisection on
            // the index; it holds even where rounding makes the counts non-monotone
            int a = -1, b = RR_G;
            while (b - a > 1) {
                const int mid = (a + b) >> 1;
                if (cnt[mid] <= tid) a = mid;
                else b = mid;
            }
            const double l = a < 0 ? gl : fma(gu - gl, (double)(a + 1) / (double)(RR_G + 1), gl);
            const double h = b >= RR_G ? gu : fma(gu - gl, (double)(b + 1) / (double)(RR_G + 1), gl);
            if (!(l < h)) sh.flag = 1;
            lo[tid] = l;
            hi[tid] = h;
            // start of the Laguerre iteration: the idx-th of the k eigenvalues in
            // the interval starts at fraction (idx + 1/2) / k of it
            const int cl = a < 0 ? 0 : cnt[a], ch = b >= RR_G ? n : cnt[b];
            sh.sc[3][tid] = (tid - cl + 0.5) / (double)max(ch - cl, 1);
        }
        __syncthreads();
        // Laguerre's method on P(x) = det(T - xI) from the middle of each isolating
        // interval (waves 0-1, one eigenvalue per lane): P, P' and P'' from the
        // recurrence of the leading minors and its derivatives, rescaled together
        // (three independent multiply-adds a step where the pivots' quotients were
        // a chain of eight); cubic convergence at simple roots. The step is
        // n P / (P' +- sqrt((n - 1) ((n - 1) P'^2 - n P P''))), the larger divisor.
        // A step leaving the interval, a non-finite value or no convergence in
        // 16 steps, or a result whose Sturm counts do not bracket index j,
        // leaves the interval to the multisection below.
        if (wv < 2) {
            const int j = tid, jc = j < n ? j : 0;
            const double l0 = lo[jc], h0 = hi[jc], nd = (double)n;
            double x = fma(h0 - l0, fmin(fmax(sh.sc[3][jc], 0.0), 1.0), l0);
            bool conv = j >= n, ok = false;
            for (int it = 0; it < 16; ++it) {
                if (__all(conv)) break;
                double p = sh.de[0][0] - x, pp = 1.0, p1 = -1.0, pp1 = 0.0, p2 = 0.0, pp2 = 0.0;
                rr_chain(sh.de, n,
                         [&](double di, double qi) {
                             const double t = di - x;
                             const double q = fma(t, p, -(qi * pp));
                             const double q1 = fma(t, p1, -fma(qi, pp1, p));
                             const double q2 = fma(t, p2, -fma(qi, pp2, 2.0 * p1));
                             pp = p;
                             pp1 = p1;
                             pp2 = p2;
                             p = q;
                             p1 = q1;
                             p2 = q2;
                         },
                         [&]() {
                             const double f = rr_range(fmax(fmax(fmax(fabs(p), fabs(pp)), fmax(fabs(p1), fabs(pp1))),
                                                            fmax(fabs(p2), fabs(pp2))));
                             p *= f;
                             pp *= f;
                             p1 *= f;
                             pp1 *= f;
                             p2 *= f;
                             pp2 *= f;
                         });
                if (!conv) {
                    // brought near 1: the squares are in range
                    const int ex = -ilogb(fmax(fmax(fabs(p), fabs(p1)), fabs(p2)));
                    p = ldexp(p, ex);
                    p1 = ldexp(p1, ex);
                    p2 = ldexp(p2, ex);
                    const double g = (nd - 1.0) * p1;
                    const double sq = sqrt(fmax(g * g - (nd - 1.0) * nd * (p * p2), 0.0));
                    const double den = p1 >= 0.0 ? p1 + sq : p1 - sq;
                    const double a = nd * p / den;
                    const double xn = x - a;
                    if (!(den != 0.0) || !isfinite(xn) || !(xn >= l0 && xn <= h0)) {
                        conv = true;
                    } else {
                        x = xn;
                        if (fabs(a) <= 2.0 * DBL_EPSILON * tnorm) {
                            conv = true;
                            ok = true;
                        }
                    }
                }
            }
            const double dl = 4.0 * DBL_EPSILON * tnorm;
            const int c1 = rr_sturm(sh.de, n, x - dl);
            const int c2 = rr_sturm(sh.de, n, x + dl);
            ok = ok && c1 <= j && j < c2;
            if (j < n && ok) {
                lo[j] = x;
                hi[j] = x;
            }
            // a start near it for the others: a wider bracket of the last iterate
            if (__any(j < n && !ok)) {
                const double l1 = fmax(l0, x - 0x1p-42 * tnorm), h1 = fmin(h0, x + 0x1p-42 * tnorm);
                const int c3 = rr_sturm(sh.de, n, l1), c4 = rr_sturm(sh.de, n, h1);
                if (j < n && !ok && l1 < h1) {
                    if (c3 <= j) lo[j] = l1;
                    else hi[j] = l1;
                    if (j < c4) hi[j] = fmin(hi[j], h1);
                    else lo[j] = h1;
                    if (!(lo[j] < hi[j])) {   // (counts out of order)
                        lo[j] = l0;
                        hi[j] = h0;
                    }
                }
            }
        }
        // multisection for what Laguerre left: the open eigenvalues (ballot of
        // waves 0-1) share the RR_G shifts, up to 64 each
        auto open = [&](int j) {
            return (hi[j] - lo[j]) > fmax(tolabs, 2.0 * DBL_EPSILON * fmax(fabs(lo[j]), fabs(hi[j])));
        };
        for (int pass = 0; pass < 96; ++pass) {
            __syncthreads();
            if (wv < 2) {
                const unsigned long long mk = __ballot(tid < n && open(tid));
                if (lane == 0) sh.open_mask[wv] = mk;
            }
            __syncthreads();
            const unsigned long long m0 = sh.open_mask[0], m1 = sh.open_mask[1];
            const int c0 = __popcll(m0), na = c0 + __popcll(m1);
            if (na == 0) break;
            // a power of two of shifts each, in one wave: the counts meet in a ballot
            int per = 64;
            while (per * na > RR_G) per >>= 1;
            const int slot = tid / per, sft = tid & (per - 1);
            int j = 0, cnt_j = 0;
            double l0 = 0.0, h0 = 0.0, x = 0.0;
            if (slot < na) {
                // eigenvalue of this slot: the slot-th set bit of (m0, m1)
                unsigned long long mk = slot < c0 ? m0 : m1;
                for (int q = slot < c0 ? slot : slot - c0; q > 0; --q) mk &= mk - 1;
                j = __builtin_ctzll(mk) + (slot < c0 ? 0 : 64);
                l0 = lo[j];
                h0 = hi[j];
                x = fma(h0 - l0, (double)(sft + 1) / (double)(per + 1), l0);
                cnt_j = rr_sturm(sh.de, n, x);
            }
            const unsigned long long le = __ballot(slot < na && cnt_j <= j);
            const unsigned long long all = per == 64 ? ~0ull : (1ull << per) - 1;
            const unsigned long long mine = (le >> (lane & ~(per - 1))) & all;
            if (slot < na && sft == 0) {   // the last shift with a count <= j, the first with one > j
                auto at = [&](int q) { return fma(h0 - l0, (double)(q + 1) / (double)(per + 1), l0); };
                if (mine) lo[j] = fmax(l0, at(63 - __builtin_clzll(mine)));
                if (mine != all) hi[j] = fmin(h0, at(__builtin_ctzll(~mine)));
            }
        }
        if (tid < n) sh.lam[tid] = 0.5 * (lo[tid] + hi[tid]);
        __syncthreads();

        // ---- eigenvectors of T: twisted factorisations, one per thread ------
        double *vinv = sh.sc[0];   // reciprocal norms
        if (wv < 2) {   // d, e, e^2 by broadcast reads: the loops below are wave-uniform
            const int j = tid, jc = j < n ? j : RR_MAX;   // idle lanes: the padding column
            const double lj = sh.lam[j < n ? j : 0];
            // top-down pivots delta+ kept in column j
            double dp = sh.d[0] - lj;
            if (dp == 0.0) dp = -DBL_MIN;
            Z[0][jc] = dp;
            rr_ahead(1, n, 1, [&](int i) { return RRTrip{sh.d[i], e2[i - 1], 0.0}; },
                     [&](int i, const RRTrip &t) {
                         dp = (t.a - lj) - t.b * rr_recip(dp);
                         if (dp == 0.0) dp = -DBL_MIN;
                         Z[i][jc] = dp;
                     });
            // bottom-up pivots delta-, twist index of smallest |gamma|
            double dm = sh.d[n - 1] - lj;
            if (dm == 0.0) dm = -DBL_MIN;
            double best = fabs(Z[n - 1][jc]);
            int r = n - 1;
            rr_ahead(n - 2, -1, -1, [&](int i) { return RRTrip{sh.d[i], e2[i], Z[i][jc]}; },
                     [&](int i, const RRTrip &t) {
                         const double di = t.a - lj;
                         dm = di - t.b * rr_recip(dm);
                         if (dm == 0.0) dm = -DBL_MIN;
                         const double g = fabs(t.c + dm - di);
                         if (g < best) {
                             best = g;
                             r = i;
                         }
                     });
            // (the two ends of this wave's twist indices bound the loops)
            int rlo = j < n ? r : n - 1, rhi = j < n ? r : 0;
            for (int o = 32; o > 0; o >>= 1) {
                rlo = min(rlo, __shfl_xor(rlo, o));
                rhi = max(rhi, __shfl_xor(rhi, o));
            }
            rlo = __builtin_amdgcn_readfirstlane(rlo);
            rhi = __builtin_amdgcn_readfirstlane(rhi);
            // ratios below the twist: z_{i+1} / z_i = -e_i / delta-_{i+1}
            dm = sh.d[n - 1] - lj;
            if (dm == 0.0) dm = -DBL_MIN;
            rr_ahead(n - 2, rlo - 1, -1, [&](int i) { return RRTrip{sh.d[i], sh.e[i], 0.0}; },
                     [&](int i, const RRTrip &t) {
                         const double rho = -t.b * rr_recip(dm);
                         if (i >= r) Z[i + 1][jc] = rho;
                         dm = (t.a - lj) + t.b * rho;
                         if (dm == 0.0) dm = -DBL_MIN;
                     });
            double nn = 1.0, z = 1.0;
            rr_ahead(rlo, n - 1, 1, [&](int i) { return RRTrip{Z[i + 1][jc], 0.0, 0.0}; },
                     [&](int i, const RRTrip &t) {
                         if (i >= r) {
                             z *= t.a;
                             nn = fma(z, z, nn);
                             Z[i + 1][jc] = z;
                         }
                     });
            // above the twist: z_i = -(e_i / delta+_i) z_{i+1}
            z = 1.0;
            rr_ahead(rhi - 1, -1, -1, [&](int i) { return RRTrip{-(sh.e[i] * rr_recip(Z[i][jc])), 0.0, 0.0}; },
                     [&](int i, const RRTrip &t) {
                         if (i < r) {
                             z *= t.a;
                             nn = fma(z, z, nn);
                             Z[i][jc] = z;
                         }
                     });
            Z[r][jc] = 1.0;
            const double inv = 1.0 / sqrt(nn);
            if (j < n) {
                vinv[j] = inv;
                if (!(nn > 0.0) || !isfinite(nn) || !(best * inv <= 1e-10 * tnorm)) sh.flag = 1;
            }
        }
        __syncthreads();
        for (int t = tid; t < n * RR_MAX; t += RR_NT) {
            const int c = t % RR_MAX;
            if (c < n) Z[t / RR_MAX][c] *= vinv[c];
        }
        {
            // ---- clusters: modified Gram-Schmidt, two passes (one wave) ------
            const int close = tid + 1 < n && sh.lam[tid + 1] - sh.lam[tid] < 1e-3 * tnorm;
            if (__syncthreads_or(close) && wv == 0) {
                int j0 = 0;
                while (j0 < n) {
                    int j1 = j0;
                    while (j1 + 1 < n && sh.lam[j1 + 1] - sh.lam[j1] < 1e-3 * tnorm) ++j1;
                    for (int a = j0 + 1; a <= j1; ++a) {
                        for (int rep = 0; rep < 2; ++rep)
                            for (int b = j0; b < a; ++b) {
                                double s = 0.0;
                                for (int i = lane; i < n; i += 64) s += Z[i][b] * Z[i][a];
                                s = rr_wsum(s);
                                for (int i = lane; i < n; i += 64) Z[i][a] -= s * Z[i][b];
                            }
                        double nn = 0.0;
                        for (int i = lane; i < n; i += 64) nn += Z[i][a] * Z[i][a];
                        nn = rr_wsum(nn);
                        if (!(nn >= 1e-4)) {
                            if (lane == 0) sh.flag = 1;
                            nn = 1.0;
                        }
                        const double inv = 1.0 / sqrt(nn);
                        for (int i = lane; i < n; i += 64) Z[i][a] *= inv;
                    }
                    j0 = j1 + 1;
                }
            }
            __syncthreads();
        }

        // ---- back-transformation Z <- H_0 H_1 ... H_{n-3} Z --------------------
        // the reflector rows first become the vectors themselves (v_{k+1} = 1,
        // v_r = x_r hinv below)
        for (int t = tid; t < n * n; t += RR_NT) {
            const int k = t / n, r = t % n;
            if (k + 2 < n && r >= k + 1 && sh.tau[k] != 0.0) A[k][r] = r == k + 1 ? 1.0 : A[k][r] * sh.hinv[k];
        }
        __syncthreads();
        {
            // blocks of 16 reflectors k0..k0+15 as I - V T V^T (T upper triangular,
            // T_ii = tau_i, T[0:i, i] = -tau_i T[0:i, 0:i] V[:, 0:i]^T v_i), applied
            // last block first: Z <- Z - V (T (V^T Z)) on FP64 MFMA 16x16x4. Wave w
            // < nt takes the 16 columns 16w.. of Z: W = V^T Z_w, W' = T W (the MFMA
            // result items are exactly the next B operand: item v of lane l is row
            // l/16 + 4v), Z_w -= V W'; a wave touches only its own columns of Z.
            // Meanwhile the last wave (never one of the nt <= 6 column waves) forms
            // S = V^T V and T of the next block into the other of two buffers (lane
            // j owns row j of T, so the recurrence needs no barrier): one barrier
            // per block.
            const int nref = n - 2, nt = (n + 15) / 16, ks = (n + 3) / 4;
            const int nblk = nref > 0 ? (nref + 15) / 16 : 0, tw = RR_NW - 1;
            double *Tb0 = &sh.sc[0][0], *Tb1 = Tb0 + 256;   // 16 x 16 each (sc is free here)
            double *Sm = sh.u.dbl;                           // 16 x 16
            const int li = lane & 15, lk = lane >> 4;
            // entry r of reflector k with tau_k = tk (zero outside the vector, or if
            // no reflection)
            auto vv = [&](int k, double tk, int r) -> double {
                return (tk != 0.0 && r > k && r < n) ? A[k][r] : 0.0;
            };
            auto tau_of = [&](int k) -> double { return k < nref ? sh.tau[k] : 0.0; };
            auto make_t = [&](int k0, double *Tm) {
                const int s_lo = (k0 + 1) / 4;   // rows r <= k0 hold no entry of the block
                const double tl = tau_of(k0 + li);
                rr_dx4 a0 = {0.0, 0.0, 0.0, 0.0}, a1 = {0.0, 0.0, 0.0, 0.0};
                int s4 = s_lo;
                for (; s4 + 1 < ks; s4 += 2) {
                    const double x0 = vv(k0 + li, tl, 4 * s4 + lk), x1 = vv(k0 + li, tl, 4 * s4 + 4 + lk);
                    a0 = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, x0, a0, 0, 0, 0);
                    a1 = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, x1, a1, 0, 0, 0);
                }
                if (s4 < ks) {
                    const double x0 = vv(k0 + li, tl, 4 * s4 + lk);
                    a0 = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, x0, a0, 0, 0, 0);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) Sm[(lk + 4 * v) * 16 + li] = a0[v] + a1[v];
                // T by columns; lane j < 16 owns row j; T[j][l] = 0 for l < j, so the
                // inner sum runs over l < i for every lane
                const int j = lane & 15;
                for (int i = 0; i < 16; ++i) {
                    double y0 = 0.0, y1 = 0.0;
                    int l = 0;
                    for (; l + 1 < i; l += 2) {
                        y0 = fma(Tm[j * 16 + l], Sm[l * 16 + i], y0);
                        y1 = fma(Tm[j * 16 + l + 1], Sm[(l + 1) * 16 + i], y1);
                    }
                    if (l < i) y0 = fma(Tm[j * 16 + l], Sm[l * 16 + i], y0);
                    const double ti = tau_of(k0 + i);
                    if (lane < 16) Tm[j * 16 + i] = j < i ? -ti * (y0 + y1) : (j == i ? ti : 0.0);
                }
            };
            if (nblk > 0 && wv == tw) make_t(16 * (nblk - 1), Tb0);
            __syncthreads();
            for (int blk = nblk - 1, buf = 0; blk >= 0; --blk, buf ^= 1) {
                const int k0 = 16 * blk;
                double *Tcur = buf ? Tb1 : Tb0;
                if (wv == tw && blk > 0) make_t(16 * (blk - 1), buf ? Tb0 : Tb1);
                if (wv < nt) {
                    const int c0 = 16 * wv, s_lo = (k0 + 1) / 4;
                    const double tl = tau_of(k0 + li);
                    rr_dx4 w0 = {0.0, 0.0, 0.0, 0.0}, w1 = {0.0, 0.0, 0.0, 0.0};
                    const bool cok = c0 + li < n;
                    int s4 = s_lo;
                    for (; s4 + 1 < ks; s4 += 2) {
                        const int r = 4 * s4 + lk;
                        const double z0 = (r < n && cok) ? Z[r][c0 + li] : 0.0;
                        const double z1 = (r + 4 < n && cok) ? Z[r + 4][c0 + li] : 0.0;
                        w0 = __builtin_amdgcn_mfma_f64_16x16x4f64(vv(k0 + li, tl, r), z0, w0, 0, 0, 0);
                        w1 = __builtin_amdgcn_mfma_f64_16x16x4f64(vv(k0 + li, tl, r + 4), z1, w1, 0, 0, 0);
                    }
                    if (s4 < ks) {
                        const int r = 4 * s4 + lk;
                        const double z0 = (r < n && cok) ? Z[r][c0 + li] : 0.0;
                        w0 = __builtin_amdgcn_mfma_f64_16x16x4f64(vv(k0 + li, tl, r), z0, w0, 0, 0, 0);
                    }
                    rr_dx4 accW;
#pragma unroll
                    for (int v = 0; v < 4; ++v) accW[v] = w0[v] + w1[v];
                    rr_dx4 accP = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        accP = __builtin_amdgcn_mfma_f64_16x16x4f64(Tcur[li * 16 + 4 * q + lk], accW[q], accP, 0, 0, 0);
                    double td[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) td[q] = tau_of(k0 + 4 * q + lk);
                    for (int rt = (k0 + 1) / 16; rt < nt; ++rt) {
                        const int r0 = 16 * rt;
                        rr_dx4 accD = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            accD = __builtin_amdgcn_mfma_f64_16x16x4f64(vv(k0 + 4 * q + lk, td[q], r0 + li), accP[q],
                                                                        accD, 0, 0, 0);
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int row = r0 + lk + 4 * v;
                            if (row < n && cok) Z[row][c0 + li] -= accD[v];
                        }
                    }
                }
                __syncthreads();
            }
        }

        // ---- Newton-Schulz: S = Z^T Z into A, then Y = Z (3I - S) / 2 ---------
        const int nt = (n + 15) / 16, kq = (n + 3) / 4;
        for (int tile = wv; tile < nt * nt; tile += RR_NW) {
            const int a0 = (tile / nt) * 16, b0 = (tile % nt) * 16;
            rr_dx4 acc = {0.0, 0.0, 0.0, 0.0};
            for (int kk = 0; kk < kq; ++kk) {
                const int i = kk * 4 + (lane >> 4);
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Z[i][a0 + (lane & 15)], Z[i][b0 + (lane & 15)], acc, 0,
                                                           0, 0);
            }
            for (int q = 0; q < 4; ++q) A[a0 + (lane >> 4) + 4 * q][b0 + (lane & 15)] = acc[q];
        }
        __syncthreads();
        double defect = 0.0;
        for (int t = tid; t < n * RR_MAX; t += RR_NT) {
            const int a = t / RR_MAX, b = t % RR_MAX;
            if (b < n) defect = fmax(defect, fabs(A[a][b] - (a == b ? 1.0 : 0.0)));
        }
        defect = bmax(defect);
        if (!(defect <= 1e-8)) sh.flag = 1;
        for (int t = tid; t < RR_MAX * RR_MAX; t += RR_NT) {
            const int a = t / RR_MAX, b = t % RR_MAX;
            A[a][b] = (a == b ? 1.5 : 0.0) - 0.5 * A[a][b];
        }
        __syncthreads();
        if (!sh.flag) {
            for (int tile = wv; tile < nt * nt; tile += RR_NW) {
                const int i0 = (tile / nt) * 16, b0 = (tile % nt) * 16;
                rr_dx4 acc = {0.0, 0.0, 0.0, 0.0};
                for (int kk = 0; kk < kq; ++kk) {
                    const int a = kk * 4 + (lane >> 4);
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Z[i0 + (lane & 15)][a], A[a][b0 + (lane & 15)], acc,
                                                               0, 0, 0);
                }
                for (int q = 0; q < 4; ++q) {
                    const int i = i0 + (lane >> 4) + 4 * q, b = b0 + (lane & 15);
                    if (i < n && b < n) Y[(int64_t)i * ldy + b] = acc[q];
                }
            }
            for (int e = tid; e < n; e += RR_NT) theta[e] = sh.lam[e] / scale;
            return;
        }
    }
    // ---- fallback: cyclic Jacobi on G ------------------------------------------
    if (tid == 0 && nfallback) atomicAdd(nfallback, 1);
    rr_jacobi(sh, G, ldg, m, theta, Y, ldy, 40);
}

hipError_t launch_jacobi_eig(const double *G, int ldg, int m, double *theta, double *Y, int ldy, hipStream_t st)
{
    if (m <= 0 || m > RR_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_jacobi_eig, dim3(1), dim3(RR_NT), 0, st, G, ldg, m, theta, Y, ldy, 40);
    return hipGetLastError();
}

hipError_t launch_rr_eig(const double *G, int ldg, int m, double *theta, double *Y, int ldy, int32_t *nfallback,
                         hipStream_t st)
{
    if (m <= 0 || m > RR_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_rr_eig, dim3(1), dim3(RR_NT), 0, st, G, ldg, m, theta, Y, ldy, nfallback);
    return hipGetLastError();
}

}  // namespace cch
