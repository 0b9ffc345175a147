// Every eigenpair of a dense real symmetric matrix in FP64 on one GPU (the
// paper's Sec. 3.2 notes that often all eigenvectors are wanted and a dense
// diagonaliser is used then):
//   1. Householder tridiagonalisation Q^T A Q = T, one reflector per column,
//      blocked in panels of TRD_NB columns with lazy updates: per column
//      one kernel for the reflector, its w and the next corrected column, and
//      the product of the trailing block with that column (the HBM-bound part:
//      from the lower triangle in tiles while the block has at least
//      TRD_TILE_MIN rows, by whole rows below that), and one rank-2 TRD_NB
//      FP64 MFMA update of the trailing block per panel.
//   2. Eigenvalues of T by multisection on Sturm counts, 8 lanes each.
//   3. Eigenvectors of T by twisted factorisations, one thread each, with
//      modified Gram-Schmidt (and inverse iteration for vectors that
//      collapse) inside clusters of close eigenvalues, one workgroup each.
//   4. Back-transformation Z = Q Z_T in blocks of 128 reflectors, each as
//      I - V T V^T (compact WY) by three FP64 MFMA products.
#include <algorithm>
#include <cmath>

#include "ccham_internal.h"

namespace cch {

// ---------------------------------------------------------------------------
// general FP64 MFMA product C = alpha A B + beta C (row-major C)
//   A(i, k) = A[i * sai + k * sak], B(k, j) = B[k * sbk + j * sbj]
// 64 x 64 tile per workgroup (4 waves of 32 x 32, on the 4x4x4 form: it
// issues faster per flop than 16x16x4 on this chip), K staged through LDS in
// slices of 16 (the next slice loaded into registers during the products);
// loads follow whichever index of an operand has stride 1; C, when the
// product adds to it, is loaded at entry
// ---------------------------------------------------------------------------
constexpr int EG_T = 64, EG_K = 16;

// With P != nullptr the K range is split over blockIdx.z (kc each) and each
// split writes its unscaled partial product to P[z][M][N]; k_eig_gemm_sum adds
// the splits in order and applies alpha and beta (deterministic).
__global__ __launch_bounds__(256) void k_eig_gemm(int M, int N, int K, double alpha, const double *__restrict__ A,
                                                  int64_t sai, int64_t sak, const double *__restrict__ B, int64_t sbk,
                                                  int64_t sbj, double beta, double *__restrict__ C, int64_t ldc,
                                                  int kc, double *__restrict__ P, int lowq)
{
    // lowq >= 0: only the tiles on and below the diagonal, and every tile of
    // the square of tile rows and columns >= lowq
    if (lowq >= 0 && (int)blockIdx.x > (int)blockIdx.y && ((int)blockIdx.x < lowq || (int)blockIdx.y < lowq)) return;
    __shared__ double As[EG_K][EG_T + 1], Bs[EG_K][EG_T + 1];
    const int i0 = blockIdx.y * EG_T, j0 = blockIdx.x * EG_T;
    const int kb0 = P ? (int)blockIdx.z * kc : 0, kb1 = P ? min(K, kb0 + kc) : K;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int wm = wv & 1, wn = wv >> 1;
    const bool a_kfast = sak == 1, b_jfast = sbj == 1;
    // C of this thread's outputs, loaded at entry when the product adds to it
    const bool addc = P == nullptr && beta != 0.0;
    // 4x4x4 FP64 MFMA, four blocks with the same A: an instruction multiplies
    // 4 rows (A at lane i + 16 k, any block) by 16 columns (B at lane
    // j + 16 k), the result D[i][j] at lane j + 16 i. A wave's 32 x 32 tile is
    // 8 row quads x 2 column groups.
    double cin[8][2];
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int i = i0 + wm * 32 + 4 * a + (lane >> 4);
            const int j = j0 + wn * 32 + 16 * b + (lane & 15);
            cin[a][b] = addc && i < M && j < N ? C[(int64_t)i * ldc + j] : 0.0;
        }
    double acc[8][2];
#pragma unroll
    for (int a = 0; a < 8; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = 0.0;
    // the K slices pass through registers: the next one is loaded while the
    // current one is multiplied from LDS
    double ra[4], rb[4];
    auto load = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            int ii, kk;
            if (a_kfast) { kk = t & 15; ii = (t >> 4) + 16 * u; }
            else { ii = t & 63; kk = (t >> 6) + 4 * u; }
            const int i = i0 + ii, k = k0 + kk;
            ra[u] = (i < M && k < kb1) ? A[(int64_t)i * sai + (int64_t)k * sak] : 0.0;
            int jj, kb;
            if (b_jfast) { jj = t & 63; kb = (t >> 6) + 4 * u; }
            else { kb = t & 15; jj = (t >> 4) + 16 * u; }
            const int j = j0 + jj, kq = k0 + kb;
            rb[u] = (j < N && kq < kb1) ? B[(int64_t)kq * sbk + (int64_t)j * sbj] : 0.0;
        }
    };
    if (kb0 < kb1) load(kb0);
    for (int k0 = kb0; k0 < kb1; k0 += EG_K) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            int ii, kk;
            if (a_kfast) { kk = t & 15; ii = (t >> 4) + 16 * u; }
            else { ii = t & 63; kk = (t >> 6) + 4 * u; }
            As[kk][ii] = ra[u];
            int jj, kb;
            if (b_jfast) { jj = t & 63; kb = (t >> 6) + 4 * u; }
            else { kb = t & 15; jj = (t >> 4) + 16 * u; }
            Bs[kb][jj] = rb[u];
        }
        __syncthreads();
        if (k0 + EG_K < kb1) load(k0 + EG_K);
#pragma unroll
        for (int ks = 0; ks < EG_K; ks += 4) {
            const int kk = ks + (lane >> 4);
            double af[8], bf[2];
#pragma unroll
            for (int a = 0; a < 8; ++a) af[a] = As[kk][wm * 32 + 4 * a + (lane & 3)];
#pragma unroll
            for (int b = 0; b < 2; ++b) bf[b] = Bs[kk][wn * 32 + 16 * b + (lane & 15)];
#pragma unroll
            for (int a = 0; a < 8; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_4x4x4f64(af[a], bf[b], acc[a][b], 0, 0, 0);
        }
        __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        const int i = i0 + wm * 32 + 4 * a + (lane >> 4);
        if (i >= M) continue;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int j = j0 + wn * 32 + 16 * b + (lane & 15);
            if (j >= N) continue;
            if (P) P[((int64_t)blockIdx.z * M + i) * N + j] = acc[a][b];
            else C[(int64_t)i * ldc + j] = alpha * acc[a][b] + (beta == 0.0 ? 0.0 : beta * cin[a][b]);
        }
    }
}

__global__ void k_eig_gemm_sum(int M, int N, int ns, const double *__restrict__ P, double alpha, double beta,
                               double *__restrict__ C, int64_t ldc)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)M * N) return;
    double s = 0.0;
    for (int z = 0; z < ns; ++z) s += P[(int64_t)z * M * N + e];
    double *c = C + (e / N) * ldc + e % N;
    *c = alpha * s + (beta == 0.0 ? 0.0 : beta * *c);
}

// P (optional, p_cap doubles): split-K scratch for products with few output
// tiles and a long K (the Gram and projection products of the
// back-transformation)
hipError_t launch_eig_gemm(int M, int N, int K, double alpha, const double *A, int64_t sai, int64_t sak,
                           const double *B, int64_t sbk, int64_t sbj, double beta, double *C, int64_t ldc,
                           hipStream_t st, double *P, int64_t p_cap, int lowq)
{
    if (M <= 0 || N <= 0) return hipSuccess;
    const dim3 g((N + EG_T - 1) / EG_T, (M + EG_T - 1) / EG_T);
    const int64_t tiles = (int64_t)g.x * g.y;
    int ns = 1;
    if (P && lowq < 0 && tiles < 512 && K >= 1024) {
        ns = (int)std::min<int64_t>({(K + 255) / 256, std::max<int64_t>(1, 1024 / tiles), 64});
        ns = (int)std::min<int64_t>(ns, p_cap / ((int64_t)M * N));
    }
    if (ns <= 1) {
        hipLaunchKernelGGL(k_eig_gemm, g, dim3(256), 0, st, M, N, K, alpha, A, sai, sak, B, sbk, sbj, beta, C, ldc,
                           K, (double *)nullptr, lowq);
        return hipGetLastError();
    }
    const int kc = ((K + ns - 1) / ns + EG_K - 1) / EG_K * EG_K;
    ns = (K + kc - 1) / kc;
    hipLaunchKernelGGL(k_eig_gemm, dim3(g.x, g.y, ns), dim3(256), 0, st, M, N, K, alpha, A, sai, sak, B, sbk, sbj,
                       beta, C, ldc, kc, P, -1);
    const int64_t e = (int64_t)M * N;
    hipLaunchKernelGGL(k_eig_gemm_sum, dim3((unsigned)((e + 255) / 256)), dim3(256), 0, st, M, N, ns, P, alpha, beta,
                       C, ldc);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 1. tridiagonalisation (lower triangle convention: reflector j annihilates
//    A[j+2:, j]; v_j[j+1] = 1 is stored explicitly in A[j+1][j] and below),
//    blocked with lazy updates: in a panel of TRD_NB columns the trailing
//    matrix A_0 is only read. The matrix after the panel's reflectors k < i is
//    A_0 - sum_k (v_k w_k^T + w_k v_k^T), so column j is read from A_0 and
//    corrected, and its product A_j v_j = A_0 v_j - sum_k (v_k (w_k . v_j) +
//    w_k (v_k . v_j)); one rank-2 TRD_NB product (FP64 MFMA) updates the
//    trailing block at the end of the panel. w_j = p - (tau_j / 2)(p . v_j) v_j
//    with p = tau_j A_j v_j.
// Two launches per column, each spread over the rows; a workgroup never waits
// for another one. The product of column j is taken with the corrected column
// x itself, before its reflector is known: with v_j = scale x below row j + 1
// and v_j[j + 1] = 1, A_0 v_j = A_0[:, j + 1] + scale A_0[:, j + 2:] x, so the
// product kernels read nothing but A_0 and x and also leave partial sums of
// x . A_0 x. The column kernel of column j + 1 then has everything: from the
// partial sums of its predecessor (sigma = |x|^2 over the part to annihilate,
// and the panel's vectors times x) every workgroup forms the reflector j and z
// alike, p . v = tau (v . A_0 v - 2 sum_k (v_k . v)(w_k . v)) follows without a
// further pass over the rows, and the workgroup finishes v_j, p and w_j for its
// rows, corrects column j + 1 and stores the partial sums for the next one.
// The range: sigma is quadratic in x and x . A_0 x cubic in the matrix. A whose
// largest entry lies outside [2^-96, 2^97) is first scaled by a power of two
// (trd_shift), and x is stored times 2^TRD_XS, which leaves v and tau as they
// are. sigma then stays below 2^870 and x . A_0 x below 2^980 (entries grow to n
// times the largest one, n < 2^16), and of a sigma from TRD_SIG_MIN = 2^-900 on
// neither loses a bit to underflow (the terms of x . A_0 x are 2^-996 then, their
// rounding 2^-1075). A smaller sigma, entries below 2^-770, counts as zero: a
// reflector formed from squares that have lost their bits would not be orthogonal.
// For trailing blocks of at least TRD_TILE_MIN rows the product reads only the
// lower triangle, in tiles, whose row and column sums the column kernel adds.
// panel buffers (ldp doubles a row): PV rows 2k, 2k + 1 = v_k, w_k; PW rows
// 2k, 2k + 1 = w_k, v_k (the update is A -= PV^T PW over 2 nb rows); PVt the
// same values by matrix row (PVt[r][d] = PV[d][r]: a row's panel entries are
// contiguous for the kernels that read them per row); z[2k] = v_k . v_j,
// z[2k + 1] = w_k . v_j. Entries below the reflector's first row are never
// read.
// ---------------------------------------------------------------------------

// sum over the 64 lanes of a whole wave (DPP: a chain of a shuffle per step
// through LDS took a third of a microsecond)
__device__ __forceinline__ double wave_sum(double x) { return rr_wsum(x); }

__device__ __forceinline__ double blk_sum(double x, double *red)
{
    // sum over the 256 threads of a workgroup (red: 4 doubles of LDS)
    x = wave_sum(x);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}

__device__ __forceinline__ double quad_sum(double x)   // over lanes 4 a .. 4 a + 3, to each of them
{
    x += rr_dpp<0xb1, 0xf, 0xf>(x);          // lanes 1, 0, 3, 2
    return x + rr_dpp<0x4e, 0xf, 0xf>(x);    // lanes 2, 3, 0, 1
}

// The column kernel of column c, panel index i (so many reflectors of the panel
// before it), rows c + TRD_CR blockIdx.x + (0 .. TRD_CR - 1), four threads a
// row. fin: finish reflector j = c - 1 (panel index i - 1): v_j, w_j into the
// panel buffers and column j of A, e[j], tau[j]. col: column c of the current
// matrix into x, d[c], and this workgroup's partial sums [sigma, PV[0] . x, ...,
// PV[2i - 1] . x] over its rows >= c + 2 into part1. TILED: the product left the
// sums of T tile rows (counted from row trd_base(c)) instead of y; rowc: column
// c may be read as row c. g2: partial sums in part2.
// Bound by latency: one level of loads (the row's panel pairs, 16 bytes each,
// eight per thread; its tile sums; the partial sums), four barriers, and the
// fetch of its own code, which every launch pays anew (unrolled further, with
// a branch around each load, it was 10.7 KB long and half a microsecond
// slower; the tiled form, with more to add up, gains from the longer batches).
// Measured: 5.8 us at n = 301, 8.5 us with tiles (n from 8000 to 3072), where
// three launches a column took 8.0 and 9.1 us for this part, and 4.8 us more
// for the tile sums; a column with its product 8.7 instead of 12.3 us at
// n = 301 and 30 instead of 42 at n = 8000 to 3072
constexpr int TRD_XS = 320;                // x is stored times 2^TRD_XS
constexpr double TRD_SIG_MIN = 0x1p-900;   // a smaller |x|^2 counts as zero
constexpr int TRD_CT = 4 * TRD_CR;         // threads of the column kernel
constexpr int TRD_CW = TRD_CT / 64;
constexpr int TRD_LS = 2 * TRD_NB + 8;     // LDS row stride of the panel rows (two rows apart: other banks)
static_assert(TRD_CR * 64 / TRD_CT == 16, "rows per wave");

template <bool TILED>
__global__ __launch_bounds__(TRD_CT) void k_trd_col(double *__restrict__ A, int64_t lda, int n, int c, int i, int fin,
                                                    int col, int T, int rowc, int g2, TrdVec V, TrdPanel P)
{
    typedef double d2 __attribute__((ext_vector_type(2)));
    __shared__ double S[TRD_CR * TRD_LS];      // the workgroup's panel rows
    __shared__ double red[TRD_CW][2 * TRD_NB + 1];
    __shared__ double p1[4][128];              // partial sums of sigma, PV[q] . x_j (four groups)
    __shared__ double pv1[2 * TRD_NB], zs[2 * TRD_NB];   // PV at row c; z
    __shared__ double xs[TRD_CR];
    __shared__ double r2[TRD_CW], sc;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int rl = t >> 2, qd = t & 3;
    const int r = c + (int)blockIdx.x * TRD_CR + rl, rr = min(r, n - 1);
    const bool in = r < n;
    const int j = c - 1, np = fin ? i - 1 : i;   // pairs of the panel already stored
    const double fx = __builtin_bit_cast(double, (uint64_t)(1023 + TRD_XS) << 52);
    const double fxi = __builtin_bit_cast(double, (uint64_t)(1023 - TRD_XS) << 52);
    const double *xj = (j & 1) ? V.x1 : V.x0;
    // item b <= rt of a row's tile sums is rowp[b][r], item b > rt colp[b - 1][r]
    auto tile_sum = [&](int b, int rt, int row) -> double {
        const double *p = b <= rt ? P.rowp : P.colp - n;
        return p[(int64_t)b * n + row];
    };
    // ---- this row ----
    d2 pr[TRD_NB / 4];
#pragma unroll
    for (int u = 0; u < TRD_NB / 4; ++u) {
        pr[u] = (d2){0.0, 0.0};
        if (!TILED || 4 * u < np) pr[u] = *reinterpret_cast<const d2 *>(P.PVt + (int64_t)rr * TRD_PT + 2 * (qd + 4 * u));
    }
    const double a1 = rowc ? A[(int64_t)c * lda + rr] : A[(int64_t)rr * lda + c];
    double x = a1, vr = 0.0, wr = 0.0;
    if (fin) {
        // ---- the reflector, alike in every workgroup ----
        const double alpha = xj[c], a1c = A[(int64_t)c * lda + c], xr = xj[rr];
        double yr = TILED || c + 1 >= n ? 0.0 : V.y[rr], yj = TILED || c + 1 >= n ? 0.0 : V.y[c];
        const double pvr = t < 2 * TRD_NB ? P.PVt[(int64_t)c * TRD_PT + t] : 0.0;
        double s1 = 0.0, s2 = 0.0;
        const int g1 = (n - j + TRD_CR - 1) / TRD_CR, rt = (rr - trd_base(c)) / TRD_TT;
        constexpr int B1 = TILED ? 16 : 8;   // 64 (32) workgroups a batch
        if (!TILED || (t & 127) < 2 * np + 1) {   // what lies past them is not used
            const double *pin = P.part1 + (j & 1) * P.part1_len + min(t & 127, TRD_PS - 1);
            for (int b = t >> 7; b < g1; b += 4 * B1) {
                double u[B1];
#pragma unroll
                for (int k = 0; k < B1; ++k) u[k] = pin[(int64_t)min(b + 4 * k, g1 - 1) * TRD_PS];
#pragma unroll
                for (int k = 0; k < B1; ++k) s1 += b + 4 * k < g1 ? u[k] : 0.0;
            }
        }
        for (int b = t; b < g2; b += 4 * TRD_CT) {
            double u[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) u[k] = P.part2[min(b + k * TRD_CT, g2 - 1)];
#pragma unroll
            for (int k = 0; k < 4; ++k) s2 += b + k * TRD_CT < g2 ? u[k] : 0.0;
        }
        if (TILED) {
            for (int b0 = qd; b0 <= T; b0 += 64) {
                double u[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) u[k] = b0 + 4 * k <= T ? tile_sum(b0 + 4 * k, rt, rr) : 0.0;
#pragma unroll
                for (int k = 0; k < 16; ++k) yr += u[k];
            }
            if (wv == TRD_CW - 1) {   // the wave that adds row c's tile sums
                for (int b = lane; b <= T; b += 64) yj += tile_sum(b, 0, c);
                yj = wave_sum(yj);
                if (lane == 0) sc = yj;
            }
        }
        p1[t >> 7][t & 127] = s1;
        s2 = wave_sum(s2);
        if (lane == 0) r2[wv] = s2;
        if (t < 2 * TRD_NB) pv1[t] = t < 2 * np ? pvr : 0.0;
        __syncthreads();
        if (TILED) yj = sc;
        auto sum1 = [&](int q) { return (p1[0][q] + p1[1][q]) + (p1[2][q] + p1[3][q]); };
        const double sig = sum1(0);
        double xax = 0.0;
#pragma unroll
        for (int k = 0; k < TRD_CW; ++k) xax += r2[k];
        // (the root and the two quotients to about one ulp: short chains)
        double tau = 0.0, beta = alpha, scale = 0.0;
        if (sig >= TRD_SIG_MIN) {
            const double h = fma(alpha, alpha, sig);
            beta = -copysign(h * rr_rsqrt(h), alpha);
            tau = fma(-alpha, rr_recip(beta), 1.0);   // (beta - alpha) / beta
            scale = rr_recip(alpha - beta);
        }
        if (t < 2 * TRD_NB) zs[t] = t < 2 * np ? pvr + scale * sum1(t + 1) : 0.0;
        if (blockIdx.x == 0 && t == 0) {
            V.e[j] = beta * fxi;
            V.tau[j] = tau;
        }
        __syncthreads();
        // sum_k z_v z_w and the correction of p at row c, in every wave alike (lane = pair k)
        const int kl = lane & (TRD_NB - 1);
        const double zv = lane < TRD_NB ? zs[2 * kl] : 0.0, zw = zs[2 * kl + 1];
        const double zz = wave_sum(zv * zw);
        const double cj = wave_sum(lane < TRD_NB ? pv1[2 * kl] * zw + pv1[2 * kl + 1] * zv : 0.0);
        const double vav = a1c + scale * (2.0 * yj + scale * xax);
        const double al = -0.5 * tau * (tau * (vav - 2.0 * zz));   // -(tau / 2) (p . v)
        const double wc = tau * (a1c + scale * yj - cj) + al;      // w_j at row c, where v_j = 1
        double cr = 0.0, cx = 0.0;
#pragma unroll
        for (int u = 0; u < TRD_NB / 4; ++u) {
            const int k = qd + 4 * u;
            if (k >= np) pr[u] = (d2){0.0, 0.0};
            cr += pr[u].x * zs[2 * k + 1] + pr[u].y * zs[2 * k];
            cx += pr[u].x * pv1[2 * k + 1] + pr[u].y * pv1[2 * k];
        }
        cr = quad_sum(cr);
        cx = quad_sum(cx);
        if (TILED) yr = quad_sum(yr);
        vr = r == c ? 1.0 : scale * xr;
        wr = tau * (a1 + scale * yr - cr) + al * vr;
        x = a1 - cx - (vr * wc + wr);
        if (in) {
            // PV rows v, w; PW rows w, v: lane qd of the row writes one each
            double *o = ((qd & 2) ? P.PW : P.PV) + (int64_t)(2 * np + (qd & 1)) * P.ldp;
            o[r] = qd == 0 || qd == 3 ? vr : wr;
            if (qd == 0) *reinterpret_cast<d2 *>(P.PVt + (int64_t)r * TRD_PT + 2 * np) = (d2){vr, wr};
            if (qd == 1) A[(int64_t)r * lda + j] = vr;   // kept for the back-transformation
        }
        if (qd == 0) *reinterpret_cast<d2 *>(&S[rl * TRD_LS + 2 * np]) = (d2){vr, wr};
    }
    if (!col) return;
    if (in && qd == 0) {
        ((c & 1) ? V.x1 : V.x0)[r] = x * fx;
        if (r == c) V.d[c] = x;
    }
    if (c >= n - 1) return;   // the last column has no reflector (one workgroup)
    // ---- partial sums over this workgroup's rows >= c + 2 ----
    const double xb = in && r >= c + 2 ? x * fx : 0.0;
#pragma unroll
    for (int u = 0; u < TRD_NB / 4; ++u)
        if (qd + 4 * u < np) *reinterpret_cast<d2 *>(&S[rl * TRD_LS + 2 * (qd + 4 * u)]) = pr[u];
    if (qd == 0) xs[rl] = xb;
    const double sg = wave_sum(qd == 0 ? xb * xb : 0.0);
    __syncthreads();
    double y = 0.0;   // PV[lane] . x over the 16 rows of this wave's share
    if (lane < 2 * i)
#pragma unroll 8
        for (int k = 16 * wv; k < 16 * wv + 16; ++k) y += S[k * TRD_LS + lane] * xs[k];
    red[wv][1 + lane] = y;
    if (lane == 0) red[wv][0] = sg;
    __syncthreads();
    if (t < 2 * i + 1) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < TRD_CW; ++k) s += red[k][t];
        P.part1[(c & 1) * P.part1_len + (int64_t)blockIdx.x * TRD_PS + t] = s;
    }
}

// y[r] = A_0[r][j + 2:] . x for the rows r >= j + 1, one wave per row, lanes
// over the columns, fixed-order reduction; this workgroup's partial sum of
// x . y over its rows >= j + 2 into part2
__global__ __launch_bounds__(256) void k_trd_pass(const double *__restrict__ A, int64_t lda, int n, int j, TrdVec V,
                                                  TrdPanel P)
{
    __shared__ double red[4];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int r = j + 1 + (int)blockIdx.x * 4 + wv;
    const double *x = (j & 1) ? V.x1 : V.x0;
    double s = 0.0, xr = 0.0;
    if (r < n) {
        // whole lines: columns from the 16-aligned one at or before j + 2 on,
        // two per lane (the rows are padded to 32 columns)
        typedef double d2 __attribute__((ext_vector_type(2)));
        const double *row = A + (int64_t)r * lda;
        if (r >= j + 2) xr = x[r];
        for (int c0 = ((j + 2) & ~15) + 2 * lane; c0 < n; c0 += 8 * 128) {
            d2 a[8], b[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int c = c0 + 128 * u;
                a[u] = b[u] = (d2){0.0, 0.0};
                if (c < n) {
                    a[u] = *reinterpret_cast<const d2 *>(row + c);
                    b[u] = *reinterpret_cast<const d2 *>(x + c);
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int c = c0 + 128 * u;
                s += c >= j + 2 && c < n ? a[u].x * b[u].x : 0.0;
                s += c + 1 >= j + 2 && c + 1 < n ? a[u].y * b[u].y : 0.0;
            }
        }
        s = wave_sum(s);
        if (lane == 0) V.y[r] = s;
    }
    if (lane == 0) red[wv] = xr * s;
    __syncthreads();
    if (t == 0) P.part2[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// the product of the trailing block (j, n) with x (its entry j + 1 taken as 0)
// from its lower triangle only, for trailing blocks of at least TRD_TILE_MIN
// rows: one workgroup per TRD_TT x TRD_TT tile (rt, ct), ct <= rt, tile rows and
// columns counted from row trd_base(j + 1), the last multiple of 16 before the
// block (so that every row of a tile is eight whole cache lines; what it holds
// before column j + 1 meets zeros of x). A tile stores the row sums of its rows
// (columns up to the diagonal) into rowp[ct], the column sums of its columns
// (rows below the diagonal) into colp[rt], and its share of x . A_0 x into
// part2; the column kernel adds them in a fixed order. Bound by memory: 22 us on
// average from 8000 to 3072 trailing rows (6.0 TB/s, what a plain read of that
// size reaches), 27.6 us with 8-byte loads of rows that began anywhere in a
// line. One group of loads in flight a wave: a second one spills at four waves a
// SIMD.
struct TrdTileShared {
    double vr[TRD_TT], vc[TRD_TT], rsum[TRD_TT];
    double cs[4][TRD_TT];
    double red[2];
};

template <bool DIAG>
__device__ __forceinline__ void trd_tile(const double *__restrict__ A, int64_t lda, int n, int R0, int C0, double ve,
                                         TrdTileShared &sh)
{
    typedef double d2 __attribute__((ext_vector_type(2)));
    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);   // scalar: row addresses stay in scalar registers
    // wave wv: tile rows 32 wv .. 32 wv + 31 in four groups of 8, two columns a
    // lane; row sums per lane, then over the lanes. The first group goes out
    // before x is in LDS, the next one as soon as a group is multiplied. Rows
    // past n are read from the last row and pairs past column n from the last
    // pair or the zero pad (the rows are padded to 32 columns): they meet zeros
    // of x.
    d2 a[8];
    const int pc = min(C0 + 2 * lane, (n - 1) & ~1) >> 1;
    auto load = [&](int g) {
        const int rg = R0 + 32 * wv + 8 * g;
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = reinterpret_cast<const d2 *>(A + (int64_t)min(rg + u, n - 1) * lda)[pc];
    };
    load(0);
    if (t < TRD_TT) sh.vr[t] = ve;
    else sh.vc[t - TRD_TT] = ve;
    __syncthreads();
    const d2 vcl = (d2){sh.vc[2 * lane], sh.vc[2 * lane + 1]};
    d2 colacc = (d2){0.0, 0.0};
#pragma unroll 1
    for (int g = 0; g < 4; ++g) {
        const int rl0 = 32 * wv + 8 * g;
        double racc[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            d2 v = a[u];
            if (DIAG) {
                if (2 * lane > rl0 + u) v.x = 0.0;
                if (2 * lane + 1 > rl0 + u) v.y = 0.0;
            }
            racc[u] = v.x * vcl.x + v.y * vcl.y;   // row part: c <= r
            if (DIAG) {
                if (2 * lane == rl0 + u) v.x = 0.0;
                if (2 * lane + 1 == rl0 + u) v.y = 0.0;
            }
            const double w = sh.vr[rl0 + u];
            colacc.x += v.x * w;                   // column part: r > c
            colacc.y += v.y * w;
        }
        if (g < 3) load(g + 1);
        // the 8 row sums over the 64 lanes (halving exchanges in a fixed pattern)
        const bool b5 = lane & 32, b4 = lane & 16;
        double h4[4], h2[2];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            h4[k] = (b5 ? racc[4 + k] : racc[k]) + __shfl_xor(b5 ? racc[k] : racc[4 + k], 32, 64);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            h2[k] = (b4 ? h4[2 + k] : h4[k]) + __shfl_xor(b4 ? h4[k] : h4[2 + k], 16, 64);
            // over the 16 lanes of a row
            h2[k] += rr_dpp<0x128, 0xf, 0xf>(h2[k]);   // row_ror 8, 4, 2, 1
            h2[k] += rr_dpp<0x124, 0xf, 0xf>(h2[k]);
            h2[k] += rr_dpp<0x122, 0xf, 0xf>(h2[k]);
            h2[k] += rr_dpp<0x121, 0xf, 0xf>(h2[k]);
        }
        if ((lane & 15) < 2) sh.rsum[rl0 + 4 * b5 + 2 * b4 + (lane & 1)] = (lane & 1) ? h2[1] : h2[0];
    }
    sh.cs[wv][2 * lane] = colacc.x;
    sh.cs[wv][2 * lane + 1] = colacc.y;
    __syncthreads();
}

__global__ __launch_bounds__(256, 4) void k_trd_tiles(const double *__restrict__ A, int64_t lda, int n, int j, TrdVec V,
                                                      TrdPanel P)
{
    __shared__ TrdTileShared sh;
    const int t = threadIdx.x, b = blockIdx.x;
    int rt = (int)((sqrt(8.0 * b + 1.0) - 1.0) * 0.5);
    while ((rt + 1) * (rt + 2) / 2 <= b) ++rt;
    while (rt * (rt + 1) / 2 > b) --rt;
    const int ct = b - rt * (rt + 1) / 2;
    const int B0 = trd_base(j + 1), R0 = B0 + TRD_TT * rt, C0 = B0 + TRD_TT * ct;
    const double *x = (j & 1) ? V.x1 : V.x0;
    const int e = t < TRD_TT ? R0 + t : C0 + t - TRD_TT;   // this thread's row (t < TT) or column of x
    const double ve = e < n && e > j + 1 ? x[e] : 0.0;
    if (rt == ct) trd_tile<true>(A, lda, n, R0, C0, ve, sh);
    else trd_tile<false>(A, lda, n, R0, C0, ve, sh);
    if (t < TRD_TT) {
        const int r = R0 + t, c = C0 + t;
        const double rs = sh.rsum[t], cl = sh.cs[0][t] + sh.cs[1][t] + sh.cs[2][t] + sh.cs[3][t];
        if (r < n) P.rowp[(int64_t)ct * n + r] = rs;
        if (c < n) P.colp[(int64_t)rt * n + c] = cl;
        const double s = wave_sum(sh.vr[t] * rs + sh.vc[t] * cl);   // (past n: 0)
        if ((t & 63) == 0) sh.red[t >> 6] = s;
    }
    __syncthreads();
    if (t == 0) P.part2[b] = sh.red[0] + sh.red[1];
}

// columns j0 .. j0 + nbp - 1 of the reduction, then the update of the
// trailing block [j0 + nbp, n)^2
hipError_t launch_trd_panel(double *A, int64_t lda, int n, int j0, int nbp, const TrdVec &V, const TrdPanel &P,
                            hipStream_t st)
{
    // the column kernel of column c, after i reflectors of the panel
    auto column = [&](int c, int i, int fin, int col) {
        const int m = n - c;   // rows from c on = rows of the product of column c - 1
        const int T = trd_tiles(n - trd_base(c)), tiled = m >= TRD_TILE_MIN;
        const int g2 = m < 2 ? 0 : (tiled ? T * (T + 1) / 2 : (m + 3) / 4);
        // the last TRD_TILE_MIN rows are updated as a whole square
        const dim3 g((m + TRD_CR - 1) / TRD_CR), b(TRD_CT);
        const int rowc = m <= TRD_TILE_MIN;
        if (tiled) hipLaunchKernelGGL(k_trd_col<true>, g, b, 0, st, A, lda, n, c, i, fin, col, T, rowc, g2, V, P);
        else hipLaunchKernelGGL(k_trd_col<false>, g, b, 0, st, A, lda, n, c, i, fin, col, 0, rowc, g2, V, P);
    };
    for (int i = 0; i < nbp; ++i) {
        const int j = j0 + i, m = n - j - 1;
        column(j, i, i > 0, 1);
        if (m < 2) continue;   // no column right of j + 1: nothing to multiply
        if (m >= TRD_TILE_MIN) {
            const int T = trd_tiles(n - trd_base(j + 1));
            hipLaunchKernelGGL(k_trd_tiles, dim3(T * (T + 1) / 2), dim3(256), 0, st, A, lda, n, j, V, P);
        } else {
            hipLaunchKernelGGL(k_trd_pass, dim3((m + 3) / 4), dim3(256), 0, st, A, lda, n, j, V, P);
        }
    }
    const int t = j0 + nbp;
    if (t < n) {
        // v and w of the panel's last reflector, then A -= PV^T PW on the trailing block
        column(t, nbp, 1, 0);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        // while the trailing block has TRD_TILE_MIN rows or more it is read
        // only below the diagonal (tiled product, column kernel, reflectors);
        // the row pass reads whole rows of the last TRD_TILE_MIN, so the
        // square from a tile row at or before n - TRD_TILE_MIN is updated whole
        const int lowq = n - TRD_TILE_MIN - t > 0 ? (n - TRD_TILE_MIN - t) / EG_T : 0;
        return launch_eig_gemm(n - t, n - t, 2 * nbp, -1.0, P.PV + t, 1, P.ldp, P.PW + t, P.ldp, 1, 1.0,
                               A + (int64_t)t * lda + t, lda, st, nullptr, 0, lowq);
    }
    return hipGetLastError();
}

// W = (W + W^T) / 2 in place (the operation is defined on a symmetric matrix), then
// scaled by the power of two of trd_shift;
// the rows' pad columns n .. ld - 1 become 0; amax: the largest |entry| as bits
// (zeroed by k_word_zero). A workgroup takes the 32 x 32 tiles (rt, ct) and
// (ct, rt), ct <= rt, through LDS, so that both are read and written by rows:
// bound by memory (one pass over W each way), 0.19 ms at n = 8000 (5.3 TB/s)
// against 0.84 with the upper triangle read and written by columns.
constexpr int SYM_T = 32;
__global__ __launch_bounds__(256) void k_symmetrize(double *__restrict__ W, int64_t ld, int n,
                                                    unsigned long long *__restrict__ amax)
{
    __shared__ double L[SYM_T][SYM_T + 1], U[SYM_T][SYM_T + 1];
    const int t = threadIdx.x, cl = t & 31, r0 = t >> 5;
    const int R0 = (int)blockIdx.y * SYM_T, C0 = (int)blockIdx.x * SYM_T;
    if (C0 > R0) return;
    if (C0 == 0 && n + cl < ld)
        for (int r = r0; r < SYM_T && R0 + r < n; r += 8) W[(int64_t)(R0 + r) * ld + n + cl] = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int r = r0 + 8 * u;
        L[r][cl] = R0 + r < n && C0 + cl < n ? W[(int64_t)(R0 + r) * ld + C0 + cl] : 0.0;
        U[r][cl] = C0 + r < n && R0 + cl < n ? W[(int64_t)(C0 + r) * ld + R0 + cl] : 0.0;
    }
    __syncthreads();
    unsigned long long m = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int r = r0 + 8 * u;
        const double lo = R0 + r == C0 + cl ? L[r][cl] : 0.5 * (L[r][cl] + U[cl][r]);
        const double up = C0 + r == R0 + cl ? U[r][cl] : 0.5 * (L[cl][r] + U[r][cl]);
        m = max(m, __builtin_bit_cast(unsigned long long, fabs(lo)));
        if (R0 + r < n && C0 + cl < n) W[(int64_t)(R0 + r) * ld + C0 + cl] = lo;
        if (C0 < R0 && C0 + r < n && R0 + cl < n) W[(int64_t)(C0 + r) * ld + R0 + cl] = up;
    }
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o));
    // (few waves find a larger entry than those before them)
    if ((t & 63) == 0 && m > __hip_atomic_load(amax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(amax, m);
}

// W times 2^-trd_shift(amax): nothing to do, and nothing read, for entries of an
// ordinary size
__global__ __launch_bounds__(256) void k_scale_pow2(double *__restrict__ W, int64_t len,
                                                    const unsigned long long *__restrict__ amax)
{
    const int sh = trd_shift(*amax);
    if (sh == 0) return;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < len; i += (int64_t)gridDim.x * 256)
        W[i] = ldexp(W[i], -sh);
}

__global__ void k_word_zero(unsigned long long *__restrict__ w) { *w = 0; }

hipError_t launch_symmetrize(double *W, int64_t ld, int n, unsigned long long *amax, hipStream_t st)
{
    if (n < 1) return hipSuccess;
    const unsigned T = (unsigned)((n + SYM_T - 1) / SYM_T);
    hipLaunchKernelGGL(k_word_zero, dim3(1), dim3(1), 0, st, amax);
    hipLaunchKernelGGL(k_symmetrize, dim3(T, T), dim3(256), 0, st, W, ld, n, amax);
    const int64_t len = (int64_t)n * ld;
    hipLaunchKernelGGL(k_scale_pow2, dim3((unsigned)std::min<int64_t>((len + 255) / 256, 2048)), dim3(256), 0, st, W, len,
                       amax);
    return hipGetLastError();
}


// ---------------------------------------------------------------------------
// 2. eigenvalues of the tridiagonal T (diagonal d[0..n), off-diagonal e[0..n-1))
// ---------------------------------------------------------------------------
// number of eigenvalues below x of the unreduced block d[0..m), e2[0..m-1)
// (Sturm sequence of the LDL^T pivots; the chain's quotient e2 / q as e2 times
// the refined hardware reciprocal, about one ulp off, which is a relative
// change of e2 by as much: at |q| >= pivmin neither it nor the product
// overflows)
__device__ __forceinline__ int sturm_count(const double *__restrict__ d, const double *__restrict__ e2, int m,
                                           double x, double pivmin)
{
    int c = 0;
    double q = d[0] - x;
    if (fabs(q) < pivmin) q = -pivmin;
    c += q < 0.0;
    int i = 1;
    for (; i + 8 <= m; i += 8) {   // the loads of 8 steps go out before the chain
        double dv[8], ev[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            dv[u] = d[i + u];
            ev[u] = e2[i + u - 1];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            q = dv[u] - x - ev[u] * rr_recip(q);
            if (fabs(q) < pivmin) q = -pivmin;
            c += q < 0.0;
        }
    }
    for (; i < m; ++i) {
        q = d[i] - x - e2[i - 1] * rr_recip(q);
        if (fabs(q) < pivmin) q = -pivmin;
        c += q < 0.0;
    }
    return c;
}

// eigenvalue t: the k-th (ascending) of the block starting at row b0 with m
// rows, by multisection on [lo, hi]: the TRI_G lanes of a group evaluate the
// Sturm count at TRI_G interior points, and the interval shrinks to the piece
// between the last point with count <= k and the first with count > k, until
// no representable point lies strictly inside. With monotone counts this ends
// on the same pair of adjacent doubles as bisection, in about a third of the
// dependent steps. Bound by the chain of dependent quotients, so a small n, which
// leaves the chip empty, takes more points a step: with 64 lanes 0.18 ms at
// n = 301 (8 lanes and the division: 0.42), with 8 lanes 9.4 ms at n = 8000
// (12.6 with the division); 16 lanes are the better ones between 1024 and 3072,
// where the chip is filled by them
template <int TRI_G>
__global__ __launch_bounds__(256) void k_tri_bisect(const double *__restrict__ d, const double *__restrict__ e2, int n,
                                                    const int32_t *__restrict__ bs, const int32_t *__restrict__ bm,
                                                    const int32_t *__restrict__ bk, double lo0, double hi0,
                                                    double pivmin, double *__restrict__ w)
{
    const int gt = blockIdx.x * blockDim.x + threadIdx.x;
    const int t = gt / TRI_G, g = gt % TRI_G;
    if (t >= n) return;   // (whole groups)
    const int b0 = bs[t], m = bm[t], k = bk[t];
    const double f = (double)(g + 1) / (double)(TRI_G + 1);
    double lo = lo0, hi = hi0;
    for (int it = 0; it < 200; ++it) {
        const double x = lo + (hi - lo) * f;
        const bool in = x > lo && x < hi;
        int any = in;
        for (int o = 1; o < TRI_G; o <<= 1) any |= __shfl_xor(any, o, TRI_G);
        if (!any) break;   // lo and hi are adjacent doubles
        const int cnt = in ? sturm_count(d + b0, e2 + b0, m, x, pivmin) : 0;
        double h = in && cnt > k ? x : hi;
        for (int o = 1; o < TRI_G; o <<= 1) h = fmin(h, __shfl_xor(h, o, TRI_G));
        double l = in && cnt <= k && x < h ? x : lo;
        for (int o = 1; o < TRI_G; o <<= 1) l = fmax(l, __shfl_xor(l, o, TRI_G));
        lo = l;
        hi = h;
    }
    if (g == 0) w[t] = 0.5 * (lo + hi);
}

__global__ void k_tri_prep(const double *__restrict__ e, int n, double *__restrict__ e2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n - 1) e2[i] = e[i] * e[i];
}

// bs/bm/bk[t]: block start, block rows and index inside the block of
// eigenvalue t (e must hold exact zeros between blocks)
hipError_t launch_tri_eigenvalues(const double *d, const double *e, double *e2, int n, const int32_t *bs,
                                  const int32_t *bm, const int32_t *bk, double lo, double hi, double pivmin,
                                  double *w, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    if (n > 1) hipLaunchKernelGGL(k_tri_prep, dim3((n + 255) / 256), dim3(256), 0, st, e, n, e2);
    // lanes per eigenvalue: as many as the chip has room for
    const int G = n <= 1024 ? 64 : (n <= 3072 ? 16 : 8);
    const dim3 g((unsigned)(((int64_t)n * G + 255) / 256)), b(256);
    if (G == 64) hipLaunchKernelGGL(k_tri_bisect<64>, g, b, 0, st, d, e2, n, bs, bm, bk, lo, hi, pivmin, w);
    else if (G == 16) hipLaunchKernelGGL(k_tri_bisect<16>, g, b, 0, st, d, e2, n, bs, bm, bk, lo, hi, pivmin, w);
    else hipLaunchKernelGGL(k_tri_bisect<8>, g, b, 0, st, d, e2, n, bs, bm, bk, lo, hi, pivmin, w);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 3. eigenvector k of T by the twisted factorisation of its block minus w_k:
//    forward L D L^T (pivots dp, multipliers l), backward U D U^T (pivots dm,
//    multipliers u), twist index r = argmin |dp_i + dm_i - (d_i - w)|, then
//    z_r = 1, z_i = -l_i z_{i+1} above r and z_{i+1} = -u_i z_i below, and
//    normalisation; rows outside the block are zero. Z[i][k] (column k):
//    consecutive threads write consecutive addresses. S is scratch of the
//    same shape (the multipliers).
// ---------------------------------------------------------------------------
__global__ void k_tri_vectors(const double *__restrict__ dg, const double *__restrict__ eg, int n,
                              const int32_t *__restrict__ bs, const int32_t *__restrict__ bm,
                              const double *__restrict__ w, double pivmin, double *__restrict__ Zg, int64_t ldz,
                              double *__restrict__ Sg, int64_t lds)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int b0 = bs[k], m = bm[k];
    const double lam = w[k];
    for (int i = 0; i < b0; ++i) Zg[(int64_t)i * ldz + k] = 0.0;
    for (int i = b0 + m; i < n; ++i) Zg[(int64_t)i * ldz + k] = 0.0;
    const double *d = dg + b0, *e = eg + b0;
    double *Z = Zg + (int64_t)b0 * ldz, *S = Sg + (int64_t)b0 * lds;
    if (m == 1) {
        Z[k] = 1.0;
        return;
    }
    // Every loop below is a dependent chain over the rows; the loads of
    // TV_B steps go out before the chain runs through them, and the quotients
    // are products with the refined hardware reciprocal (about one ulp).
    constexpr int TV_B = 8;
    // forward: dp_i into S, l_i into Z (both column k)
    double dp = d[0] - lam;
    if (fabs(dp) < pivmin) dp = -pivmin;
    S[k] = dp;
    int i = 0;
    for (; i + TV_B <= m - 1; i += TV_B) {
        double dv[TV_B], ev[TV_B];
#pragma unroll
        for (int u = 0; u < TV_B; ++u) {
            dv[u] = d[i + u + 1];
            ev[u] = e[i + u];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < TV_B; ++u) {
            const double l = ev[u] * rr_recip(dp);
            Z[(int64_t)(i + u) * ldz + k] = l;
            dp = dv[u] - lam - l * ev[u];
            if (fabs(dp) < pivmin) dp = -pivmin;
            S[(int64_t)(i + u + 1) * lds + k] = dp;
        }
    }
    for (; i < m - 1; ++i) {
        const double l = e[i] * rr_recip(dp);
        Z[(int64_t)i * ldz + k] = l;
        dp = d[i + 1] - lam - l * e[i];
        if (fabs(dp) < pivmin) dp = -pivmin;
        S[(int64_t)(i + 1) * lds + k] = dp;
    }
    // backward: dm_i, twist index
    double dm = d[m - 1] - lam;
    if (fabs(dm) < pivmin) dm = -pivmin;
    int r = m - 1;
    double best = fabs(S[(int64_t)(m - 1) * lds + k] + dm - (d[m - 1] - lam));
    i = m - 2;
    for (; i - (TV_B - 1) >= 0; i -= TV_B) {
        double dv[TV_B], ev[TV_B], sv[TV_B];
#pragma unroll
        for (int u = 0; u < TV_B; ++u) {
            dv[u] = d[i - u];
            ev[u] = e[i - u];
            sv[u] = S[(int64_t)(i - u) * lds + k];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < TV_B; ++u) {
            const double uu = ev[u] * rr_recip(dm);
            dm = dv[u] - lam - uu * ev[u];
            if (fabs(dm) < pivmin) dm = -pivmin;
            const double g = fabs(sv[u] + dm - (dv[u] - lam));
            if (g < best) {
                best = g;
                r = i - u;
            }
        }
    }
    for (; i >= 0; --i) {
        const double u = e[i] * rr_recip(dm);
        dm = d[i] - lam - u * e[i];
        if (fabs(dm) < pivmin) dm = -pivmin;
        const double g = fabs(S[(int64_t)i * lds + k] + dm - (d[i] - lam));
        if (g < best) {
            best = g;
            r = i;
        }
    }
    // u_i for i >= r again (backward from the end), into S rows i >= r
    dm = d[m - 1] - lam;
    if (fabs(dm) < pivmin) dm = -pivmin;
    i = m - 2;
    for (; i - (TV_B - 1) >= r; i -= TV_B) {
        double dv[TV_B], ev[TV_B];
#pragma unroll
        for (int u = 0; u < TV_B; ++u) {
            dv[u] = d[i - u];
            ev[u] = e[i - u];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < TV_B; ++u) {
            const double uu = ev[u] * rr_recip(dm);
            S[(int64_t)(i - u) * lds + k] = uu;
            dm = dv[u] - lam - uu * ev[u];
            if (fabs(dm) < pivmin) dm = -pivmin;
        }
    }
    for (; i >= r; --i) {
        const double u = e[i] * rr_recip(dm);
        S[(int64_t)i * lds + k] = u;
        dm = d[i] - lam - u * e[i];
        if (fabs(dm) < pivmin) dm = -pivmin;
    }
    // the vector (z_r = 1), its norm
    double nrm = 1.0, z = 1.0;
    i = r - 1;
    for (; i - (TV_B - 1) >= 0; i -= TV_B) {
        double lv[TV_B];
#pragma unroll
        for (int u = 0; u < TV_B; ++u) lv[u] = Z[(int64_t)(i - u) * ldz + k];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < TV_B; ++u) {
            z = -lv[u] * z;
            Z[(int64_t)(i - u) * ldz + k] = z;
            nrm += z * z;
        }
    }
    for (; i >= 0; --i) {
        z = -Z[(int64_t)i * ldz + k] * z;
        Z[(int64_t)i * ldz + k] = z;
        nrm += z * z;
    }
    Z[(int64_t)r * ldz + k] = 1.0;
    z = 1.0;
    i = r;
    for (; i + TV_B <= m - 1; i += TV_B) {
        double uv[TV_B];
#pragma unroll
        for (int u = 0; u < TV_B; ++u) uv[u] = S[(int64_t)(i + u) * lds + k];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < TV_B; ++u) {
            z = -uv[u] * z;
            Z[(int64_t)(i + u + 1) * ldz + k] = z;
            nrm += z * z;
        }
    }
    for (; i < m - 1; ++i) {
        z = -S[(int64_t)i * lds + k] * z;
        Z[(int64_t)(i + 1) * ldz + k] = z;
        nrm += z * z;
    }
    const double inv = 1.0 / sqrt(nrm);
    i = 0;
    for (; i + TV_B <= m; i += TV_B) {
        double zv[TV_B];
#pragma unroll
        for (int u = 0; u < TV_B; ++u) zv[u] = Z[(int64_t)(i + u) * ldz + k];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < TV_B; ++u) Z[(int64_t)(i + u) * ldz + k] = zv[u] * inv;
    }
    for (; i < m; ++i) Z[(int64_t)i * ldz + k] *= inv;
}

hipError_t launch_tri_vectors(const double *d, const double *e, int n, const int32_t *bs, const int32_t *bm,
                              const double *w, double pivmin, double *Z, int64_t ldz, double *S, int64_t lds,
                              hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tri_vectors, dim3((n + 63) / 64), dim3(64), 0, st, d, e, n, bs, bm, w, pivmin, Z, ldz, S,
                       lds);
    return hipGetLastError();
}

// modified Gram-Schmidt over the columns cols[0..nc) of Z (one cluster of
// close eigenvalues inside the unreduced block of rows [b0, b0 + m)), in
// order, each column projected twice. A column that keeps less than half of
// its norm after the projection has collapsed towards the ones before it
// (twisted vectors of nearly equal eigenvalues can come out nearly
// parallel): it is refined by two steps of inverse iteration with its own
// eigenvalue, each followed by the projection, from what is left of it, or
// from a fixed spread vector when almost nothing is left. The solve is
// (T_b - lambda I) y = x by the LDL^T recurrence with pivots floored at
// piv (one thread; rare path), the product kept in Z, the pivots in column c
// of S.
__device__ __forceinline__ double mgs_project(double *Z, int64_t ldz, int b0, int m, const int32_t *cols, int a,
                                              int c, double *red)
{
    const int t = threadIdx.x;
    for (int pass = 0; pass < 2; ++pass)
        for (int q = 0; q < a; ++q) {
            const int cq = cols[q];
            double s = 0.0;
            for (int i = b0 + t; i < b0 + m; i += 256) s += Z[(int64_t)i * ldz + cq] * Z[(int64_t)i * ldz + c];
            const double dot = blk_sum(s, red);
            for (int i = b0 + t; i < b0 + m; i += 256) Z[(int64_t)i * ldz + c] -= dot * Z[(int64_t)i * ldz + cq];
            __syncthreads();
        }
    double s = 0.0;
    for (int i = b0 + t; i < b0 + m; i += 256) s += Z[(int64_t)i * ldz + c] * Z[(int64_t)i * ldz + c];
    return blk_sum(s, red);
}

__device__ __forceinline__ void mgs_scale(double *Z, int64_t ldz, int b0, int m, int c, double nrm2)
{
    const double inv = nrm2 > 0.0 ? 1.0 / sqrt(nrm2) : 0.0;
    for (int i = b0 + threadIdx.x; i < b0 + m; i += 256) Z[(int64_t)i * ldz + c] *= inv;
    __syncthreads();
}

// one workgroup per cluster; cluster b is desc[4b .. 4b + 3] = (offset of its
// columns in cols_all, number of columns, block start, block rows). The
// clusters have disjoint columns (of Z and of S) and run concurrently.
__global__ __launch_bounds__(256) void k_cluster_mgs(double *__restrict__ Z, int64_t ldz,
                                                     const int32_t *__restrict__ desc,
                                                     const int32_t *__restrict__ cols_all,
                                                     const double *__restrict__ dg, const double *__restrict__ eg,
                                                     const double *__restrict__ w, double *__restrict__ S,
                                                     int64_t lds, double piv)
{
    __shared__ double red[4];
    const int t = threadIdx.x;
    const int32_t *dsc = desc + 4 * (int64_t)blockIdx.x;
    const int32_t *cols = cols_all + dsc[0];
    const int nc = dsc[1], b0 = dsc[2], m = dsc[3];
    for (int a = 0; a < nc; ++a) {
        const int c = cols[a];
        double nrm2 = mgs_project(Z, ldz, b0, m, cols, a, c, red);
        if (a > 0 && nrm2 < 0.25) {
            if (nrm2 <= 1e-6) {
                for (int i = b0 + t; i < b0 + m; i += 256)
                    Z[(int64_t)i * ldz + c] = sin(1.0 + 0.7 * (double)(i - b0) + 1.3 * (double)a);
                __syncthreads();
                nrm2 = mgs_project(Z, ldz, b0, m, cols, a, c, red);
            }
            for (int it = 0; it < 2; ++it) {
                mgs_scale(Z, ldz, b0, m, c, nrm2);
                if (t == 0) {
                    const double lam = w[c];
                    const double *d = dg + b0, *e = eg + b0;
                    double *z = Z + (int64_t)b0 * ldz + c, *dp = S + (int64_t)b0 * lds + c;
                    // forward: L z' = z and the pivots
                    double p = d[0] - lam;
                    if (fabs(p) < piv) p = p < 0.0 ? -piv : piv;
                    dp[0] = p;
                    for (int i = 1; i < m; ++i) {
                        const double l = e[i - 1] / p;
                        z[(int64_t)i * ldz] -= l * z[(int64_t)(i - 1) * ldz];
                        p = d[i] - lam - l * e[i - 1];
                        if (fabs(p) < piv) p = p < 0.0 ? -piv : piv;
                        dp[(int64_t)i * lds] = p;
                    }
                    // backward: D L^T y = z'
                    double y = z[(int64_t)(m - 1) * ldz] / dp[(int64_t)(m - 1) * lds];
                    z[(int64_t)(m - 1) * ldz] = y;
                    for (int i = m - 2; i >= 0; --i) {
                        const double q = dp[(int64_t)i * lds];
                        y = z[(int64_t)i * ldz] / q - (e[i] / q) * y;
                        z[(int64_t)i * ldz] = y;
                    }
                }
                __syncthreads();
                nrm2 = mgs_project(Z, ldz, b0, m, cols, a, c, red);
            }
        }
        mgs_scale(Z, ldz, b0, m, c, nrm2);
    }
}

hipError_t launch_cluster_mgs(double *Z, int64_t ldz, const int32_t *desc, int ncl, const int32_t *cols,
                              const double *d, const double *e, const double *w, double *S, int64_t lds, double piv,
                              hipStream_t st)
{
    if (ncl <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_cluster_mgs, dim3(ncl), dim3(256), 0, st, Z, ldz, desc, cols, d, e, w, S, lds, piv);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 4. back-transformation helpers
// ---------------------------------------------------------------------------
// Vb[r][i] = v_{j0+i}[j0+1+r] (zero above the reflector's first row), rows
// r < m = n - j0 - 1, i < nb
__global__ void k_copy_reflectors(const double *__restrict__ A, int64_t lda, int n, int j0, int nb,
                                  double *__restrict__ Vb)
{
    // consecutive threads: consecutive reflectors of one row (both sides contiguous)
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int r = (int)(e / nb), i = (int)(e % nb);
    if (r >= n - j0 - 1) return;
    Vb[e] = r >= i ? A[(int64_t)(j0 + 1 + r) * lda + j0 + i] : 0.0;   // reflector j starts at row j + 1
}

hipError_t launch_copy_reflectors(const double *A, int64_t lda, int n, int j0, int nb, double *Vb, hipStream_t st)
{
    const int m = n - j0 - 1;
    if (m <= 0 || nb <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_copy_reflectors, dim3((unsigned)(((int64_t)m * nb + 255) / 256)), dim3(256), 0, st, A, lda, n,
                       j0, nb, Vb);
    return hipGetLastError();
}

// T (nb x nb, upper triangular) of the compact WY form from the Gram matrix
// G = Vb^T Vb and the scalars tau: T[i][i] = tau_i,
// T[0:i, i] = -tau_i T[0:i, 0:i] G[0:i, i]. One workgroup, all in LDS: the
// four diagonal blocks of 16 by that column recurrence side by side (one
// wave each; thread r forms entry r, its sum in order), then neighbouring
// blocks joined, 16 -> 32 -> 64, by T12 = -T11 G12 T22 (the same T: the
// product of the first reflectors times that of the next ones). The sums run
// over whole blocks (T is zero below its diagonal), unrolled, so that their LDS
// reads overlap. Workgroup h of two forms the diagonal block of reflectors
// [64 h, 64 h + 64) of nb_all and zeroes the block left of it.
constexpr int LARFT_MAX = 64;
__global__ __launch_bounds__(256) void k_larft(const double *__restrict__ G_all, int ldg,
                                               const double *__restrict__ tau_all, int nb_all,
                                               double *__restrict__ T_all, int ldt)
{
    const int off = LARFT_MAX * blockIdx.x, nb = min(LARFT_MAX, nb_all - off);
    const double *G = G_all + (int64_t)off * ldg + off, *tau = tau_all + off;
    double *T = T_all + (int64_t)off * ldt + off;
    for (int e = threadIdx.x; e < nb * off; e += 256) T_all[(int64_t)(off + e / off) * ldt + e % off] = 0.0;
    __shared__ double Ts[LARFT_MAX][LARFT_MAX + 1];
    __shared__ double Gs[LARFT_MAX][LARFT_MAX + 1];
    __shared__ double Ws[LARFT_MAX / 2][LARFT_MAX / 2 + 1];
    __shared__ double ts[LARFT_MAX];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
#pragma unroll 4
    for (int e = t; e < LARFT_MAX * LARFT_MAX; e += 256) {
        const int r = e / LARFT_MAX, c = e % LARFT_MAX;
        Ts[r][c] = 0.0;
        Gs[r][c] = r < nb && c < nb ? G[(int64_t)r * ldg + c] : 0.0;
    }
    if (t < nb) ts[t] = tau[t];
    __syncthreads();
    // the diagonal blocks [16 wv, 16 wv + 16)
    const int b0 = 16 * wv, bl = max(0, min(16, nb - b0));
    for (int i = 0; i < 16; ++i) {
        if (i < bl) {
            const int c = b0 + i;
            if (lane < i) {
                double acc = 0.0;
#pragma unroll
                for (int q = 0; q < 16; ++q) acc += Ts[b0 + lane][b0 + q] * Gs[b0 + q][c];   // (columns from i on: 0)
                Ts[b0 + lane][c] = -ts[c] * acc;
            } else if (lane == i) {
                Ts[c][c] = ts[c];
            }
        }
        __syncthreads();
    }
    // joins: rows [a0, a0 + h) (T11) with columns [c0, c0 + h2) (T22), c0 = a0 + h
    for (int h = 16; h < nb; h *= 2) {
        const int np = (nb + 2 * h - 1) / (2 * h);
        // W = G12 T22 (h x h2 per pair; T22 upper triangular)
        for (int p = 0; p < np; ++p) {
            const int a0 = 2 * h * p, c0 = a0 + h;
            if (c0 >= nb) break;
            const int h2 = min(h, nb - c0);
            for (int e = t; e < h * h2; e += 256) {
                const int r = e / h2, cc = e % h2;
                double acc = 0.0;
#pragma unroll 16
                for (int q = 0; q < h2; ++q) acc += Gs[a0 + r][c0 + q] * Ts[c0 + q][c0 + cc];
                Ws[r][cc] = acc;
            }
            __syncthreads();
            // T12 = -T11 W (T11 upper triangular)
            for (int e = t; e < h * h2; e += 256) {
                const int r = e / h2, cc = e % h2;
                double acc = 0.0;
#pragma unroll 16
                for (int q = 0; q < h; ++q) acc += Ts[a0 + r][a0 + q] * Ws[q][cc];
                Ts[a0 + r][c0 + cc] = -acc;
            }
            __syncthreads();
        }
    }
    for (int e = t; e < nb * nb; e += 256) T[(int64_t)(e / nb) * ldt + e % nb] = Ts[e / nb][e % nb];
}

// T (nb x nb, row-major) for nb <= 2 LARFT_MAX: up to LARFT_MAX in one
// workgroup; above, the two diagonal blocks of LARFT_MAX and n2 = nb -
// LARFT_MAX reflectors, joined by T12 = -T1 (G12 T2) (two FP64 MFMA
// products; X: LARFT_MAX x n2 doubles of scratch)
hipError_t launch_larft(const double *G, const double *tau, int nb, double *T, double *X, hipStream_t st)
{
    if (nb > 2 * LARFT_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_larft, dim3((nb + LARFT_MAX - 1) / LARFT_MAX), dim3(256), 0, st, G, nb, tau, nb, T, nb);
    hipError_t e = hipGetLastError();
    if (nb <= LARFT_MAX || e != hipSuccess) return e;
    const int h = LARFT_MAX, n2 = nb - h;
    // X = G12 T2, then T12 = -T1 X
    if ((e = launch_eig_gemm(h, n2, n2, 1.0, G + h, nb, 1, T + (int64_t)h * nb + h, nb, 1, 0.0, X, n2, st, nullptr,
                             0, -1)) != hipSuccess)
        return e;
    return launch_eig_gemm(h, n2, h, -1.0, T, nb, 1, X, n2, 1, 0.0, T + h, nb, st, nullptr, 0, -1);
}

// out[k][i] = Z[i][k]
__global__ __launch_bounds__(256) void k_transpose_sq(const double *__restrict__ Z, int64_t ldz, int n,
                                                      double *__restrict__ out, int64_t ldo)
{
    __shared__ double tl[32][33];
    const int i0 = blockIdx.y * 32, k0 = blockIdx.x * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int a = ty; a < 32; a += 8) {
        const int i = i0 + a, k = k0 + tx;
        tl[a][tx] = (i < n && k < n) ? Z[(int64_t)i * ldz + k] : 0.0;
    }
    __syncthreads();
    for (int a = ty; a < 32; a += 8) {
        const int k = k0 + a, i = i0 + tx;
        if (k < n && i < n) out[(int64_t)k * ldo + i] = tl[tx][a];
    }
}

hipError_t launch_transpose_sq(const double *Z, int64_t ldz, int n, double *out, int64_t ldo, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_transpose_sq, dim3((n + 31) / 32, (n + 31) / 32), dim3(256), 0, st, Z, ldz, n, out, ldo);
    return hipGetLastError();
}

}  // namespace cch
