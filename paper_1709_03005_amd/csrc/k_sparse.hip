// A mat-vec for L2-heavy matrices (Sec. 2.2: the off-diagonal pure-L2 class
// is the sparse one): W = H V with H split at Dc, the first L2 row, into
//   [ Hcc  Hcl ]   dense continuum rows and columns: the lower-triangle product
//   [ Hlc  Hll ]   of k_davidson.hip over the columns < Dc, which reads Hcc's
//                  lower triangle and Hlc once for both of their products;
//                  Hll (classes 2 and 8) as CSR,
// so that a block of b <= 16 vectors costs one read of the continuum columns
// plus the non-zeros of the L2 block instead of the whole dense matrix.
// Every sum has a fixed order, so the result does not depend on timing.
#include <algorithm>

#include "ccham_internal.h"

namespace cch {

// ---------------------------------------------------------------------------
// CSR of the L2 block from the dense matrix (both triangles present)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_l2_nnz(const double *__restrict__ H, int64_t ld, int Dc, int nl2,
                                                int64_t *__restrict__ cnt)
{
    __shared__ int red[256];
    const int r = blockIdx.x;
    const double *row = H + (int64_t)(Dc + r) * ld + Dc;
    int c = 0;
    for (int j = threadIdx.x; j < nl2; j += 256) c += row[j] != 0.0;
    red[threadIdx.x] = c;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) cnt[r] = red[0];
}

// the non-zeros of L2 row r in column order, from offset off[r]
__global__ __launch_bounds__(256) void k_l2_fill(const double *__restrict__ H, int64_t ld, int Dc, int nl2,
                                                 const int64_t *__restrict__ off, int32_t *__restrict__ col,
                                                 double *__restrict__ val)
{
    __shared__ int wsum[4];
    const int r = blockIdx.x;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const double *row = H + (int64_t)(Dc + r) * ld + Dc;
    int64_t base = off[r];
    for (int j0 = 0; j0 < nl2; j0 += 256) {
        const int j = j0 + threadIdx.x;
        const double v = j < nl2 ? row[j] : 0.0;
        const bool nz = v != 0.0;
        const unsigned long long m = __ballot(nz);
        const int before = __popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) wsum[wv] = __popcll(m);
        __syncthreads();
        int woff = 0;
        for (int w = 0; w < wv; ++w) woff += wsum[w];
        const int tot = wsum[0] + wsum[1] + wsum[2] + wsum[3];
        if (nz) {
            col[base + woff + before] = j;
            val[base + woff + before] = v;
        }
        base += tot;
        __syncthreads();   // wsum is written again by the next tile
    }
}

hipError_t launch_l2_csr_count(const double *H, int64_t ld, int Dc, int nl2, int64_t *cnt, hipStream_t st)
{
    if (nl2 <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_l2_nnz, dim3(nl2), dim3(256), 0, st, H, ld, Dc, nl2, cnt);
    return hipGetLastError();
}

hipError_t launch_l2_csr_fill(const double *H, int64_t ld, int Dc, int nl2, const int64_t *off, int32_t *col,
                              double *val, hipStream_t st)
{
    if (nl2 <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_l2_fill, dim3(nl2), dim3(256), 0, st, H, ld, Dc, nl2, off, col, val);
    return hipGetLastError();
}

// VT[i][q] = V[q][i] (0 for q >= b), i < n, q < 2 LPR: the vectors of one row
// side by side for the gathers of the sparse product; record n is zero
template <int LPR>
__global__ __launch_bounds__(256) void k_vt(const double *__restrict__ V, int64_t ldv, int n, int b,
                                            double *__restrict__ VT)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n) return;
#pragma unroll
    for (int q = 0; q < 2 * LPR; ++q) VT[(int64_t)i * (2 * LPR) + q] = i < n && q < b ? V[(int64_t)q * ldv + i] : 0.0;
}

// W[q][Dc + r] (+)= sum over the non-zeros (j, v) of L2 row r of v VT[j][q]
// (added to the continuum part's sums when there are continuum rows, else
// assigned): one wave per row. LPR lanes take one non-zero, two vectors (16
// bytes) each, so an instruction gathers 64 / LPR records of 16 LPR bytes that
// lie in one cache line each. The columns and values of a batch of eight
// gathers go to the lanes through LDS, those of the batch after it are on their
// way, and the gathers of the next batch are issued before the sums of this one:
// with each batch's gathers waited for, the wave was idle most of the time. The
// groups' sums are added across lanes in a fixed order. 88 million non-zeros
// (50000 functions) take 0.90 / 0.64 / 0.56 ms for records of 128 / 64 / 32
// bytes (1.07 / 0.89 / 0.88 before): bound by the records' lines from L2 and,
// for the longest, which do not fit it (6.4 MB), from the last-level cache; the
// three waves a SIMD that the registers leave keep more of them there than four
// do (1.00). A lane per non-zero, with the 16 vectors in its registers, took
// 1.95 ms: each of its eight loads touched 64 different lines.
typedef double px2 __attribute__((ext_vector_type(2)));

struct alignas(16) SpEntry {
    double v;
    int32_t c, pad;
};

template <int LPR>
__global__ __launch_bounds__(256) void k_l2_spmm(const int64_t *__restrict__ off, const int32_t *__restrict__ col,
                                                 const double *__restrict__ val, int Dc, int nl2,
                                                 const double *__restrict__ VT, int b, double *__restrict__ W,
                                                 int64_t ldw, int accumulate)
{
    constexpr int NPS = 64 / LPR;   // non-zeros per instruction
    constexpr int U = 8, C = U / LPR, CH = 64 * C;   // gathers and non-zeros of a batch
    const int lane = threadIdx.x & 63, g = lane / LPR, q2 = lane % LPR;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= nl2) return;   // the whole wave
    const px2 *vl = reinterpret_cast<const px2 *>(VT) + q2;
    const int64_t e1 = off[r + 1];
    px2 acc = (px2){0.0, 0.0};
    int c1[C];
    double v1[C];
    px2 xa[U], xb[U];
    double aa[U], ab[U];
    __shared__ SpEntry ring[4][CH];
    SpEntry *mine = ring[threadIdx.x >> 6];   // this wave's batch
    auto load = [&](int64_t e) {   // past the end: the zero record with the value 0 (a
                                   // column's would spread what is not finite in it)
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const bool in = e + 64 * k + lane < e1;
            c1[k] = in ? col[e + 64 * k + lane] : nl2;
            v1[k] = in ? val[e + 64 * k + lane] : 0.0;
        }
    };
    auto gather = [&](px2 (&x)[U], double (&a)[U]) {
#pragma unroll
        for (int k = 0; k < C; ++k) mine[64 * k + lane] = SpEntry{v1[k], c1[k], 0};
        wave_order();
#pragma unroll
        for (int s = 0; s < U; ++s) {
            const SpEntry t = mine[s * NPS + g];
            a[s] = t.v;
            x[s] = vl[(int64_t)t.c * LPR];
        }
        wave_order();
    };
    auto add = [&](const px2 (&x)[U], const double (&a)[U]) {
#pragma unroll
        for (int s = 0; s < U; ++s) {
            acc.x = fma(a[s], x[s].x, acc.x);
            acc.y = fma(a[s], x[s].y, acc.y);
        }
    };
    int64_t e = off[r];
    load(e);
    gather(xa, aa);
    load(e + CH);
    // a batch: the gathers of the next one, the columns and values of the one
    // after that, then the sums of this one
    auto batch = [&](const px2 (&x)[U], const double (&a)[U], px2 (&xn)[U], double (&an)[U]) {
        if (e + CH < e1) gather(xn, an);
        load(e + 2 * CH);
        add(x, a);
        e += CH;
    };
    while (e < e1) {
        batch(xa, aa, xb, ab);
        if (e >= e1) break;
        batch(xb, ab, xa, aa);
    }
#pragma unroll
    for (int o = 32; o >= LPR; o >>= 1) {
        acc.x += __shfl_xor(acc.x, o, 64);
        acc.y += __shfl_xor(acc.y, o, 64);
    }
    if (lane < LPR) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int q = 2 * q2 + t;
            const double s = t ? acc.y : acc.x;
            if (q < b) W[(int64_t)q * ldw + Dc + r] = accumulate ? W[(int64_t)q * ldw + Dc + r] + s : s;
        }
    }
}

template <int LPR>
static void spmm_launch(const int64_t *off, const int32_t *col, const double *val, int Dc, int nl2, const double *V,
                        int64_t ldv, int b, double *W, int64_t ldw, double *VT, hipStream_t st)
{
    hipLaunchKernelGGL((k_vt<LPR>), dim3(nl2 / 256 + 1), dim3(256), 0, st, V + Dc, ldv, nl2, b, VT);
    hipLaunchKernelGGL((k_l2_spmm<LPR>), dim3((nl2 + 3) / 4), dim3(256), 0, st, off, col, val, Dc, nl2, VT, b, W, ldw,
                       Dc > 0 ? 1 : 0);
}

// doubles of scratch that launch_matvec_l2csr needs
int64_t l2csr_scratch(int D, int Dc)
{
    // the continuum part's sums (a multiple of 16 doubles), then the transposed block
    // with its zero record
    return symv_scratch_doubles(D, Dc) + (int64_t)16 * (D + 1);
}

// P: rows 0..D-1, columns < Dc (leading dimension ldp)
hipError_t launch_matvec_l2csr(const double *P, int64_t ldp, int D, int Dc, const int64_t *off, const int32_t *col,
                               const double *val, const double *V, int64_t ldv, int b, double *W, int64_t ldw,
                               double *Wp, hipStream_t st)
{
    if (D <= 0 || b <= 0) return hipSuccess;
    if (Dc < 0 || Dc > D) return hipErrorInvalidValue;
    const int nl2 = D - Dc;
    double *VT = Wp + symv_scratch_doubles(D, Dc);   // 128-byte aligned
    if (Dc > 0) {
        const hipError_t e = launch_symv(P, ldp, D, Dc, V, ldv, b, W, ldw, Wp, st);
        if (e != hipSuccess) return e;
    }
    for (int q0 = 0; q0 < b && nl2 > 0; q0 += 16) {
        const int bb = std::min(16, b - q0);
        const double *Vq = V + (int64_t)q0 * ldv;
        double *Wq = W + (int64_t)q0 * ldw;
        // the shortest record that holds the vectors: 32, 64 or 128 bytes
        if (bb <= 4) spmm_launch<2>(off, col, val, Dc, nl2, Vq, ldv, bb, Wq, ldw, VT, st);
        else if (bb <= 8) spmm_launch<4>(off, col, val, Dc, nl2, Vq, ldv, bb, Wq, ldw, VT, st);
        else spmm_launch<8>(off, col, val, Dc, nl2, Vq, ldv, bb, Wq, ldw, VT, st);
    }
    return hipGetLastError();
}

}  // namespace cch
