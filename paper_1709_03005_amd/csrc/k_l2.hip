// Classes 2 and 8: the pure L2 block <chi_l | H | chi_l'> with no
// contraction (Sec. 2.2), evaluated by Slater's rules on bitstrings for the
// lower triangle (Sec. 3.1 collapses the triangular double loop into one
// loop; here each workgroup takes one tile of TR rows x 64 columns of the
// flattened lower triangle).
//
// A tile is scanned first: every pair takes an XOR and a popcount per word,
// and the few within a double substitution (1.3% of the pairs at 40000
// functions) go to a list in LDS, single substitutions from one end and
// double ones from the other. The list is then evaluated by full waves on
// like work -- in one pass over the tile half of the waves had at least one
// connected lane, and the other 63 waited for its integrals -- and the tile
// is written from LDS to both triangles, so no later pass reads the L2 block
// back. 40000 functions, both triangles (12.8 GB) in 5.1 ms alone, where the
// writes by themselves would take 2.0: a tile's scan, evaluation and writes follow
// one another, and three workgroups (43 KB of LDS each) a compute unit hide part
// of that. Beside class 4 the one-pass form took 6.9 ms for the lower triangle
// and the mirror 3.0 ms for the rest, this one 7.6 in all; 2997 functions 0.06 ms
// instead of 0.320 + 0.03.
#include <algorithm>

#include "ccham_internal.h"

namespace cch {

// tiles of TR rows x 64 columns (TR divides 64) in the rows before tile row i
template <int TR>
__host__ __device__ __forceinline__ int64_t l2_tiles_before(int64_t i)
{
    constexpr int64_t f = 64 / TR;   // tile rows per 64 rows: tile row i has i / f + 1 tiles
    const int64_t m = i / f, r = i % f;
    return f * (m * (m + 1) / 2) + r * (m + 1);
}

template <int TR>
__device__ __forceinline__ void tri_decode(int64_t b, int64_t *ti, int64_t *tj)
{
    int64_t i = (int64_t)((sqrt(8.0 * (double)b * (TR / 64.0) + 1.0) - 1.0) * 0.5 * (64 / TR));
    while (l2_tiles_before<TR>(i) > b) --i;
    while (l2_tiles_before<TR>(i + 1) <= b) ++i;
    *ti = i;
    *tj = b - l2_tiles_before<TR>(i);
}

template <int W, int TR>
struct L2Shared {
    uint64_t bra[TR][W], ket[64][W];
    double tile[TR][65];
    uint16_t list[TR * 64];
    int n1, n2;
};

template <int W, int TR>
__device__ __forceinline__ void l2_tile(const L2Args &a, int64_t b, L2Shared<W, TR> &sh)
{
    int64_t ti, tj;
    tri_decode<TR>(b, &ti, &tj);
    const int l0 = (int)(ti * TR), k0 = (int)(tj * 64);
    __syncthreads();   // the LDS of the previous tile of a persistent loop
    for (int t = threadIdx.x; t < 64 * W; t += 256) {
        const int r = t / W, w = t % W;
        if (r < TR) sh.bra[r][w] = (l0 + r < a.n_l2) ? a.dets[(size_t)(l0 + r) * W + w] : 0ull;
        sh.ket[r][w] = (k0 + r < a.n_l2) ? a.dets[(size_t)(k0 + r) * W + w] : 0ull;
    }
    if (threadIdx.x == 0) sh.n1 = sh.n2 = 0;
    __syncthreads();
    const int c = threadIdx.x & 63, lc = k0 + c;
    {
        uint64_t B[W];
#pragma unroll
        for (int w = 0; w < W; ++w) B[w] = sh.ket[c][w];
#pragma unroll 4
        for (int r = threadIdx.x >> 6; r < TR; r += 4) {
            const int lr = l0 + r;
            int x = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) x += __popcll(sh.bra[r][w] ^ B[w]);
            sh.tile[r][c] = 0.0;
            if (x <= 4 && lc <= lr && lr < a.n_l2) {
                const int at = x <= 2 ? atomicAdd(&sh.n1, 1) : TR * 64 - 1 - atomicAdd(&sh.n2, 1);
                sh.list[at] = (uint16_t)(r * 64 + c);
            }
        }
    }
    __syncthreads();
    const int n1 = sh.n1, n2 = sh.n2;
    for (int t = threadIdx.x; t < n1 + n2; t += 256) {
        const int rc = t < n1 ? sh.list[t] : sh.list[TR * 64 - 1 - (t - n1)];
        uint64_t A[W], B[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            A[w] = sh.bra[rc >> 6][w];
            B[w] = sh.ket[rc & 63][w];
        }
        int h[2], p[2], s;
        const int deg = excite<W>(A, B, h, p, &s);
        sh.tile[rc >> 6][rc & 63] = sc_value<W>(a.I, A, B, deg, h, p, s);
    }
    __syncthreads();
    double *H = a.H + a.row0 * a.ld + a.row0;
    if (lc < a.n_l2) {
#pragma unroll 4
        for (int r = threadIdx.x >> 6; r < TR; r += 4) {
            const int lr = l0 + r;
            if (lr < a.n_l2 && lc <= lr) H[(int64_t)lr * a.ld + lc] = sh.tile[r][c];
        }
    }
    if (!a.both) return;
    // column by column: row k0 + cc of the upper triangle, TR elements
    const int rr = threadIdx.x % TR;
#pragma unroll 4
    for (int cc = threadIdx.x / TR; cc < 64; cc += 256 / TR) {
        const int lr = l0 + rr, lk = k0 + cc;
        if (lr < a.n_l2 && lk < lr) H[(int64_t)lk * a.ld + lr] = sh.tile[rr][cc];
    }
}

template <int W, int TR>
__global__ __launch_bounds__(256) void k_l2_block(L2Args a)
{
    __shared__ L2Shared<W, TR> sh;
    l2_tile<W, TR>(a, blockIdx.x, sh);
}

template <int W>
static void l2_launch(const L2Args &a, hipStream_t st)
{
    // 64 x 64 tiles write whole 512-byte runs of both triangles; below 1024 of
    // them (2900 functions) the chip is not full and four times as many tiles of
    // 16 rows finish sooner
    const int64_t T = (a.n_l2 + 63) / 64, T16 = (a.n_l2 + 15) / 16;
    if (T * (T + 1) / 2 >= 1024)
        hipLaunchKernelGGL((k_l2_block<W, 64>), dim3((unsigned)l2_tiles_before<64>(T)), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((k_l2_block<W, 16>), dim3((unsigned)l2_tiles_before<16>(T16)), dim3(256), 0, st, a);
}

hipError_t launch_l2_block(int W, const L2Args &a, hipStream_t st)
{
    if (a.n_l2 <= 0) return hipSuccess;
    switch (W) {
    case 1: l2_launch<1>(a, st); break;
    case 2: l2_launch<2>(a, st); break;
    case 3: l2_launch<3>(a, st); break;
    case 4: l2_launch<4>(a, st); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// L2 functions given as CSFs, chi_l = sum_t coef_t |det_t> (Eq. 1's second
// sum over configuration state functions): the lower triangle of the matrix
// over the CSFs from the lower triangle of the one built over the distinct L2
// determinants (Hd, not mirrored): continuum rows are copied, a class-4 row
// is sum_t coef_t Hd[det_t][c], an L2 x L2 element sum_t sum_u coef_t coef_u
// Hd[det_t][det_u] (read from the lower triangle), terms in input order. One
// workgroup per row.
__global__ __launch_bounds__(256) void k_l2csf_gather(const double *__restrict__ Hd, int64_t ldd, int Dc,
                                                      const int32_t *__restrict__ start,
                                                      const int32_t *__restrict__ det,
                                                      const double *__restrict__ coef, double *__restrict__ H,
                                                      int64_t ld)
{
    const int64_t r = blockIdx.x;
    double *out = H + r * ld;
    if (r < Dc) {
        const double *in = Hd + r * ldd;
        for (int64_t c = threadIdx.x; c <= r; c += blockDim.x) out[c] = in[c];
        return;
    }
    const int a = (int)(r - Dc);
    const int t0 = start[a], t1 = start[a + 1];
    for (int64_t c = threadIdx.x; c <= r; c += blockDim.x) {
        double v = 0.0;
        if (c < Dc) {
            for (int t = t0; t < t1; ++t) v += coef[t] * Hd[(Dc + (int64_t)det[t]) * ldd + c];
        } else {
            const int b = (int)(c - Dc), u0 = start[b], u1 = start[b + 1];
            for (int t = t0; t < t1; ++t) {
                const int64_t x = Dc + (int64_t)det[t];
                double s = 0.0;
                for (int u = u0; u < u1; ++u) {
                    const int64_t y = Dc + (int64_t)det[u];
                    s += coef[u] * (x >= y ? Hd[x * ldd + y] : Hd[y * ldd + x]);
                }
                v += coef[t] * s;
            }
        }
        out[c] = v;
    }
}

hipError_t launch_l2csf_gather(const double *Hd, int64_t ldd, int Dc, int ncsf, const int32_t *start,
                               const int32_t *det, const double *coef, double *H, int64_t ld, hipStream_t st)
{
    const int64_t D = (int64_t)Dc + ncsf;
    if (D <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_l2csf_gather, dim3((unsigned)D), dim3(256), 0, st, Hd, ldd, Dc, start, det, coef, H, ld);
    return hipGetLastError();
}

// tiles of an instance in the persistent form
int64_t l2_tiles(int n_l2)
{
    const int64_t T = (n_l2 + 63) / 64;
    return T * (T + 1) / 2;
}

// persistent form over many instances with the same word count
template <int W>
__global__ __launch_bounds__(256) void k_l2_batched(const L2Task *__restrict__ tasks, int ntask, int64_t total)
{
    __shared__ L2Shared<W, 64> sh;
    for (int64_t t = blockIdx.x; t < total; t += gridDim.x) {
        int lo = 0, hi = ntask - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (tasks[mid].first <= t) lo = mid;
            else hi = mid - 1;
        }
        l2_tile<W, 64>(tasks[lo].a, t - tasks[lo].first, sh);
    }
}

hipError_t launch_l2_batched(int W, const L2Task *tasks, int ntask, int64_t total, int grid, hipStream_t st)
{
    if (total <= 0) return hipSuccess;
    const dim3 g((unsigned)std::min<int64_t>(total, grid)), bl(256);
    switch (W) {
    case 1: hipLaunchKernelGGL((k_l2_batched<1>), g, bl, 0, st, tasks, ntask, total); break;
    case 2: hipLaunchKernelGGL((k_l2_batched<2>), g, bl, 0, st, tasks, ntask, total); break;
    case 3: hipLaunchKernelGGL((k_l2_batched<3>), g, bl, 0, st, tasks, ntask, total); break;
    case 4: hipLaunchKernelGGL((k_l2_batched<4>), g, bl, 0, st, tasks, ntask, total); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace cch
