// Excitation scan over determinant pairs (Sec. 2.1, Slater's rules on
// bitstrings): every ket of a row is XORed with the row's bra and popcounted;
// pairs within a double substitution are compacted, in ket order, with their
// holes/particles packed into four 16-bit fields and the sign from masks.
// A count pass sizes the lists at plan time, the emit pass (same scan) writes them
// during the build. Integer work, bit-exact.
// One wave per bra row, 64 kets a step. The connected kets, some hundred of some
// thousand, are listed in LDS as their population counts show them and worked out
// 64 at a time, which also writes the row's pairs side by side: with the labels
// and signs worked out where the pairs were found, nearly every step went through
// all of that for a few lanes, between two barriers of a workgroup per row.
// Bound by the population counts and the reading of the kets from the caches:
// 8000 x 8000 determinants in 0.12 ms, 28000 L2 functions x 8000 in 0.19 (0.40
// and 0.46).
#include "ccham_internal.h"

namespace cch {

constexpr int SCAN_THREADS = 256, SCAN_WAVES = SCAN_THREADS / 64;

template <int W, int MODE, bool EMIT>
__global__ __launch_bounds__(SCAN_THREADS) void k_scan(ScanJob one, const ScanJob *__restrict__ many, int top)
{
    const ScanJob J = many ? many[blockIdx.y] : one;
    const uint64_t *A = J.A, *B = J.B;
    const int nA = J.nA, nB = J.nB;
    const PairList out = J.out;
    if (EMIT) {
        for (int i = blockIdx.x * SCAN_THREADS + threadIdx.x; i < J.nz; i += gridDim.x * SCAN_THREADS)
            J.zero0[i] = J.zero1[i] = 0;
        for (int i = blockIdx.x * SCAN_THREADS + threadIdx.x; i < J.no; i += gridDim.x * SCAN_THREADS) J.ones[i] = -1;
    }
    __shared__ int32_t found[SCAN_WAVES][128];   // connected kets: fewer than 64 and one step's
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int x = blockIdx.x * SCAN_WAVES + wv;
    if (x >= nA) return;   // the whole wave
    int32_t *list = found[wv];
    uint64_t a[W];
#pragma unroll
    for (int w = 0; w < W; ++w) a[w] = A[(size_t)x * W + w];
    const int ylim = (MODE == SCAN_LL) ? x + 1 : nB;
    int64_t at = EMIT ? J.row_off[x] : 0;
    int n = 0;   // listed
    // kets are read two steps ahead
    uint64_t b0[W], b1[W];
    auto load = [&](int y0, uint64_t (&b)[W]) {
#pragma unroll
        for (int w = 0; w < W; ++w) b[w] = B[(size_t)min(y0 + lane, ylim - 1) * W + w];
    };
    if (ylim > 0) {
        load(0, b0);
        load(64, b1);
    }
    for (int y0 = 0; y0 < ylim; y0 += 64) {
        uint64_t b[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            b[w] = b0[w];
            b0[w] = b1[w];
        }
        if (y0 + 128 < ylim) load(y0 + 128, b1);
        int d = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) d += __popcll(a[w] ^ b[w]);
        // L2 x target: one electron more on one side (the continuum one)
        const bool conn = y0 + lane < ylim && (MODE == SCAN_LT ? d <= 3 && (d & 1) : d <= 4);
        const uint64_t bal = __ballot(conn);
        if (!EMIT) {
            at += __popcll(bal);
            continue;
        }
        if (conn) list[n + __popcll(bal & ((1ull << lane) - 1ull))] = y0 + lane;
        n += __popcll(bal);
        wave_order();
        const bool last = y0 + 64 >= ylim;
        while (n >= 64 || (last && n > 0)) {
            const int m = min(n, 64);
            if (lane < m) {
                const int y = list[lane];
#pragma unroll
                for (int w = 0; w < W; ++w) b[w] = B[(size_t)y * W + w];
                int deg, h[2] = {-1, -1}, p[2] = {-1, -1}, s = 1, pt = -1;
                if (MODE == SCAN_LT)
                    deg = excite_cont_l2<W>(b, a, top, h, &pt, &s);   // bra = det y + continuum, ket = L2 x
                else
                    deg = excite<W>(a, b, h, p, &s);
                const int64_t pos = at + lane;
                out.x[pos] = x;
                out.y[pos] = y;
                out.deg[pos] = (int8_t)deg;
                out.phase[pos] = (int8_t)s;
                uint64_t lab;
                if (MODE == SCAN_LT)
                    lab = pack_label(deg == 2 ? pt : CCH_NOLAB, h[0], deg == 2 ? h[1] : CCH_NOLAB, CCH_NOLAB);
                else
                    lab = pack_label(deg >= 1 ? p[0] : CCH_NOLAB, deg >= 1 ? h[0] : CCH_NOLAB,
                                     deg >= 2 ? p[1] : CCH_NOLAB, deg >= 2 ? h[1] : CCH_NOLAB);
                out.label[pos] = lab;
            }
            at += m;
            n -= m;
            const int k = lane < n ? list[64 + lane] : 0;
            wave_order();
            if (lane < n) list[lane] = k;
            wave_order();
        }
    }
    if (!EMIT && lane == 0) J.row_cnt[x] = at;
}

template <int MODE>
static hipError_t scan_mode(int W, const ScanJob &one, const ScanJob *many, int njob, int rows, bool emit, int top,
                            hipStream_t st)
{
    const dim3 g((rows + SCAN_WAVES - 1) / SCAN_WAVES, njob), b(SCAN_THREADS);
#define SCAN_CASE(W_)                                                                                \
    case W_:                                                                                         \
        if (emit) hipLaunchKernelGGL((k_scan<W_, MODE, true>), g, b, 0, st, one, many, top);         \
        else hipLaunchKernelGGL((k_scan<W_, MODE, false>), g, b, 0, st, one, many, top);             \
        return hipGetLastError();
    switch (W) {
        SCAN_CASE(1)
        SCAN_CASE(2)
        SCAN_CASE(3)
        SCAN_CASE(4)
    }
#undef SCAN_CASE
    return hipErrorInvalidValue;
}

static hipError_t scan_any(int mode, int W, const ScanJob &one, const ScanJob *many, int njob, int rows, bool emit,
                           int top, hipStream_t st)
{
    if (rows <= 0 || njob <= 0) return hipSuccess;
    switch (mode) {
    case SCAN_TT: return scan_mode<SCAN_TT>(W, one, many, njob, rows, emit, top, st);
    case SCAN_LL: return scan_mode<SCAN_LL>(W, one, many, njob, rows, emit, top, st);
    case SCAN_LT: return scan_mode<SCAN_LT>(W, one, many, njob, rows, emit, top, st);
    }
    return hipErrorInvalidValue;
}

// mode SCAN_TT/SCAN_LL/SCAN_LT; row_off == nullptr: count pass into row_cnt,
// else emit pass writing pairs from row_off[x].
hipError_t launch_scan(int mode, int W, const ScanJob &one, int top, hipStream_t st)
{
    return scan_any(mode, W, one, nullptr, 1, one.nA, one.row_off != nullptr, top, st);
}

// emit passes of a table of scans on the device, the longest of max_rows rows
hipError_t launch_scans(int mode, int W, const ScanJob *jobs, int njob, int max_rows, int top, hipStream_t st)
{
    hipError_t e = hipSuccess;
    for (int j0 = 0; j0 < njob && e == hipSuccess; j0 += GRID_YZ)
        e = scan_any(mode, W, ScanJob{}, jobs + j0, min(GRID_YZ, njob - j0), max_rows, true, top, st);
    return e;
}

// ---------------------------------------------------------------------------
// exclusive prefix sum of int64 counts, one workgroup (n up to a few 1e5)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void exscan_block(const int64_t *__restrict__ in, int64_t *__restrict__ out, int n,
                                             int64_t *__restrict__ total)
{
    __shared__ int64_t wave[16];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int64_t carry = 0;
    for (int b0 = 0; b0 < n; b0 += 1024) {
        const int i = b0 + threadIdx.x;
        const int64_t v = i < n ? in[i] : 0;
        int64_t s = v;   // inclusive over the wave
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t t = __shfl_up(s, o, 64);
            if (lane >= o) s += t;
        }
        __syncthreads();   // the sums of the chunk before have been read
        if (lane == 63) wave[wv] = s;
        __syncthreads();
        int64_t before = 0, all = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            before += k < wv ? wave[k] : 0;
            all += wave[k];
        }
        if (i < n) out[i] = carry + before + s - v;
        carry += all;
    }
    if (threadIdx.x == 0 && total) *total = carry;
}

__global__ __launch_bounds__(1024) void k_exscan(const int64_t *__restrict__ in, int64_t *__restrict__ out, int n,
                                                 int64_t *__restrict__ total)
{
    exscan_block(in, out, n, total);
}

// first entries of the label buckets, a symmetry pair a workgroup
__global__ __launch_bounds__(1024) void k_slot_start(const PairJob *__restrict__ jobs)
{
    const PairJob &J = jobs[blockIdx.x];
    exscan_block(J.count, J.start, J.n_slot, nullptr);
}

hipError_t launch_slot_start(const PairJob *jobs, int njob, hipStream_t st)
{
    if (njob <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_slot_start, dim3(njob), dim3(1024), 0, st, jobs);
    return hipGetLastError();
}

hipError_t launch_exclusive_scan(const int64_t *in, int64_t *out, int n, int64_t *total, hipStream_t st)
{
    hipLaunchKernelGGL(k_exscan, dim3(1), dim3(1024), 0, st, in, out, n, total);
    return hipGetLastError();
}

}  // namespace cch
