// Target-space pieces of the continuum-continuum blocks (classes 1, 3, 5,
// 6, 7; Sec. 2.1-2.2 and Eq. 8):
//   * Slater-Condon values H_T[m, m'] of the connected target pairs;
//   * the CI projection (C_i^T H_T C_i')_{nn'} and overlap (C_i^T O C_i')_{nn'}
//     as a row-wise sparse product followed by a small dense product;
//   * the contracted symbolic coefficients D^beta of Eq. 8 for the integral
//     labels (P Q | j j') and (P j' | j Q): spin-summed and alpha-resolved
//     transition densities Gamma_{nn',PQ} = sum_mm' c_imn c_i'm'n' <m|E_PQ|m'>,
//     accumulated per label from the pairs bucketed by label (deterministic).
#include <algorithm>
#include <vector>

#include "ccham_internal.h"

namespace cch {

// ---------------------------------------------------------------------------
// H_T values of the connected pairs, and their buckets by integral label (P, Q):
// key = slot of a degree-1 pair, counted; degree-0 pairs are recorded per bra row;
// degree 2 has no density term. (Counters and records were cleared by the scan.)
// ---------------------------------------------------------------------------
template <int W>
__global__ __launch_bounds__(256) void k_pair_values(TgtInts I, int n_o, const PairJob *__restrict__ jobs)
{
    const PairJob &J = jobs[blockIdx.y];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= J.n) return;
    const int deg = J.pl.deg[i], x = J.pl.x[i], y = J.pl.y[i];
    const uint64_t lab = J.pl.label[i];
    int h[2] = {lab_field(lab, 1), lab_field(lab, 3)};
    int p[2] = {lab_field(lab, 0), lab_field(lab, 2)};
    int k = -1;
    if (deg == 1) k = J.pqidx[(p[0] >> 1) * n_o + (h[0] >> 1)];
    else if (deg == 0) J.d0[x] = i;   // distinct determinants: at most one per bra row
    J.key[i] = k;
    if (k >= 0) atomicAdd((unsigned long long *)&J.count[k], 1ull);
    uint64_t A[W], B[W];
    int dm = 0;   // alpha electrons of the bra minus those of the ket
#pragma unroll
    for (int w = 0; w < W; ++w) {
        A[w] = J.da[(size_t)x * W + w];
        B[w] = J.db[(size_t)y * W + w];
        dm += __popcll(A[w] & 0x5555555555555555ull) - __popcll(B[w] & 0x5555555555555555ull);
    }
    // target determinants of different M_S (given with continuum electrons of
    // different spin): the spin-free H_T has no element between them
    J.hv[i] = dm ? 0.0 : sc_value<W>(I, A, B, deg, h, p, J.pl.phase[i]);
}

// ---------------------------------------------------------------------------
// Y[m][n] = sum over the connected pairs p of row m of hv[p] cb[y_p][n]
// (Yo likewise with weight 1 on degree-0 pairs): one workgroup per row m, each
// of its waves taking every SP_W-th batch of 64 pairs, its lanes split into G
// pair groups x (64 / G) states; the G partial sums of a state are combined by
// xor-shuffles over the group bits and the waves' in order. The pairs' indices
// and values come one pair a lane (the next batch while this one is added) and
// go to the lanes by shuffles, and the CI entries of SP_B steps are on their way
// together. Bound by the longest rows: the low substitutions connect to every
// determinant, the mean row is a tenth of that (3.4 M pairs of 8000
// determinants with 40 states: 1.79 ms with a wave a row that waits for two
// loads a step, 0.77 with the batches, 0.16 with both).
// ---------------------------------------------------------------------------
constexpr int SP_B = 8, SP_W = 8;

__global__ __launch_bounds__(64 * SP_W) void k_spmm_rows(const PairJob *__restrict__ jobs)
{
    const PairJob &J = jobs[blockIdx.y];
    if ((int)blockIdx.x >= J.Ma) return;
    const PairList pl = J.pl;
    const double *hv = J.hv, *cb = J.cb;
    const int Sb = J.Sb;
    int lg_states = 0;   // state lanes: the power of two >= Sb, at most 64
    while ((1 << lg_states) < Sb && lg_states < 6) ++lg_states;
    __shared__ double red[2][SP_W][64];
    const int m = blockIdx.x;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ns = 1 << lg_states;              // state lanes (power of two, <= 64)
    const int lg_g = 6 - lg_states;             // pair groups: 1 << lg_g
    const int nl = lane & (ns - 1), g = lane >> lg_states;
    const int64_t p0 = J.row_off[m], np = J.row_cnt[m];
    // (the flag of a degree-0 pair in the sign bit of its row; a lane past the
    // row's end holds the row's first pair with value 0)
    auto pair = [&](int64_t q, int32_t &y, double &h) {
        const int64_t p = p0 + (q < np ? q : 0);
        y = pl.y[p] | (q < np && pl.deg[p] == 0 ? INT32_MIN : 0);
        h = q < np ? hv[p] : 0.0;
    };
    for (int n0 = 0; n0 < Sb; n0 += ns) {
        const int n = n0 + nl, nc = min(n, Sb - 1);
        double acc = 0.0, acco = 0.0;
        int32_t y = 0;
        double h = 0.0;
        if (64 * wv < np) pair(64 * wv + lane, y, h);
        for (int64_t q0 = 64 * wv; q0 < np; q0 += 64 * SP_W) {
            const int32_t yq = y;
            const double hq = h;
            if (q0 + 64 * SP_W < np) pair(q0 + 64 * SP_W + lane, y, h);
            const int steps = (int)((min<int64_t>(64, np - q0) + (1 << lg_g) - 1) >> lg_g);
            for (int k0 = 0; k0 < steps; k0 += SP_B) {
                double c[SP_B], hh[SP_B];
                int32_t yy[SP_B];
#pragma unroll
                for (int u = 0; u < SP_B; ++u) {
                    const int src = (g + ((k0 + u) << lg_g)) & 63;
                    yy[u] = __shfl(yq, src);
                    hh[u] = __shfl(hq, src);
                    c[u] = cb[(size_t)(yy[u] & INT32_MAX) * Sb + nc];
                }
#pragma unroll
                for (int u = 0; u < SP_B; ++u)
                    if (q0 + g + ((k0 + u) << lg_g) < np && k0 + u < steps) {
                        acc = fma(hh[u], c[u], acc);
                        if (yy[u] < 0) acco += c[u];
                    }
            }
        }
        for (int o = ns; o < 64; o <<= 1) {
            acc += __shfl_xor(acc, o, 64);
            acco += __shfl_xor(acco, o, 64);
        }
        __syncthreads();   // the sums of the previous states have been read
        red[0][wv][lane] = acc;
        red[1][wv][lane] = acco;
        __syncthreads();
        if (wv < 2 && g == 0 && n < Sb) {   // wave 0 adds up Y, wave 1 Yo
            double s = 0.0;
#pragma unroll
            for (int z = 0; z < SP_W; ++z) s += red[wv][z][lane];
            (wv ? J.Yo : J.Y)[(size_t)m * Sb + n] = s;
        }
    }
}

// HT[r] = sum_m ca[m][na[r]] Y[m][nb[r]],  O[r] likewise with Yo.
__global__ __launch_bounds__(256) void k_project(const PairJob *__restrict__ jobs)
{
    const PairJob &J = jobs[blockIdx.y];
    const int r = blockIdx.x, M = J.Ma, Sa = J.Sa, Sb = J.Sb;
    if (r >= J.nrows) return;
    const double *ca = J.ca, *Y = J.Y, *Yo = J.Yo;
    const int n = J.rn[r], n2 = J.rn2[r];
    double a = 0.0, b = 0.0;
    for (int m = threadIdx.x; m < M; m += 256) {
        const double c = ca[(size_t)m * Sa + n];
        a = fma(c, Y[(size_t)m * Sb + n2], a);
        b = fma(c, Yo[(size_t)m * Sb + n2], b);
    }
    __shared__ double ra[256], rb[256];
    ra[threadIdx.x] = a;
    rb[threadIdx.x] = b;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            ra[threadIdx.x] += ra[threadIdx.x + o];
            rb[threadIdx.x] += rb[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        J.HT[r] = ra[0];
        J.O[r] = rb[0];
    }
}

// Target energies on the diagonal (Sec. 3.1, classes 1, 3, 5, 6 and 7): the
// target-only part of every state row (n, n') is replaced by delta_nn' E[n]
// for a symmetry with itself (E given) and by zero between two symmetries.
__global__ __launch_bounds__(256) void k_energy_rows(int nrows, const int32_t *__restrict__ rn,
                                                     const int32_t *__restrict__ rn2,
                                                     const double *__restrict__ E, double *__restrict__ HT)
{
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r < nrows) HT[r] = (E != nullptr && rn[r] == rn2[r]) ? E[rn[r]] : 0.0;
}

hipError_t launch_energy_rows(int nrows, const int32_t *rn, const int32_t *rn2, const double *E, double *HT,
                              hipStream_t st)
{
    if (nrows <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_energy_rows, dim3((nrows + 255) / 256), dim3(256), 0, st, nrows, rn, rn2, E, HT);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// bucketing of pairs by integral label: counting sort with a per-bucket ordering
// by pair index so the accumulation order is fixed.
// ---------------------------------------------------------------------------
__global__ void k_slot_scatter(const PairJob *__restrict__ jobs)
{
    const PairJob &J = jobs[blockIdx.y];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= J.n) return;
    const int k = J.key[i];
    if (k < 0) return;
    const int64_t pos = J.start[k] + (int64_t)atomicAdd((unsigned long long *)&J.cursor[k], 1ull);
    J.sorted[pos] = i;
}

// sort inside each bucket (values are distinct pair indices), one workgroup
// per bucket: chunks of BS_CHUNK sorted in LDS by a bitonic network (padded
// with the largest value), then neighbouring runs merged pass by pass between
// sorted and tmp: an element goes to its index in its own run plus the number
// of the other run's elements below it (binary search). O(n log^2 n) per
// bucket; the result is the ascending order.
constexpr int BS_CHUNK = 512;
__global__ __launch_bounds__(256) void k_bucket_sort(const PairJob *__restrict__ jobs)
{
    const PairJob &J = jobs[blockIdx.y];
    if ((int)blockIdx.x >= J.n_slot) return;
    const int64_t *start = J.start, *count = J.count;
    int64_t *sorted = J.sorted, *tmp = J.tmp;
    __shared__ int64_t buf[BS_CHUNK];
    const int k = blockIdx.x;
    const int64_t s0 = start[k], n = count[k];
    if (n <= 1) return;
    const int64_t big = 0x7fffffffffffffffLL;
    for (int64_t c0 = 0; c0 < n; c0 += BS_CHUNK) {
        const int cn = (int)min((int64_t)BS_CHUNK, n - c0);
        int p2 = 1;
        while (p2 < cn) p2 <<= 1;
        for (int a = threadIdx.x; a < p2; a += 256) buf[a] = a < cn ? sorted[s0 + c0 + a] : big;
        __syncthreads();
        for (int size = 2; size <= p2; size <<= 1)
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                for (int a = threadIdx.x; a < p2 / 2; a += 256) {
                    const int i = 2 * a - (a & (stride - 1)), jx = i + stride;   // bit `stride` of i clear
                    const bool up = (i & size) == 0;
                    const int64_t x = buf[i], y = buf[jx];
                    if ((x > y) == up) {
                        buf[i] = y;
                        buf[jx] = x;
                    }
                }
                __syncthreads();
            }
        for (int a = threadIdx.x; a < cn; a += 256) sorted[s0 + c0 + a] = buf[a];
        __syncthreads();
    }
    int64_t *src = sorted + s0, *dst = tmp + s0;
    for (int64_t run = BS_CHUNK; run < n; run *= 2) {
        for (int64_t a = threadIdx.x; a < n; a += 256) {
            const int64_t r0 = a / (2 * run) * (2 * run);
            const int64_t mid = min(n, r0 + run), end = min(n, r0 + 2 * run);
            const int64_t v = src[a];
            int64_t lo = mid, hi = end, pos = a - r0;   // v in the left run: count the right run's smaller
            if (a >= mid) {
                lo = r0;
                hi = mid;
                pos = a - mid;
            }
            const int64_t base = lo;
            while (lo < hi) {
                const int64_t m = (lo + hi) / 2;
                if (src[m] < v) lo = m + 1;
                else hi = m;
            }
            dst[r0 + pos + (lo - base)] = v;
        }
        __syncthreads();
        int64_t *t = src;
        src = dst;
        dst = t;
    }
    if (src != sorted + s0) {
        for (int64_t a = threadIdx.x; a < n; a += 256) sorted[s0 + a] = src[a];
    }
}

// ---------------------------------------------------------------------------
// Gamma: one workgroup per label slot (P, Q), or in the folded layouts per pair
// of slots (P, Q), (Q, P). Per slot,
//   J[r] = sum over degree-1 pairs with label (P,Q) of s c_a[m][n] c_b[m'][n']
//          (+ for P == Q the degree-0 pairs weighted by the occupation of P)
//   K[r] = the exchange weights: excitations from a hole of the bra's continuum
//          spin to a particle of the ket's (alpha -> alpha when both continuum
//          electrons are alpha) / occupation of P with the continuum spin.
// Output At[k][r], by layout (J, K of slot k1, J', K' of slot k2):
//   GAM_PLAIN  At[t] = J, At[nt + t] = K;
//   GAM_RECT   At[t] = J + J', At[nt + 2t] = K, At[nt + 2t + 1] = K';
//   GAM_SQUARE At[t] = J + J', At[nt + t] = -(K + K') / 2, and for t < n_off
//              At[2 nt + t] = -(K - K') / 2; a single slot (k2 < 0):
//              At[nt + t] = -K.
// ---------------------------------------------------------------------------
// The two weights make J and K products of the CI rows' columns, ca[x]^T w
// cb[y] over the entries of the slot: on the FP64 matrix cores (16x16x4: four
// entries an instruction), a workgroup per slot, 16 states of the bra and NB x
// 16 of the ket. Each of its eight waves takes every eighth batch of 64 entries
// with no barrier: one entry a lane is looked up (the next batch while this one
// is multiplied) and handed out by shuffles, and the CI rows of GAM_U
// instructions are on their way together (NB > 2 leaves two waves a SIMD and
// spills). The waves' sums are added in order.
// Bound by the longest slots: those with P = Q hold every target determinant
// (they are launched first), the others some hundred pairs. 0.20 ms for 8000
// determinants with 40 states and 40 orbitals (3.69 with one batch of 16 entries
// at a time through LDS), 9 us for 500 with 5 states (95).
// ---------------------------------------------------------------------------
constexpr int GAM_W = 8;        // waves
constexpr int GAM_U = 4;        // instructions' operands loaded together

typedef double gam4 __attribute__((ext_vector_type(4)));

template <int W, int NB>
__global__ __launch_bounds__(64 * GAM_W) void k_gamma(const PairJob *__restrict__ jobs, int groups)
{
    const PairJob &J_ = jobs[blockIdx.z / groups];
    const GammaList gl = J_.gl;
    const int Sa = J_.Sa, Sb = J_.Sb, tri = J_.tri, nrows = J_.nrows, M0 = J_.M0;
    const PairList pl = J_.pl;
    const int64_t *sorted = J_.sorted, *d0 = J_.d0;
    const uint64_t *da = J_.da;
    const int8_t *spa = J_.spa, *spb = J_.spb;
    double *At = J_.At;
    __shared__ double red[GAM_W][NB * 256];
    const int t0 = gl.n - 1 - (int)blockIdx.x;
    const int na0 = (int)blockIdx.y * 16, nb0 = (int)blockIdx.z % groups * 16 * NB;
    if (t0 < 0 || na0 >= Sa || nb0 >= Sb || (tri && nb0 > na0 + 15)) return;   // tri: rows n >= n' only
    const int nbt = min(NB, (min(Sb, tri ? na0 + 16 : Sb) - nb0 + 15) / 16);   // ket tiles with an output
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int lo = lane & 15, hi = lane >> 4;
    const int ks[2] = {gl.k1 ? gl.k1[t0] : t0, gl.k2 ? gl.k2[t0] : -1};
    const double *ca_l = J_.ca + min(na0 + lo, Sa - 1);
    const double *cb_l[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) cb_l[b] = J_.cb + min(nb0 + 16 * b + lo, Sb - 1);
    gam4 J[NB], K[2][NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) J[b] = K[0][b] = K[1][b] = (gam4){0.0, 0.0, 0.0, 0.0};
    int waves = 1;   // that had entries
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int k = ks[half];
        if (k < 0) continue;
        const int P = J_.slotP[k], Q = J_.slotQ[k];
        const int64_t s1 = J_.start[k], n1 = J_.count[k];
        const int64_t ntot = n1 + (P == Q ? M0 : 0);
        waves = max(waves, (int)min<int64_t>(GAM_W, (ntot + 63) / 64));
        // entry e: its CI rows and weights (whole numbers from -1 to 2, two apart
        // from 0 in four bits each); past the end the last entry with weights 0
        auto entry = [&](int64_t e, int32_t &x, int32_t &y, int32_t &w) {
            const bool in = e < ntot;
            e = min(e, ntot - 1);
            const int64_t pidx = e < n1 ? sorted[s1 + e] : d0[e - n1];
            int a = 0, b = 0;
            x = y = 0;
            if (pidx >= 0) {   // else no identical ket for this bra row
                x = pl.x[pidx];
                y = pl.y[pidx];
                if (e < n1) {
                    // particle p (in the bra), hole q (in the ket); the Coulomb weight
                    // needs equal continuum spins and a spin-conserving excitation, the
                    // exchange weight a particle of the ket's continuum spin and a hole
                    // of the bra's (the spin-flip pairs of doublet-coupled triplets)
                    const int s = pl.phase[pidx];
                    const uint64_t lab = pl.label[pidx];
                    const int sp = lab_field(lab, 0) & 1, sq = lab_field(lab, 1) & 1;
                    const int sx = spa ? spa[x] : 0, sy = spb ? spb[y] : 0;
                    a = (sx == sy && sp == sq) ? s : 0;
                    b = (sp == sy && sq == sx) ? s : 0;
                } else {
                    // occupation of spatial orbital P in the bra determinant (both spins;
                    // the continuum spin's for the exchange weight)
                    const uint64_t *d = da + (size_t)x * W;
                    const int ka = 2 * P, kb = 2 * P + 1;
                    const int oa = (int)((d[ka >> 6] >> (ka & 63)) & 1ull);
                    const int ob = (int)((d[kb >> 6] >> (kb & 63)) & 1ull);
                    const int sx = spa ? spa[x] : 0;
                    a = oa + ob;
                    b = sx ? ob : oa;
                }
            }
            w = in ? (a + 2) | ((b + 2) << 4) : 0x22;
        };
        int32_t xn = 0, yn = 0, wn = 0;
        if (64 * wv < ntot) entry(64 * wv + lane, xn, yn, wn);
        for (int64_t e0 = 64 * wv; e0 < ntot; e0 += 64 * GAM_W) {
            const int32_t x = xn, y = yn, w = wn;
            if (e0 + 64 * GAM_W < ntot) entry(e0 + 64 * GAM_W + lane, xn, yn, wn);
            const int steps = (int)((min<int64_t>(64, ntot - e0) + 3) / 4);
            for (int u0 = 0; u0 < steps; u0 += GAM_U) {   // (entries past the end: weights 0)
                double av[GAM_U], bv[GAM_U][NB];
                int32_t ww[GAM_U];
#pragma unroll
                for (int u = 0; u < GAM_U; ++u) {
                    const int src = 4 * (u0 + u) + hi;
                    const size_t xx = (size_t)__shfl(x, src) * Sa, yy = (size_t)__shfl(y, src) * Sb;
                    ww[u] = __shfl(w, src);
                    av[u] = ca_l[xx];
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        if (b < nbt) bv[u][b] = cb_l[b][yy];
                }
#pragma unroll
                for (int u = 0; u < GAM_U; ++u) {
                    const double aj = av[u] * (double)((ww[u] & 15) - 2), ak = av[u] * (double)((ww[u] >> 4) - 2);
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        if (b < nbt) {
                            J[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(aj, bv[u][b], J[b], 0, 0, 0);
                            K[half][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ak, bv[u][b], K[half][b], 0, 0, 0);
                        }
                }
            }
        }
    }
    // the waves' sums, in order; a lane holds states na0 + hi + 4 v of the bra
    // and nb0 + 16 b + lo of the ket
    constexpr int NO = (NB * 256 + 64 * GAM_W - 1) / (64 * GAM_W);   // outputs a thread
    double out[3][NO];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        if (q == 2 && ks[1] < 0) break;
        __syncthreads();
        if (wv < waves)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    red[wv][256 * b + 16 * (hi + 4 * v) + lo] = q == 0 ? J[b][v] : K[q - 1][b][v];
        __syncthreads();
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            const int e = (int)threadIdx.x + 64 * GAM_W * o;
            double s = 0.0;
            if (e < 256 * nbt)
                for (int z = 0; z < waves; ++z) s += red[z][e];
            out[q][o] = s;
        }
    }
    const size_t t = t0, nt = gl.n;
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int e = (int)threadIdx.x + 64 * GAM_W * o;
        const int n = na0 + ((e >> 4) & 15), n2 = nb0 + 16 * (e >> 8) + (e & 15);
        if (e >= 256 * nbt || n >= Sa || n2 >= Sb || (tri && n2 > n)) continue;
        const size_t r = tri ? (size_t)n * (n + 1) / 2 + n2 : (size_t)n * Sb + n2;
        At[t * nrows + r] = out[0][o];
        if (gl.mode == GAM_PLAIN) {
            At[(nt + t) * nrows + r] = out[1][o];
        } else if (gl.mode == GAM_RECT) {
            At[(nt + 2 * t) * nrows + r] = out[1][o];
            At[(nt + 2 * t + 1) * nrows + r] = out[2][o];
        } else if (ks[1] < 0) {
            At[(nt + t) * nrows + r] = -out[1][o];
        } else {
            At[(nt + t) * nrows + r] = -0.5 * (out[1][o] + out[2][o]);
            At[(2 * nt + t) * nrows + r] = -0.5 * (out[1][o] - out[2][o]);
        }
    }
}

hipError_t launch_slot_start(const PairJob *jobs, int njob, hipStream_t st);   // k_scan.hip

// the stages for the symmetry pairs h[0 .. nj - 1] of the table jobs
static hipError_t target_sums(int W, const TgtInts &I, int n_o, const PairJob *h, const PairJob *jobs, unsigned nj,
                              int NB, int groups, hipStream_t st)
{
    int64_t n = 0;
    int M = 0, nrows = 0, slots = 0, gl = 0, Sa = 0;
    for (unsigned i = 0; i < nj; ++i) {
        const PairJob &p = h[i];
        n = std::max(n, p.n);
        M = std::max(M, p.Ma);
        nrows = std::max(nrows, p.nrows);
        slots = std::max(slots, p.n_slot);
        gl = std::max(gl, p.gl.n);
        Sa = std::max(Sa, p.Sa);
    }
    const dim3 gp((unsigned)((n + 255) / 256), nj), b(256);
    if (n > 0) {
        switch (W) {
        case 1: hipLaunchKernelGGL((k_pair_values<1>), gp, b, 0, st, I, n_o, jobs); break;
        case 2: hipLaunchKernelGGL((k_pair_values<2>), gp, b, 0, st, I, n_o, jobs); break;
        case 3: hipLaunchKernelGGL((k_pair_values<3>), gp, b, 0, st, I, n_o, jobs); break;
        case 4: hipLaunchKernelGGL((k_pair_values<4>), gp, b, 0, st, I, n_o, jobs); break;
        default: return hipErrorInvalidValue;
        }
    }
    if (M > 0) hipLaunchKernelGGL(k_spmm_rows, dim3(M, nj), dim3(64 * SP_W), 0, st, jobs);
    if (nrows > 0) hipLaunchKernelGGL(k_project, dim3(nrows, nj), b, 0, st, jobs);
    if (slots > 0) {
        const hipError_t e = launch_slot_start(jobs, (int)nj, st);
        if (e != hipSuccess) return e;
        if (n > 0) {
            hipLaunchKernelGGL(k_slot_scatter, gp, b, 0, st, jobs);
            hipLaunchKernelGGL(k_bucket_sort, dim3(slots, nj), b, 0, st, jobs);
        }
    }
    if (gl > 0 && nrows > 0) {
        const dim3 g(gl, (Sa + 15) / 16, groups * nj), t(64 * GAM_W);
#define GAMMA(W_, NB_) \
    case 8 * W_ + NB_: hipLaunchKernelGGL((k_gamma<W_, NB_>), g, t, 0, st, jobs, groups); break;
        switch (8 * W + NB) {
            GAMMA(1, 1) GAMMA(1, 2) GAMMA(2, 1) GAMMA(2, 2) GAMMA(3, 1) GAMMA(3, 2) GAMMA(4, 1) GAMMA(4, 2)
        default: return hipErrorInvalidValue;
        }
#undef GAMMA
    }
    return hipGetLastError();
}

// every symmetry pair's target elements, projections, label buckets and densities;
// h: the table's copy on the host (its sizes), jobs: the table. One launch a stage
// for as many pairs as a grid holds (k_gamma has up to eight workgroups a pair
// along z): a pair's own launches, eleven each, cost more than their work below
// some thousand determinants.
hipError_t launch_target_sums(int W, const TgtInts &I, int n_o, const std::vector<PairJob> &h, const PairJob *jobs,
                              hipStream_t st)
{
    int Sb = 1;
    for (const PairJob &p : h) Sb = std::max(Sb, p.Sb);
    const int NB = Sb > 16 ? 2 : 1, groups = (Sb + 16 * NB - 1) / (16 * NB);
    const size_t most = (size_t)(GRID_YZ / groups);
    hipError_t e = hipSuccess;
    for (size_t j0 = 0; j0 < h.size() && e == hipSuccess; j0 += most)
        e = target_sums(W, I, n_o, h.data() + j0, jobs + j0, (unsigned)std::min(most, h.size() - j0), NB, groups, st);
    return e;
}

}  // namespace cch
