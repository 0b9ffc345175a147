// Class 4: continuum x L2 elements with the one-dimensional contraction of
// Eq. 5, Ht[(i,n,j), l] = sum_m c_imn <eta_im u_j | H | chi_l>
// (Sec. 2.2 "Class 4"; Sec. 3.1: the work is split over the L2 functions).
//
// For one L2 function chi_l the connected target determinants D_m (from the
// excitation scan) give a prototype symbolic element whose integral labels
// carry the continuum index j in one slot; contracting the coefficients over
// m (Eq. 8 in one dimension) and expanding over j is a product
//     out[n][j] = sum_t (coef_t c_{m_t n}) X_t[j]
// where each term t is a row of the one-electron integrals h[H][j] or of
// the (tt|tc) integrals (ab|c j), read for a tile of j:
//   single substitution (chi_l = D_m + h, h of the continuum spin sigma_m), sign s:
//       s [ h_{hj} + sum_{k in D_m} (KK|Hj) - sum_{k in D_m, spin sigma_m} (KH|Kj) ]
//   double (chi_l = D_m - p + h1 + h2), sign s:
//       s [ (P H1|H2 j) d(sp,sh1) d(sigma_m,sh2) - (P H2|H1 j) d(sp,sh2) d(sigma_m,sh1) ]
// (sigma_m the continuum spin given with D_m, alpha unless stated).
// The product runs on the FP64 matrix cores in the 4x4x4 form (a quad of states
// by 16 continuum orbitals by 4 terms): its rows come in fours, so 4 or 5 states
// are not padded to 16, and it issues faster per flop than 16x16x4. A workgroup
// takes a few L2 functions, up to 16 quads of states and up to four tiles of 32
// orbitals, a wave each, two neighbouring orbitals a lane (16-byte loads and
// stores: the rows begin anywhere in a line, and shorter pieces touch more of
// them); the sums stay in registers over all terms. Each function's terms are
// listed in LDS by one wave, a pair a lane; blocks of c4_tb of them are
// multiplied, (coef_t c_{m_t n}) staged in LDS for all waves and the integral
// rows read straight from memory, both for the next block (of the next function
// too) while this one is multiplied: two buffers, one barrier a block. Pairs are
// turned into terms in order and terms are added in order, so the accumulation
// order is fixed.
// Bound by the chain of an item (pairs, determinants, terms, then rows block by
// block) against the items that a CU holds, and by the stores: with the products
// left out it takes three quarters of its time, with the blocks left out a third.
// Measured alone at 40 states, 300 orbitals, 28000 functions of 35 pairs: 1.69 ms
// (0.8 of it matrix-core time, 2.7 GB written); 5.01 with blocks of 64 terms of
// one function on 16x16x4, staged and multiplied in turn. At 5 states, 150
// orbitals, 5000 functions of 5 pairs: 30 us (115).
#include <algorithm>

#include "ccham_internal.h"

namespace cch {

constexpr int C4_TERMS = 400;      // terms listed at a time (>= the most that a pair gives)
constexpr int C4_W = 4;            // waves of a workgroup (more: fewer of them fit a CU, and they wait for each other)
constexpr int C4_LPW = C4_W;       // L2 functions of a workgroup at most: a wave lists each one's terms
// terms per block: the registers of 16 leave one workgroup a CU with many states
constexpr int c4_tb(int nq) { return nq <= 4 ? 16 : 8; }
static_assert(C4_TERMS >= 96 * CCH_MAX_WORDS, "terms of a single substitution: one, the electrons, those of a spin");

// LDS row stride of the staged operand: 4 doubles past a multiple of 16 or the
// like, so that the four terms of an instruction lie in different banks
constexpr int c4_stride(int nq) { return 4 * nq + (nq % 2 ? 0 : 4); }

struct C4List {
    const double *trow[C4_TERMS];
    int32_t tm[C4_TERMS];          // target determinant, the sign of the term in the top bit
    int32_t nt, left;              // terms; pairs of the function not yet turned into terms
};

// one wave lists the terms of the pairs p0 + (0 .. n - 1) behind the first nt,
// as many pairs as fit (at most 64): the terms then, and the pairs taken
__device__ __forceinline__ int c4_pairs(const Class4Args &a, int64_t p0, int64_t n, int lane, int &nt, C4List &sh)
{
    const bool in = lane < n;
    const int64_t pi = p0 + (in ? lane : 0);
    const int deg = a.pl.deg[pi], m = a.pl.y[pi];
    const uint64_t lab = a.pl.label[pi];
    const int neg = a.pl.phase[pi] < 0;
    const int sg = a.cspin ? a.cspin[m] : 0;   // continuum spin
    const int pt = lab_field(lab, 0), h1 = lab_field(lab, 1), h2 = lab_field(lab, 2);
    const size_t n_o = a.n_o;
    // (deg 1: the hole is h1)
    const bool one = in && deg == 1 && (h1 & 1) == sg;
    const bool ta = in && deg != 1 && (pt & 1) == (h1 & 1) && (h2 & 1) == sg;
    const bool tb = in && deg != 1 && (pt & 1) == (h2 & 1) && (h1 & 1) == sg;
    int cnt = (int)ta + (int)tb;
    if (one) {
        const uint64_t mask = sg ? 0xAAAAAAAAAAAAAAAAull : 0x5555555555555555ull;
        cnt = 1;
        for (int w = 0; w < a.W; ++w) {
            const uint64_t d = a.tdets[(size_t)m * a.W + w];
            cnt += __popcll(d) + __popcll(d & mask);
        }
    }
    int incl = cnt + (lane == 0 ? nt : 0);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
    }
    const int taken = __popcll(__ballot(in && incl <= C4_TERMS));   // (incl ascends)
    if (taken > 0) nt = __shfl(incl, taken - 1);
    int o = incl - cnt;
    if (lane < taken) {
        const size_t P = pt >> 1, H1 = h1 >> 1, H2 = h2 >> 1;
        if (ta) {
            sh.trow[o] = a.tttc + ((P * n_o + H1) * n_o + H2) * a.n_cont + a.ja0;
            sh.tm[o++] = m | (neg ? INT32_MIN : 0);
        }
        if (tb) {
            sh.trow[o] = a.tttc + ((P * n_o + H2) * n_o + H1) * a.n_cont + a.ja0;
            sh.tm[o] = m | (neg ? 0 : INT32_MIN);
        }
    }
    // single substitutions, one after another: a spin-orbital of D_m a lane
    for (uint64_t todo = __ballot(one && lane < taken); todo; todo &= todo - 1) {
        const int src = (int)__builtin_ctzll(todo);
        const int mm = __shfl(m, src), sgn = __shfl(neg, src), sp = __shfl(sg, src);
        const size_t H = (size_t)(__shfl(h1, src) >> 1);
        int at = __shfl(incl - cnt, src);
        const int32_t plus = mm | (sgn ? INT32_MIN : 0), minus = mm | (sgn ? 0 : INT32_MIN);
        const uint64_t mask = sp ? 0xAAAAAAAAAAAAAAAAull : 0x5555555555555555ull;
        if (lane == 0) {
            sh.trow[at] = a.h + H * a.n_orb + a.n_o + a.ja0;
            sh.tm[at] = plus;
        }
        ++at;
        for (int w = 0; w < a.W; ++w) {
            const uint64_t d = a.tdets[(size_t)mm * a.W + w], below = d & ((1ull << lane) - 1);
            if ((d >> lane) & 1) {
                const size_t K = (size_t)(64 * w + lane) >> 1;
                const int q = at + __popcll(below) + __popcll(below & mask);
                sh.trow[q] = a.tttc + ((K * n_o + K) * n_o + H) * a.n_cont + a.ja0;
                sh.tm[q] = plus;
                if ((lane & 1) == sp) {
                    sh.trow[q + 1] = a.tttc + ((K * n_o + H) * n_o + K) * a.n_cont + a.ja0;
                    sh.tm[q + 1] = minus;
                }
            }
            at += __popcll(d) + __popcll(d & mask);
        }
    }
    return taken;
}

// one wave lists the next terms of a function whose last `left` pairs end at p1
__device__ __forceinline__ void c4_list(const Class4Args &a, int64_t p1, int left, int lane, C4List &sh)
{
    int nt = 0;
    while (left > 0) {
        const int k = c4_pairs(a, p1 - left, left, lane, nt, sh);
        if (k == 0) break;
        left -= k;
    }
    if (lane == 0) {
        sh.nt = nt;
        sh.left = left;
    }
}

typedef double c4d2 __attribute__((ext_vector_type(2), aligned(8)));

// the states s0 + (0 .. 4 NQ - 1) and the tiles t0 + (0 .. tiles - 1) of 32
// orbitals, one a wave, of the L2 rows l0 .. l0 + nl - 1, nl <= C4_LPW
template <int NQ, bool PAIR>
__device__ __forceinline__ void class4_item(const Class4Args &a, int l0, int nl, int s0, int t0, int tiles,
                                            C4List *__restrict__ lists, double *__restrict__ stage)
{
    constexpr int C4_TB = c4_tb(NQ), LA = c4_stride(NQ), NE = (C4_TB * 4 * NQ + 64 * C4_W - 1) / (64 * C4_W);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lo = lane & 15, hi = lane >> 4;
    const bool mine = wv < tiles;   // this wave has a tile
    // this lane's two orbitals; past the end the last two again, which then are
    // computed and stored twice alike
    const int jo = PAIR ? min(32 * (t0 + wv) + 2 * lo, a.nc - 2) : 0;
    double *out0 = a.H + a.row_l2 * a.ld + a.col0 + jo;

    double acc[2][NQ], st[NE];
    int32_t sg[NE];   // sign of st (applied when it is used, not to wait for it before the products), 0: no term
    c4d2 b[C4_TB / 4];
    auto clear = [&]() {
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[0][q] = acc[1][q] = 0.0;
    };
    // the block of terms tb .. of function il: this thread's part of the staged
    // operand and this wave's rows (past the end the last term again, times 0)
    auto load = [&](int il, int tb) {
        const C4List &sh = lists[il];
        const int tn = min(C4_TB, sh.nt - tb);
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            const int e = (int)threadIdx.x + 64 * C4_W * u, t = e / (4 * NQ), s = e % (4 * NQ);
            const int32_t tm = sh.tm[tb + min(t, tn - 1)];
            st[u] = a.ci[(size_t)(tm & INT32_MAX) * a.S + min(s0 + s, a.S - 1)];
            sg[u] = t < tn ? (tm | 1) : 0;
        }
        if (mine)
#pragma unroll
            for (int u = 0; u < C4_TB / 4; ++u) {
                const double *row = sh.trow[tb + min(4 * u + hi, tn - 1)] + jo;
                if (PAIR) b[u] = *reinterpret_cast<const c4d2 *>(row);
                else b[u] = (c4d2){row[0], 0.0};
            }
    };
    auto multiply = [&](const double *A, const c4d2 (&c)[C4_TB / 4], int u0, int u1) {
#pragma unroll
        for (int u = u0; u < u1; ++u) {
            const double *Au = A + (4 * u + hi) * LA + (lane & 3);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const double av = Au[4 * q];
                acc[0][q] = __builtin_amdgcn_mfma_f64_4x4x4f64(av, c[u].x, acc[0][q], 0, 0, 0);
                if (PAIR) acc[1][q] = __builtin_amdgcn_mfma_f64_4x4x4f64(av, c[u].y, acc[1][q], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);   // (the operands of every step at once would spill)
        }
    };
    // lane holds state 4 q + hi of its orbitals
    auto store = [&](int il) {
        if (!mine) return;
        int nc = a.nc, S = a.S;
        asm volatile("" : "+s"(nc), "+s"(S));   // (the offsets of every quad kept over the functions would spill)
        double *o = out0 + (int64_t)(l0 + il) * a.ld + (int64_t)(s0 + hi) * nc;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if (s0 + 4 * q + hi < S) {
                if (PAIR) *reinterpret_cast<c4d2 *>(o) = (c4d2){acc[0][q], acc[1][q]};
                else if (lo == 0) *o = acc[0][q];
            }
            o += 4 * (int64_t)nc;
        }
    };

    __syncthreads();   // the lists of the item before are no longer read
    if (wv < nl) c4_list(a, a.row_off[l0 + wv] + a.row_cnt[l0 + wv], (int)a.row_cnt[l0 + wv], lane, lists[wv]);
    __syncthreads();
    clear();
    for (int il = 0; il < nl; ++il)   // no terms: the row of the block is zero
        if (lists[il].nt == 0) store(il);
    int il = 0, buf = 0;
    auto next = [&](int i) {   // the next function with terms
        do ++i;
        while (i < nl && lists[i].nt == 0);
        return i;
    };
    il = next(-1);
    if (il < nl) load(il, 0);
    while (il < nl) {
        clear();
        const int ni = next(il);
        for (;;) {
            const int nt = lists[il].nt, left = lists[il].left;
            for (int tb = 0; tb < nt; tb += C4_TB) {
                double *A = stage + buf * C4_TB * LA;
                buf ^= 1;   // (its last readers are behind the barrier of the block between)
#pragma unroll
                for (int u = 0; u < NE; ++u) {
                    const int e = (int)threadIdx.x + 64 * C4_W * u;
                    if (e < C4_TB * 4 * NQ)
                        A[e / (4 * NQ) * LA + e % (4 * NQ)] = sg[u] > 0 ? st[u] : (sg[u] < 0 ? -st[u] : 0.0);
                }
                c4d2 c[C4_TB / 4];
#pragma unroll
                for (int u = 0; u < C4_TB / 4; ++u) c[u] = b[u];
                __syncthreads();
                // the next block, unless its terms are yet to be listed
                const bool more = tb + C4_TB < nt;
                if (more || (left == 0 && ni < nl)) load(more ? il : ni, more ? tb + C4_TB : 0);
                if (mine) {
                    multiply(A, c, 0, C4_TB / 8);
                    if (nt - tb > C4_TB / 2) multiply(A, c, C4_TB / 8, C4_TB / 4);
                }
            }
            if (left == 0) break;
            __syncthreads();   // the list has been read
            if (wv == 0) c4_list(a, a.row_off[l0 + il] + a.row_cnt[l0 + il], left, lane, lists[il]);
            __syncthreads();
            // (the last pairs may give no terms)
            if (lists[il].nt > 0) load(il, 0);
            else if (ni < nl) load(ni, 0);
        }
        store(il);
        il = ni;
    }
}

// how the states and orbitals of a block are split: passes of at most 16 quads
// of states, blocks of at most C4_W tiles of 32 orbitals. Functions go four to a
// workgroup once that leaves 1024 of them
__host__ __device__ inline C4Split c4_split(int S, int nc, int n_l2)
{
    C4Split p;
    const int quads = (S + 3) / 4, tiles = (nc + 31) / 32;
    p.passes = (quads + 15) / 16;
    p.nq = (quads + p.passes - 1) / p.passes;
    p.blocks = (tiles + C4_W - 1) / C4_W;
    p.bt = (tiles + p.blocks - 1) / p.blocks;
    p.blocks = (tiles + p.bt - 1) / p.bt;
    p.lpw = (int64_t)n_l2 * p.passes * p.blocks >= 4096 ? C4_LPW : 1;
    return p;
}

int c4_items(int S, int nc, int n_l2)   // work items of a block
{
    const C4Split p = c4_split(S, nc, n_l2);
    return p.passes * p.blocks * ((n_l2 + p.lpw - 1) / p.lpw);
}

template <int NQ, bool PAIR>
__device__ __forceinline__ void class4_at(const Class4Args &a, const C4Split &p, int n_l2, int g, int part,
                                          C4List *lists, double *stage)
{
    const int t0 = part % p.blocks * p.bt, s0 = part / p.blocks * 4 * p.nq, l0 = g * p.lpw;
    class4_item<NQ, PAIR>(a, l0, min(p.lpw, n_l2 - l0), s0, t0, min(p.bt, (a.nc + 31) / 32 - t0), lists, stage);
}

template <int NQ, bool PAIR>
__global__ __launch_bounds__(64 * C4_W, NQ <= 13 ? 4 : 3) void k_class4(Class4Args a, C4Split p, int n_l2)
{
    __shared__ C4List lists[C4_LPW];
    __shared__ double stage[2 * c4_tb(NQ) * c4_stride(NQ)];
    class4_at<NQ, PAIR>(a, p, n_l2, blockIdx.x, blockIdx.y, lists, stage);
}

// the smallest instance that holds p.nq quads; a single continuum orbital is no
// pair to load
#define C4_INSTANCES(X)                                                                             \
    X(a.nc > 1, 1, true) X(a.nc > 1, 2, true) X(a.nc > 1, 3, true) X(a.nc > 1, 4, true)             \
    X(a.nc > 1, 6, true) X(a.nc > 1, 8, true) X(a.nc > 1, 10, true) X(a.nc > 1, 13, true)           \
    X(a.nc > 1, 16, true) X(true, 4, false) X(true, 16, false)

hipError_t launch_class4(const Class4Args &a, int n_l2, hipStream_t st)
{
    if (n_l2 <= 0 || a.nc <= 0 || a.S <= 0) return hipSuccess;
    if (a.W < 1 || a.W > CCH_MAX_WORDS) return hipErrorInvalidValue;
    const C4Split p = c4_split(a.S, a.nc, n_l2);
    const dim3 g((n_l2 + p.lpw - 1) / p.lpw, p.passes * p.blocks), b(64 * C4_W);
#define C4_RUN(COND, NQ, PAIR)                                              \
    if ((COND) && p.nq <= NQ) {                                                 \
        hipLaunchKernelGGL((k_class4<NQ, PAIR>), g, b, 0, st, a, p, n_l2);        \
        return hipGetLastError();                                               \
    }
    C4_INSTANCES(C4_RUN)
#undef C4_RUN
    return hipErrorInvalidValue;
}

// persistent form over many (instance, symmetry) blocks
__global__ __launch_bounds__(64 * C4_W, 2) void k_class4_batched(const C4Task *__restrict__ tasks, int ntask, int64_t total)
{
    __shared__ C4List lists[C4_LPW];
    __shared__ double stage[2 * c4_tb(16) * c4_stride(16)];
    for (int64_t t = blockIdx.x; t < total; t += gridDim.x) {
        int lo = 0, hi = ntask - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (tasks[mid].first <= t) lo = mid;
            else hi = mid - 1;
        }
        const C4Task &k = tasks[lo];
        const int64_t local = t - k.first;
        const Class4Args &a = k.a;
        const C4Split p = c4_split(a.S, a.nc, k.n_l2);
        const int parts = p.passes * p.blocks, g = (int)(local / parts), part = (int)(local % parts);
#define C4_RUN(COND, NQ, PAIR)                  \
    if ((COND) && p.nq <= NQ) {                     \
        class4_at<NQ, PAIR>(a, p, k.n_l2, g, part, lists, stage); \
        continue;                                   \
    }
        C4_INSTANCES(C4_RUN)
#undef C4_RUN
    }
}

hipError_t launch_class4_batched(const C4Task *tasks, int ntask, int64_t total, int grid, hipStream_t st)
{
    if (total <= 0) return hipSuccess;
    const dim3 g((unsigned)std::min<int64_t>(total, grid)), bl(64 * C4_W);
    hipLaunchKernelGGL(k_class4_batched, g, bl, 0, st, tasks, ntask, total);
    return hipGetLastError();
}

}  // namespace cch
