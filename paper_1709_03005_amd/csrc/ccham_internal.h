// Internal declarations shared by the ccham kernels and the host runtime.
// Device helpers here implement Slater's rules on bitstring determinants
// (Sec. 2.1 of the MPI-SCATCI paper: XOR + popcount for the excitation
// degree, masks counting the occupied spin-orbitals between the differing
// ones for the sign), written for 64-bit words on gfx950.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define CCH_MAXW 4          // up to 256 target spin-orbitals per determinant
#define CCH_NOLAB 0xFFFFu

namespace cch {

// ---------------------------------------------------------------------------
// bit helpers (no shift by 64 anywhere: an index that is a multiple of 64 is
// the case the paper singles out for wrong masks)
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t lowmask(int x)   // bits [0, x), x clamped to [0, 64]
{
    return x >= 64 ? ~0ull : (x <= 0 ? 0ull : ((1ull << x) - 1ull));
}

template <int W>
__device__ __forceinline__ int count_between(const uint64_t *d, int lo, int hi)
{
    // set bits of d strictly between spin-orbitals lo < hi
    int c = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const int b = 64 * w;
        uint64_t m = lowmask(hi - b) & ~lowmask(lo + 1 - b);
        c += __popcll(d[w] & m);
    }
    return c;
}

template <int W>
__device__ __forceinline__ int first_bits(const uint64_t *x, int *out, int maxn)
{
    // ascending indices of the set bits of x (at most maxn)
    int n = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        uint64_t v = x[w];
        while (v && n < maxn) {
            out[n++] = 64 * w + (int)__builtin_ctzll(v);
            v &= v - 1;
        }
    }
    return n;
}

// the two lowest set bits of x, ascending (-1 where absent), without loops
// or branches: each word offers its lowest bit and the bit after it, and the
// first two offers found in word order are kept (the excitation scan runs
// this for every determinant pair, with lanes of one wave on different pairs)
template <int W>
__device__ __forceinline__ void low_two(const uint64_t *x, int *b0, int *b1)
{
    int f0 = -1, f1 = -1;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const uint64_t v = x[w], rest = v & (v - 1ull);
        const int t0 = v ? 64 * w + (int)__builtin_ctzll(v) : -1;
        const int t1 = rest ? 64 * w + (int)__builtin_ctzll(rest) : -1;
        f1 = f0 < 0 ? t1 : (f1 < 0 ? t0 : f1);
        f0 = f0 < 0 ? t0 : f0;
    }
    *b0 = f0;
    *b1 = f1;
}

__device__ __forceinline__ uint64_t pack_label(int f0, int f1, int f2, int f3)
{
    return (uint64_t)(uint16_t)f0 | ((uint64_t)(uint16_t)f1 << 16) |
           ((uint64_t)(uint16_t)f2 << 32) | ((uint64_t)(uint16_t)f3 << 48);
}

__device__ __forceinline__ int lab_field(uint64_t lab, int f) { return (int)((lab >> (16 * f)) & 0xFFFFu); }

// Excitation of bra A from ket B, equal electron counts. Returns the degree
// (0..2) or 3 when more than a double substitution apart. Holes = B & ~A,
// particles = A & ~B, ascending, paired in order; sign of
// A = s a+_p2 a_h2 a+_p1 a_h1 B.
template <int W>
__device__ __forceinline__ int excite(const uint64_t *A, const uint64_t *B, int *h, int *p, int *sign)
{
    int x = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) x += __popcll(A[w] ^ B[w]);
    if (x > 4) return 3;
    const int deg = x >> 1;
    if (deg == 0) { *sign = 1; return 0; }
    uint64_t hb[W], pb[W];
#pragma unroll
    for (int w = 0; w < W; ++w) { hb[w] = B[w] & ~A[w]; pb[w] = A[w] & ~B[w]; }
    low_two<W>(hb, &h[0], &h[1]);
    low_two<W>(pb, &p[0], &p[1]);
    int c = count_between<W>(B, min(h[0], p[0]), max(h[0], p[0]));
    if (deg == 2) {
        uint64_t B2[W];
#pragma unroll
        for (int w = 0; w < W; ++w) B2[w] = B[w];
        B2[h[0] >> 6] ^= 1ull << (h[0] & 63);
        B2[p[0] >> 6] ^= 1ull << (p[0] & 63);
        c += count_between<W>(B2, min(h[1], p[1]), max(h[1], p[1]));
    }
    *sign = (c & 1) ? -1 : 1;
    return deg;
}

// Continuum function (target det D of N electrons plus the alpha continuum
// electron above every target spin-orbital, index `top` = 2 n_o) as bra,
// against an L2 det L (N+1 target electrons) as ket. Returns the degree of
// the (N+1)-electron pair (1..2) or 3. h[0..deg) = holes (in L), pt = the
// target particle (in D) for degree 2.
template <int W>
__device__ __forceinline__ int excite_cont_l2(const uint64_t *D, const uint64_t *L, int top, int *h,
                                              int *pt, int *sign)
{
    int x = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) x += __popcll(D[w] ^ L[w]);
    if (x > 3 || !(x & 1)) return 3;
    const int deg = (x + 1) >> 1;   // 1 or 2
    uint64_t hb[W], pb[W];
#pragma unroll
    for (int w = 0; w < W; ++w) { hb[w] = L[w] & ~D[w]; pb[w] = D[w] & ~L[w]; }
    low_two<W>(hb, &h[0], &h[1]);
    int c;
    if (deg == 1) {
        *pt = -1;
        c = count_between<W>(L, h[0], top);
    } else {
        int unused;
        low_two<W>(pb, pt, &unused);
        c = count_between<W>(L, min(h[0], *pt), max(h[0], *pt));
        uint64_t L2[W];
#pragma unroll
        for (int w = 0; w < W; ++w) L2[w] = L[w];
        L2[h[0] >> 6] ^= 1ull << (h[0] & 63);
        L2[*pt >> 6] ^= 1ull << (*pt & 63);
        c += count_between<W>(L2, h[1], top);
    }
    *sign = (c & 1) ? -1 : 1;
    return deg;
}

// ---------------------------------------------------------------------------
// short scalar chains and wave reductions
// ---------------------------------------------------------------------------
// the wave's LDS accesses before this one are done before those after it (a wave's
// LDS instructions run in order: no instruction is needed, only their order kept)
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// 1/q from the hardware estimate and two Newton-Raphson corrections
// r <- r + r (1 - q r), each squaring the relative error: a short dependent
// chain for the recurrences below, within about one ulp of the quotient
__device__ __forceinline__ double rr_recip(double q)
{
    double r = __builtin_amdgcn_rcp(q);
    double e = fma(-q, r, 1.0);
    r = fma(r, e, r);
    e = fma(-q, r, 1.0);
    return fma(r, e, r);
}

// 1/sqrt(x), x > 0, from the hardware estimate and two Newton-Raphson
// corrections r <- r + r (1 - x r^2) / 2
__device__ __forceinline__ double rr_rsqrt(double x)
{
    double r = __builtin_amdgcn_rsq(x);
    double e = fma(-x * r, r, 1.0);
    r = fma(0.5 * r, e, r);
    e = fma(-x * r, r, 1.0);
    return fma(0.5 * r, e, r);
}

// Cross-lane helpers on doubles as two 32-bit halves: DPP moves (row shifts
// and row broadcasts) and readlane with a wave-uniform lane index.
struct RrI2 {
    int x, y;
};

template <int CTRL, int ROW_MASK, int BANK_MASK>
__device__ __forceinline__ double rr_dpp(double v)
{
    RrI2 a = __builtin_bit_cast(RrI2, v);
    a.x = __builtin_amdgcn_update_dpp(0, a.x, CTRL, ROW_MASK, BANK_MASK, true);
    a.y = __builtin_amdgcn_update_dpp(0, a.y, CTRL, ROW_MASK, BANK_MASK, true);
    return __builtin_bit_cast(double, a);
}

__device__ __forceinline__ double rr_rl(double v, int lane)
{
    RrI2 a = __builtin_bit_cast(RrI2, v);
    a.x = __builtin_amdgcn_readlane(a.x, lane);
    a.y = __builtin_amdgcn_readlane(a.y, lane);
    return __builtin_bit_cast(double, a);
}

// sum over the 64 lanes, returned to every lane: partial sums of 4 within
// each row of 16 (row_shr 1..3), of 8 and 16 (row_shr 4, 8 on the upper
// banks), then rows 0+1 and 2+3 (row_bcast15) and all four (row_bcast31)
// collect in lane 63. Fixed order, so every wave gets the same bits.
__device__ __forceinline__ double rr_wsum(double v)
{
    double s = v + rr_dpp<0x111, 0xf, 0xf>(v);
    s += rr_dpp<0x112, 0xf, 0xf>(v);
    s += rr_dpp<0x113, 0xf, 0xf>(v);
    s += rr_dpp<0x114, 0xf, 0xe>(s);
    s += rr_dpp<0x118, 0xf, 0xc>(s);
    s += rr_dpp<0x142, 0xa, 0xf>(s);
    s += rr_dpp<0x143, 0xc, 0xf>(s);
    return rr_rl(s, 63);
}

// ---------------------------------------------------------------------------
// integrals over target orbitals
// ---------------------------------------------------------------------------
struct TgtInts {
    const double *h;      // full one-electron matrix [n_orb][n_orb]
    const double *tttt;   // [n_o]^4
    int n_o, n_orb;
    double e_core;
};

__device__ __forceinline__ double g4(const TgtInts &I, int P, int Q, int R, int S)
{
    return I.tttt[(((size_t)P * I.n_o + Q) * I.n_o + R) * I.n_o + S];
}

// the next four set bits of x (taken out of it); where fewer are left, `ok`
// is false and the index 0
__device__ __forceinline__ void next_four(uint64_t &x, int base, int *k, bool *ok)
{
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        ok[u] = x != 0;
        k[u] = ok[u] ? base + (int)__builtin_ctzll(x) : 0;
        x &= x - 1;
    }
}

// <A|H|B> for target-only determinants connected by degree 0..2, from the
// excitation (holes h, particles p, sign s). The degree-1 sum runs over all
// of B: its k = h term cancels exactly. The sums over electrons take their
// integrals four electrons at a time and add them in order (one load after
// the other left a diagonal element of ten electrons at 45 dependent steps).
template <int W>
__device__ double sc_value(const TgtInts &I, const uint64_t *A, const uint64_t *B, int deg,
                           const int *h, const int *p, int s)
{
    if (deg == 0) {
        int occ[64];
        uint64_t t[W];
#pragma unroll
        for (int w = 0; w < W; ++w) t[w] = A[w];
        const int n = first_bits<W>(t, occ, 64);
        double e = I.e_core, e2 = 0.0;
        for (int a = 0; a < n; ++a) {
            const int ka = occ[a], Pa = ka >> 1;
            e += I.h[(size_t)Pa * I.n_orb + Pa];
#pragma unroll
            for (int w = 0; w < W; ++w) {
                uint64_t x = A[w] & lowmask(ka - 64 * w);
                while (x) {
                    int k[4];
                    bool ok[4];
                    double gc[4], gx[4];
                    next_four(x, 64 * w, k, ok);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int Pb = k[u] >> 1;
                        gc[u] = g4(I, Pa, Pa, Pb, Pb);
                        gx[u] = g4(I, Pa, Pb, Pb, Pa);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        double v = gc[u];
                        if ((ka & 1) == (k[u] & 1)) v -= gx[u];
                        if (ok[u]) e2 += v;
                    }
                }
            }
        }
        return e + e2;
    }
    if (deg == 1) {
        if ((h[0] & 1) != (p[0] & 1)) return 0.0;
        const int P = p[0] >> 1, H = h[0] >> 1, sp = p[0] & 1;
        double v = I.h[(size_t)P * I.n_orb + H];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            uint64_t x = B[w];
            while (x) {
                int k[4];
                bool ok[4];
                double gc[4], gx[4];
                next_four(x, 64 * w, k, ok);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int K = k[u] >> 1;
                    gc[u] = g4(I, P, H, K, K);
                    gx[u] = (k[u] & 1) == sp ? g4(I, P, K, K, H) : 0.0;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (ok[u]) v += gc[u];
                    if (ok[u] && (k[u] & 1) == sp) v -= gx[u];
                }
            }
        }
        return s * v;
    }
    // degree 2
    double v = 0.0;
    if ((p[0] & 1) == (h[0] & 1) && (p[1] & 1) == (h[1] & 1))
        v += g4(I, p[0] >> 1, h[0] >> 1, p[1] >> 1, h[1] >> 1);
    if ((p[0] & 1) == (h[1] & 1) && (p[1] & 1) == (h[0] & 1))
        v -= g4(I, p[0] >> 1, h[1] >> 1, p[1] >> 1, h[0] >> 1);
    return s * v;
}

// ---------------------------------------------------------------------------
// pair lists
// ---------------------------------------------------------------------------
struct PairList {
    int32_t *x, *y;      // bra index, ket index
    int8_t *deg;
    int8_t *phase;
    uint64_t *label;
};

enum ScanMode { SCAN_TT = 0, SCAN_LL = 1, SCAN_LT = 2 };

// workgroups of a launch along y or z at most
constexpr int GRID_YZ = 65535;

// one excitation scan: bras A against kets B; emits from row_off[x], or counts
// into row_cnt (row_off = nullptr). An emitting scan may also clear words that
// later kernels of the stream count in: zero0 and zero1 (nz each), ones (no words
// set to -1)
struct ScanJob {
    const uint64_t *A, *B;
    int nA, nB;
    const int64_t *row_off;
    int64_t *row_cnt;
    PairList out;
    int64_t *zero0, *zero1, *ones;
    int nz, no;
};

// the symmetry-packed two-continuum integrals, for one relayout launch: record
// of the target pair (P, Q) at rec[P * n_o + Q]; inside it, the (tt|cc) rows
// of this launch start at boffJ (row length ncb), the (tc|tc) block of the
// second symmetry's irrep at boffK (row length nca_full, rows from column jr0)
struct PackedCC {
    const int64_t *rec;
    int64_t boffJ, boffK;
    int jr0, nca_full;
};

// the blocks of the two-continuum integrals that symmetry allows, for a pass over
// them: n[a] continuum orbitals of irrep a from start[a] on; packed layout: record
// of the pair (P, Q) at rec[P * n_o + Q], the block of rows of irrep a at blk[x][a]
// of it where the target orbitals' irreps differ by x; dense layout: rec = nullptr
struct CcBlocks {
    const int64_t *rec;
    int64_t blk[8][8];
    int32_t n[8], start[8];
    uint8_t irrep[32 * CCH_MAXW];
    int n_irrep, n_o, n_cont;
};

// the slots (or pairs of slots) a density launch forms, and how it lays the
// rows out for the expansion product (k_target.hip); k1 = nullptr: slot t
enum GammaMode { GAM_PLAIN = 0, GAM_RECT = 1, GAM_SQUARE = 2 };
struct GammaList {
    int mode, n;
    const int32_t *k1, *k2;
};

// the target-space sums of one symmetry pair (k_target.hip): every kernel of a
// build takes all pairs in one launch, pair blockIdx.y of a table on the device
struct PairJob {
    const uint64_t *da, *db;     // determinants of the two symmetries
    const int8_t *spa, *spb;     // continuum spins per determinant or nullptr
    const double *ca, *cb;       // [Ma][Sa], [Mb][Sb]
    int Ma, Sa, Sb, tri, nrows;  // tri: a symmetry with itself, states n' <= n
    int M0;                      // Ma if the symmetries share an irrep, else 0
    int64_t n;                   // connected pairs
    const int64_t *row_off, *row_cnt;
    PairList pl;
    double *hv, *Y, *Yo, *HT, *O;
    const int32_t *rn, *rn2, *pqidx, *slotP, *slotQ;
    int n_slot;
    int32_t *key;
    int64_t *count, *start, *cursor, *sorted, *tmp, *d0;
    GammaList gl;
    double *At;
};

// the power of two that the Householder tridiagonalisation takes out of a matrix
// whose largest |entry| has the bits amax: none for entries between 2^-96 and 2^97
// or a non-finite matrix, else the one that brings the largest entry to [1, 2)
// (subnormal ones: to 2^-51 or more)
__host__ __device__ inline int trd_shift(unsigned long long amax)
{
    const int ex = (int)(amax >> 52);
    const bool fits = (ex >= 1023 - 96 && ex <= 1023 + 96) || ex == 2047 || amax == 0;
    return fits ? 0 : ex - 1023;
}

// work vectors of the Householder tridiagonalisation (length n each): x = the
// current column after the panel's corrections times a power of two (two
// buffers, by column parity), y = A_0 x as the row pass leaves it; the diagonal
// d, the off-diagonal e and the reflector scalars tau of T; amax: the largest
// |entry| of the matrix before trd_shift (its bits). x0, x1: 16-byte aligned
struct TrdVec {
    double *x0, *x1, *y;
    double *d, *e, *tau;
    unsigned long long *amax;
};

// columns per panel of the blocked tridiagonalisation
constexpr int TRD_NB = 32;
// rows per workgroup of the column kernel, and the stride of its partial sums
constexpr int TRD_CR = 128, TRD_PS = 2 * TRD_NB + 8;
constexpr int TRD_PT = 2 * TRD_NB;   // doubles per row of PVt
// trailing blocks of at least TRD_TILE_MIN rows are multiplied from their
// lower triangle in TRD_TT x TRD_TT tiles (below that the row pass reads
// whole rows)
constexpr int TRD_TT = 128, TRD_TILE_MIN = 3072;
struct TrdPanel {
    double *PV, *PW;   // 2 TRD_NB rows each, ldp doubles a row (the panel update's operands)
    int64_t ldp;
    double *PVt;       // PV by matrix row: PVt[r][d] = PV[d][r], 2 TRD_NB doubles a row
    double *part1;     // column kernel: TRD_PS partial sums per workgroup (two buffers, by column parity)
    int64_t part1_len; // doubles of one of them
    double *part2;     // product: one partial sum of x . A_0 x per workgroup
    double *rowp, *colp;   // tiled product: [tile column][n] row sums, [tile row][n] column sums
};

// first row of the tiles of the trailing block that starts at row r
__host__ __device__ inline int trd_base(int r) { return r & ~15; }
// tiles per side over m rows
__host__ __device__ inline int trd_tiles(int m) { return (m + TRD_TT - 1) / TRD_TT; }

// the panel buffers for dimension n with rows of ldp doubles, carved from one
// allocation (base = nullptr: only the size in doubles is wanted)
inline size_t trd_panel_layout(int n, int64_t ldp, double *base, TrdPanel *P)
{
    const size_t T = (size_t)trd_tiles(n);
    size_t at = 0;
    auto take = [&](size_t len) {
        double *p = base ? base + at : nullptr;
        at += (len + 3) / 4 * 4;
        return p;
    };
    P->ldp = ldp;
    P->PVt = take((size_t)TRD_PT * n);
    P->PV = take((size_t)2 * TRD_NB * ldp);
    P->PW = take((size_t)2 * TRD_NB * ldp);
    P->part1_len = (int64_t)((n + TRD_CR - 1) / TRD_CR) * TRD_PS;
    P->part1 = take(2 * (size_t)P->part1_len);
    const size_t tiles = T * (T + 1) / 2, rows = (size_t)(n + 3) / 4;
    P->part2 = take(tiles > rows ? tiles : rows);
    P->rowp = take(T * (size_t)n);
    P->colp = take(T * (size_t)n);
    return at;
}

// class 4 of one target symmetry (k_class4.hip)
struct Class4Args {
    const uint64_t *tdets;   // target dets of the symmetry [M][W]
    const int8_t *cspin;     // continuum spin per target det (0 alpha, 1 beta); nullptr: alpha
    const double *ci;        // [M][S]
    int S;
    const double *h;         // [n_orb][n_orb]
    const double *tttc;      // [n_o][n_o][n_o][n_cont]
    int n_o, n_orb, n_cont;
    int ja0, nc;             // continuum range of the symmetry
    const int64_t *row_off, *row_cnt;   // L2 x target pairs per L2 row
    PairList pl;
    double *H;
    int64_t ld;
    int64_t row_l2;          // first L2 row of the matrix
    int64_t col0;            // first column of the symmetry block
    int W;                   // words per determinant
};

constexpr int CCH_MAX_WORDS = 4;   // words per determinant at most

// passes over the states of nq quads each, blocks of bt tiles of 16 orbitals,
// lpw L2 functions a workgroup
struct C4Split {
    int passes, nq, blocks, bt, lpw;
};

// one (instance, symmetry) block of the persistent class-4 launch
struct C4Task {
    Class4Args a;
    int n_l2;
    int64_t first;   // first global work item of this block
};

// where the expansion product's results go, and what is added to them
struct ExpandEpi {
    double *H;            // contracted matrix, row-major
    int64_t ld;
    int64_t row0a, row0b; // first row of symmetry a / b
    int nca, ncb;         // continuum orbitals of a / b
    int ja0, jb0;         // first global continuum index of a / b
    const int32_t *rn, *rn2;
    const double *HT, *O; // per GEMM row
    const double *h;      // one-electron matrix [n_orb][n_orb]
    int n_o, n_orb;
};

// one product: rect, N = (rows j of the pass) x ncb columns, KA = 0; or square,
// columns j >= j' of j0 <= j < j1
struct ExpandOp {
    const double *At, *B;
    int nrows, KS, KA;
    int sq, j0, j1;
    int N;                // columns of B (the leading dimension)
    ExpandEpi ep;
};

// one product of a persistent launch (k_gemm.hip): tiles [first, first + tiles_m *
// tiles_n) of the list, `height` rows each
struct GemmTask {
    ExpandOp op;
    int height, tiles_m, tiles_n;
    int64_t first;
};

// the dense L2 block, classes 2 and 8 (k_l2.hip)
struct L2Args {
    const uint64_t *dets;   // [n_l2][W]
    int n_l2;
    TgtInts I;
    double *H;
    int64_t ld;
    int64_t row0;           // first L2 row / column of the matrix
    int both;               // write the upper triangle as well
};

struct L2Task {   // one instance of a persistent launch
    L2Args a;
    int64_t first;   // first global tile of this instance
};

// a matrix whose L2 block (classes 2 and 8) is held as CSR: P[r][c] for
// c < Dc (every row), R[r][c - Dc] for r < Dc <= c, and the L2 block's rows
// as CSR (columns relative to Dc, ascending)
struct SparseMat {
    const double *P;
    int64_t ldp;
    const double *R;
    int64_t ldr;
    const int64_t *off;
    const int32_t *col;
    const double *val;
    int64_t Dc;
};

}  // namespace cch

// ---------------------------------------------------------------------------
// kernel launchers (host side, defined in the .hip files)
// ---------------------------------------------------------------------------
namespace cch {
// the Ritz pairs whose corrections a Davidson step forms (output c uses pair
// e[c]), passed to the kernels by value
struct DavSel {
    int32_t e[32];
};

// device memory that is no context's work space; idle work space on the device
// makes room for it
__attribute__((visibility("hidden"))) hipError_t dev_malloc(int device, void **p, size_t bytes);
hipError_t launch_scan(int mode, int W, const ScanJob &one, int top, hipStream_t st);
hipError_t launch_scans(int mode, int W, const ScanJob *jobs, int njob, int max_rows, int top, hipStream_t st);
hipError_t launch_exclusive_scan(const int64_t *in, int64_t *out, int n, int64_t *total,
                                 hipStream_t st);
hipError_t launch_symv(const double *H, int64_t ld, int D, int C, const double *V, int64_t ldv, int b, double *W,
                       int64_t ldw, double *Wp, hipStream_t st);
int64_t symv_scratch_doubles(int D, int C);
hipError_t launch_fill_i64(int64_t *p, int64_t v, int64_t n, hipStream_t st);
hipError_t launch_fill_f64(double *p, double v, int64_t n, hipStream_t st);
}  // namespace cch
