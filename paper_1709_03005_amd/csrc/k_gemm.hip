// Expansion of the contracted symbols over the continuum pairs (j, j')
// (Sec. 2.1, end; Sec. 3.1 "expansion"): the integral labels of a
// contracted element keep their target part (P, Q) while (j, j') runs over
// the continuum orbitals of the two symmetries. Written as one dense product
// per target-symmetry pair:
//   Ht[(n,n'), (j,j')] = sum_{PQ} Gamma_{nn',PQ} (PQ|jj')
//                      - sum_{PQ} Gamma^alpha_{nn',PQ} (Pj'|jQ)
//                      + delta_{jj'} (C^T H_T C')_{nn'} + (C^T O C')_{nn'} h_{jj'}
// K0 lays the integral rows out as B[k][(j,j')]; K5 multiplies with FP64
// MFMA (v_mfma_f64_4x4x4) and scatters each (n,n',j,j') to its row
// (i,n,j) / column (i',n',j') of the contracted matrix (lower triangle).
//
// The FP64 product multiplies each distinct integral once, by the
// permutational symmetry of real orbitals, (PQ|jj') = (QP|jj') = (PQ|j'j) and
// (Pj'|jQ) = (Qj|j'P):
//   * the Coulomb rows hold one (P, Q) of each pair P >= Q, with
//     Gamma_PQ + Gamma_QP;
//   * between two symmetries coupled to one continuum range (the "square"
//     form) the exchange sum over {PQ, QP} splits into a part symmetric in
//     j, j' (the mean of the two densities times the sum of the two integrals)
//     and an antisymmetric one (half the difference times the difference), so
//     only j >= j' is multiplied: H(j,j') = S + A, H(j',j) = S - A.
// The square form takes 3/4 of the rows and half the columns of the plain
// product (0.38 of its flops; 2420 rows x 80200 columns instead of 3200 x
// 160000 at 40 target and 400 continuum orbitals), the other pairs ("rect")
// 3/4 of the rows. The reduced-precision forms keep the plain layout, and so does
// the FP64 product of integrals given without those symmetries (launch_cc_sym).
#include <algorithm>

#include "ccham_internal.h"

namespace cch {

// ---------------------------------------------------------------------------
// Do the two-continuum integrals have the symmetries that the folded product
// reads one value for, (PQ|jj') = (QP|jj') = (PQ|j'j) and (Pj|Qj') = (Qj'|Pj)?
// Values that differ by more than 2^-49 of the larger (what the factors of a
// transformation leave when multiplied in another order), or are not finite, set
// *flag; the expansion then reads every value as given. A workgroup takes a pair
// P >= Q and the tiles (j, j') and (j', j) of the blocks of the irreps (a, b) and
// (b, a) that symmetry allows, the values that a build reads. Once per plan, bound
// by reading them.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool cc_differ(double a, double b)
{
    return !(fabs(a - b) <= 0x1p-49 * fmax(fabs(a), fabs(b)));
}

__global__ __launch_bounds__(256) void k_cc_sym(CcBlocks B, const double *__restrict__ ttcc,
                                                const double *__restrict__ tctc, int32_t *__restrict__ flag)
{
    __shared__ double tb[32][33], tf[32][33], te[32][33];
    int P = (int)((sqrt(8.0 * blockIdx.z + 1.0) - 1.0) * 0.5);
    while ((P + 1) * (P + 2) / 2 <= (int)blockIdx.z) ++P;
    while (P * (P + 1) / 2 > (int)blockIdx.z) --P;
    const int Q = (int)blockIdx.z - P * (P + 1) / 2;
    const int r0 = blockIdx.x * 32, c0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int x = B.irrep[P] ^ B.irrep[Q];
    // (P Q | j j') and (P j | Q j'), j of irrep a, j' of irrep a ^ x
    auto coul = [&](int p, int q, int a) -> const double * {
        if (B.rec) return ttcc + B.rec[(size_t)p * B.n_o + q] + B.blk[x][a];
        return ttcc + (((int64_t)p * B.n_o + q) * B.n_cont + B.start[a]) * B.n_cont + B.start[a ^ x];
    };
    auto exch = [&](int p, int q, int a) -> const double * {
        if (B.rec) return tctc + B.rec[(size_t)p * B.n_o + q] + B.blk[x][a];
        return tctc + (((int64_t)p * B.n_cont + B.start[a]) * B.n_o + q) * B.n_cont + B.start[a ^ x];
    };
    bool bad = false;
    for (int a = 0; a < B.n_irrep; ++a) {
        const int b = a ^ x, na = B.n[a], nb = B.n[b];
        if (b < a || (b == a && c0 > r0) || r0 >= na || c0 >= nb) continue;   // (the whole workgroup)
        const int64_t lc = B.rec ? nb : B.n_cont, lct = B.rec ? na : B.n_cont;   // row lengths of the two blocks
        const int64_t le = B.rec ? nb : (int64_t)B.n_o * B.n_cont, let = B.rec ? na : le;
        const double *A1 = coul(P, Q, a), *A2 = coul(P, Q, b), *C1 = coul(Q, P, a), *C2 = coul(Q, P, b);
        const double *E1 = exch(P, Q, a), *E2 = exch(P, Q, b), *F1 = exch(Q, P, b), *F2 = exch(Q, P, a);
        __syncthreads();
        for (int r = ty; r < 32; r += 8) {   // row c0 + r, column r0 + tx of the blocks (b, a)
            const int j = c0 + r, k = r0 + tx;
            const bool in = j < nb && k < na;
            const int64_t oc = j * lct + k, oe = j * let + k;
            tb[r][tx] = in ? A2[oc] : 0.0;
            tf[r][tx] = in ? F1[oe] : 0.0;
            te[r][tx] = in ? E2[oe] : 0.0;
            if (in) bad |= cc_differ(tb[r][tx], C2[oc]);
        }
        __syncthreads();
        for (int r = ty; r < 32; r += 8) {   // row r0 + r, column c0 + tx of the blocks (a, b)
            const int j = r0 + r, k = c0 + tx;
            if (j >= na || k >= nb) continue;
            const double v = A1[j * lc + k];
            bad |= cc_differ(v, C1[j * lc + k]) || cc_differ(v, tb[tx][r]);
            bad |= cc_differ(E1[j * le + k], tf[tx][r]) || cc_differ(F2[j * le + k], te[tx][r]);
        }
    }
    if (__any(bad) && (threadIdx.x & 63) == 0) *flag = 1;
}

__global__ void k_flag_zero(int32_t *__restrict__ flag) { *flag = 0; }

// *flag = 1 if the integrals lack a symmetry, else 0
hipError_t launch_cc_sym(const CcBlocks &B, const double *ttcc, const double *tctc, int32_t *flag, hipStream_t st)
{
    hipLaunchKernelGGL(k_flag_zero, dim3(1), dim3(1), 0, st, flag);
    int most = 0;
    for (int a = 0; a < B.n_irrep; ++a) most = std::max(most, B.n[a]);
    const int T = (most + 31) / 32;
    if (T > 0)
        hipLaunchKernelGGL(k_cc_sym, dim3(T, T, B.n_o * (B.n_o + 1) / 2), dim3(256), 0, st, B, ttcc, tctc, flag);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// K0: B[k][jj*ncb + jj'] for one symmetry pair (plain and rect forms).
//   k <  nJ: (P Q | J J')    = ttcc[P][Q][J][J']       (row copy)
//   k >= nJ: -(P J' | J Q)   = -tctc[P][J'][Q][J]     (tile transpose)
// over two lists of (P, Q): every slot in both (plain), or the pairs P > Q in
// the first and P Q, Q P alternating in the second (rect).
// ---------------------------------------------------------------------------
// B[k][jj][jj'] = (P Q | ja0+jj, jb0+jj'): the slab of slot k is one contiguous
// nca x ncb block of B, gathered from nca rows of ttcc; a workgroup copies
// RJ_PER consecutive elements of a slab (all its loads issued before its stores)
constexpr int RJ_U = 4, RJ_PER = 256 * RJ_U;

__global__ __launch_bounds__(256) void k_relayout_J(const double *__restrict__ ttcc, int n_o, int n_cont,
                                                    const int32_t *__restrict__ slotP,
                                                    const int32_t *__restrict__ slotQ, int ja0, int nca,
                                                    int jb0, int ncb, double *__restrict__ B)
{
    const int k = blockIdx.y;
    const int P = slotP[k], Q = slotQ[k];
    const double *src = ttcc + ((size_t)P * n_o + Q) * n_cont * n_cont + (size_t)ja0 * n_cont + jb0;
    double *dst = B + (size_t)k * nca * ncb;
    const int64_t slab = (int64_t)nca * ncb, e0 = (int64_t)blockIdx.x * RJ_PER + threadIdx.x;
    double v[RJ_U];
#pragma unroll
    for (int u = 0; u < RJ_U; ++u) {
        const int64_t e = e0 + 256 * u;
        v[u] = e < slab ? src[(e / ncb) * n_cont + e % ncb] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < RJ_U; ++u) {
        const int64_t e = e0 + 256 * u;
        if (e < slab) dst[e] = v[u];
    }
}

__global__ __launch_bounds__(256) void k_relayout_K(const double *__restrict__ tctc, int n_o, int n_cont,
                                                    const int32_t *__restrict__ slotP,
                                                    const int32_t *__restrict__ slotQ, int n_slot, int ja0,
                                                    int nca, int jb0, int ncb, double *__restrict__ B)
{
    __shared__ double tile[32][33];
    const int k = blockIdx.z;
    const int P = slotP[k], Q = slotQ[k];
    const int jj0 = blockIdx.x * 32, jp0 = blockIdx.y * 32;   // jj (unprimed) / jj' tiles
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;    // 32 x 8
    // read tctc[P][J'][Q][J]: contiguous in J
    for (int r = ty; r < 32; r += 8) {
        const int jp = jp0 + r, jj = jj0 + tx;
        double v = 0.0;
        if (jp < ncb && jj < nca)
            v = tctc[(((size_t)P * n_cont + (jb0 + jp)) * n_o + Q) * n_cont + (ja0 + jj)];
        tile[r][tx] = v;
    }
    __syncthreads();
    // write B[n_slot + k][jj][jj']: contiguous in jj'
    double *dst = B + (size_t)(n_slot + k) * nca * ncb;
    for (int r = ty; r < 32; r += 8) {
        const int jj = jj0 + r, jp = jp0 + tx;
        if (jj < nca && jp < ncb) dst[(size_t)jj * ncb + jp] = -tile[tx][r];
    }
}

// the same rows from the symmetry-packed layout: one record per target pair,
// the (tt|cc) rows of this launch contiguous (row length ncb), the (tc|tc)
// block read row by row over j and turned through LDS
__global__ __launch_bounds__(256) void k_relayout_Jp(const double *__restrict__ ttcc, PackedCC pk, int n_o,
                                                     const int32_t *__restrict__ slotP,
                                                     const int32_t *__restrict__ slotQ, int nca, int ncb,
                                                     double *__restrict__ B)
{
    const int k = blockIdx.y;
    const double *src = ttcc + pk.rec[(size_t)slotP[k] * n_o + slotQ[k]] + pk.boffJ;
    double *dst = B + (size_t)k * nca * ncb;
    const int64_t slab = (int64_t)nca * ncb, e0 = (int64_t)blockIdx.x * RJ_PER + threadIdx.x;
    double v[RJ_U];
#pragma unroll
    for (int u = 0; u < RJ_U; ++u) {
        const int64_t e = e0 + 256 * u;
        v[u] = e < slab ? src[e] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < RJ_U; ++u) {
        const int64_t e = e0 + 256 * u;
        if (e < slab) dst[e] = v[u];
    }
}

__global__ __launch_bounds__(256) void k_relayout_Kp(const double *__restrict__ tctc, PackedCC pk, int n_o,
                                                     const int32_t *__restrict__ slotP,
                                                     const int32_t *__restrict__ slotQ, int n_slot, int nca,
                                                     int ncb, double *__restrict__ B)
{
    __shared__ double tile[32][33];
    const int k = blockIdx.z;
    const double *src = tctc + pk.rec[(size_t)slotP[k] * n_o + slotQ[k]] + pk.boffK;
    const int jj0 = blockIdx.x * 32, jp0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    // (P j' | Q j): row j' of the block, contiguous in j
    for (int r = ty; r < 32; r += 8) {
        const int jp = jp0 + r, jj = jj0 + tx;
        tile[r][tx] = (jp < ncb && jj < nca) ? src[(int64_t)jp * pk.nca_full + pk.jr0 + jj] : 0.0;
    }
    __syncthreads();
    double *dst = B + (size_t)(n_slot + k) * nca * ncb;
    for (int r = ty; r < 32; r += 8) {
        const int jj = jj0 + r, jp = jp0 + tx;
        if (jj < nca && jp < ncb) dst[(size_t)jj * ncb + jp] = -tile[tx][r];
    }
}

hipError_t launch_relayout(const double *ttcc, const double *tctc, int n_o, int n_cont, const int32_t *slotPJ,
                           const int32_t *slotQJ, int nJ, const int32_t *slotPK, const int32_t *slotQK, int nK,
                           int ja0, int nca, int jb0, int ncb, double *B, hipStream_t st, const PackedCC *pk)
{
    if (nK <= 0 || nca <= 0 || ncb <= 0) return hipSuccess;
    const dim3 gJ((int)(((int64_t)nca * ncb + RJ_PER - 1) / RJ_PER), nJ), gK((nca + 31) / 32, (ncb + 31) / 32, nK);
    if (pk) {
        hipLaunchKernelGGL(k_relayout_Jp, gJ, dim3(256), 0, st, ttcc, *pk, n_o, slotPJ, slotQJ, nca, ncb, B);
        hipLaunchKernelGGL(k_relayout_Kp, gK, dim3(256), 0, st, tctc, *pk, n_o, slotPK, slotQK, nJ, nca, ncb, B);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_relayout_J, gJ, dim3(256), 0, st, ttcc, n_o, n_cont, slotPJ, slotQJ, ja0, nca, jb0, ncb, B);
    hipLaunchKernelGGL(k_relayout_K, gK, dim3(256), 0, st, tctc, n_o, n_cont, slotPK, slotQK, nJ, ja0, nca, jb0, ncb,
                       B);
    return hipGetLastError();
}

// K0 of the square form: rows of the pairs P >= Q (the nF - n_off diagonal ones
// last), columns j >= j' packed by rows j, j0 <= j < j1:
//   B[t][tri(j) - tri(j0) + j']           = (P Q | j j')
//   B[nF + t]                             = (P j'|Q j) + (P j|Q j')   (once for P = Q)
//   B[2 nF + t], t < n_off                = (P j'|Q j) - (P j|Q j')
// One launch: blockIdx.z < nF copies (tt|cc) rows, a wave per row j; the rest
// read the pair of 32 x 32 tiles of (P x|Q y) that mirror each other. Bound by
// HBM: every value of a pair P > Q is read once and 12 bytes move per plain
// element instead of 32.
__host__ __device__ __forceinline__ int64_t tri64(int64_t j) { return j * (j + 1) / 2; }

template <bool PACKED>
__global__ __launch_bounds__(256) void k_relayout_sq(const double *__restrict__ ttcc, const double *__restrict__ tctc,
                                                     PackedCC pk, int n_o, int n_cont,
                                                     const int32_t *__restrict__ fP, const int32_t *__restrict__ fQ,
                                                     int nF, int n_off, int ja0, int nc, int j0, int j1,
                                                     double *__restrict__ B)
{
    __shared__ double ta[32][33], tb[32][33];
    const int64_t ldb = tri64(j1) - tri64(j0);
    const int jt = j0 + blockIdx.x * 32, pt = blockIdx.y * 32;
    if (pt > min(jt + 31, j1 - 1)) return;   // no j' <= j in this tile (the whole workgroup)
    const bool coul = (int)blockIdx.z < nF;
    const int t = coul ? blockIdx.z : blockIdx.z - nF;
    const int P = fP[t], Q = fQ[t];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;    // 32 x 8
    if (coul) {
        const double *src = PACKED ? ttcc + pk.rec[(size_t)P * n_o + Q] + pk.boffJ
                                   : ttcc + ((size_t)P * n_o + Q) * n_cont * n_cont + (size_t)ja0 * n_cont + ja0;
        const int64_t ls = PACKED ? nc : n_cont;
        double *dst = B + t * ldb - tri64(j0);
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = jt + ty + 8 * u, jp = pt + tx;
            v[u] = (j < j1 && jp <= j) ? src[j * ls + jp] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = jt + ty + 8 * u, jp = pt + tx;
            if (j < j1 && jp <= j) dst[tri64(j) + jp] = v[u];
        }
        return;
    }
    // T[x][y] = (P x | Q y)
    const double *src = PACKED ? tctc + pk.rec[(size_t)P * n_o + Q] + pk.boffK
                               : tctc + (((size_t)P * n_cont + ja0) * n_o + Q) * n_cont + ja0;
    const int64_t ls = PACKED ? nc : (int64_t)n_o * n_cont;
    for (int r = ty; r < 32; r += 8) {
        ta[r][tx] = (jt + r < j1 && pt + tx < nc) ? src[(jt + r) * ls + pt + tx] : 0.0;
        tb[r][tx] = (pt + r < nc && jt + tx < j1) ? src[(pt + r) * ls + jt + tx] : 0.0;
    }
    __syncthreads();
    double *dp = B + (nF + t) * ldb - tri64(j0), *dm = B + (2 * (int64_t)nF + t) * ldb - tri64(j0);
    for (int r = ty; r < 32; r += 8) {
        const int j = jt + r, jp = pt + tx;
        if (j >= j1 || jp > j) continue;
        const double x = tb[tx][r], y = ta[r][tx];   // T[j'][j], T[j][j']
        if (t < n_off) {
            dp[tri64(j) + jp] = x + y;
            dm[tri64(j) + jp] = x - y;
        } else {
            dp[tri64(j) + jp] = x;
        }
    }
}

hipError_t launch_relayout_sq(const double *ttcc, const double *tctc, int n_o, int n_cont, const int32_t *fP,
                              const int32_t *fQ, int nF, int n_off, int ja0, int nc, int j0, int j1, double *B,
                              hipStream_t st, const PackedCC *pk)
{
    if (nF <= 0 || j1 <= j0) return hipSuccess;
    const dim3 g((j1 - j0 + 31) / 32, (j1 + 31) / 32, 2 * nF);
    if (pk)
        hipLaunchKernelGGL(k_relayout_sq<true>, g, dim3(256), 0, st, ttcc, tctc, *pk, n_o, n_cont, fP, fQ, nF, n_off,
                           ja0, nc, j0, j1, B);
    else
        hipLaunchKernelGGL(k_relayout_sq<false>, g, dim3(256), 0, st, ttcc, tctc, PackedCC{}, n_o, n_cont, fP, fQ, nF,
                           n_off, ja0, nc, j0, j1, B);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// K5: C = A * B with A given K-major (At[k][r]), FP64 MFMA 4x4x4 (four
// blocks). Workgroup tile BM (r) x 128 (col), 4 waves; each wave has up to 32
// rows x (128 / waves along the columns) = 8 x NT instructions of 4 rows x 16
// columns. K staged through LDS in slices of 16. Operand layout of the
// four-block 4x4x4 f64 MFMA (lane l = j + 4 blk + 16 i, checked on gfx950):
// A[blk][i][k] at lane i + 4 blk + 16 k, B[blk][k][j] at lane j + 4 blk + 16 k,
// D[blk][i][j] at lane j + 4 blk + 16 i. With the same A slab in every block,
// an instruction multiplies 4 rows by 16 columns (B's column 4 blk + j); on
// this chip it issues faster per flop than the 16x16x4 form.
//
// Square form: a tile's 128 columns are 8 values of j x 16 of j' (so a wave's
// 16 lanes write 128 contiguous bytes of a row, and the mirrored elements of
// its values of j lie side by side in theirs); the rows of the symmetric part
// (k < KS) and of the antisymmetric one (KS <= k < KS + KA) go to two sets of
// accumulators.
// ---------------------------------------------------------------------------

constexpr int GBN = 128, GBK = 16, GBJ = 8;

__device__ __forceinline__ int xcd_remap(int b, int nb)
{
    // consecutive logical tiles land on one XCD (blocks are dealt round-robin
    // over the 8 XCDs), so tiles sharing a B column panel share an L2
    const int per = nb / 8;
    if (b >= per * 8) return b;
    return (b % 8) * per + b / 8;
}

// square form: column tiles of the eight rows j from jt on (16 j' each)
__host__ __device__ __forceinline__ int sq_tiles(int jt, int j1)
{
    return ((jt + GBJ < j1 ? jt + GBJ : j1) - 1) / 16 + 1;
}

template <int BM, bool SQ>
__device__ __forceinline__ void expand_tile_f64(const ExpandOp &op, int tm, int tn, double (*As)[BM],
                                                double (*Bs)[GBN])
{
    constexpr int WAVES_M = BM >= 64 ? 2 : 1, WAVES_N = 4 / WAVES_M;
    constexpr int MA = BM / WAVES_M / 4;                    // 4-row steps per wave
    constexpr int WCOLS = GBN / WAVES_N, NT = WCOLS / 16;   // MFMA tiles along N per wave
    constexpr int AQ = BM * GBK / 256, BQ = GBN * GBK / 256;
    const double *__restrict__ At = op.At;
    const int nrows = op.nrows;
    const int64_t ldb = op.N;
    const ExpandEpi &ep = op.ep;
    const int r0 = tm * BM, c0 = tn * GBN;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int wm = wv % WAVES_M, wn = wv / WAVES_M;
    // the column of B that this thread stages
    const int cc = threadIdx.x & (GBN - 1), kc = threadIdx.x / GBN;
    int jt = 0, jp0 = 0;
    bool cok;
    int64_t coff;
    if (SQ) {
        jt = op.j0;
        for (int left = tn;;) {
            const int n = sq_tiles(jt, op.j1);
            if (left < n) {
                jp0 = 16 * left;
                break;
            }
            left -= n;
            jt += GBJ;
        }
        const int j = jt + (cc >> 4), jp = jp0 + (cc & 15);
        cok = j < op.j1 && jp <= j;
        coff = tri64(j) - tri64(op.j0) + jp;
    } else {
        cok = c0 + cc < op.N;
        coff = c0 + cc;
    }
    const double *__restrict__ Bc = op.B + (cok ? coff : 0);

    // 4x4x4 FP64 MFMA (four blocks sharing the A slab): one instruction is 4
    // rows x 16 columns x 4 k; lane l holds row 4 m + (l >> 4), column 16 n +
    // (l & 15) of the wave's tile
    double acc[MA][NT], acca[SQ ? MA : 1][SQ ? NT : 1];
    double ra[AQ], rb[BQ];
    auto gload = [&](int k0, int ke) {
#pragma unroll
        for (int q = 0; q < AQ; ++q) {
            const int e = threadIdx.x + 256 * q;
            const int k = k0 + e / BM, r = r0 + e % BM;
            ra[q] = (k < ke && r < nrows) ? At[(size_t)k * nrows + r] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < BQ; ++q) {
            const int k = k0 + kc + 2 * q;
            rb[q] = (k < ke && cok) ? Bc[(int64_t)k * ldb] : 0.0;
        }
    };
    auto product = [&](int kb, int ke, auto &ac) {
#pragma unroll
        for (int a = 0; a < MA; ++a)
#pragma unroll
            for (int b = 0; b < NT; ++b) ac[a][b] = 0.0;
        if (kb >= ke) return;
        gload(kb, ke);
        for (int k0 = kb; k0 < ke; k0 += GBK) {
            __syncthreads();
#pragma unroll
            for (int q = 0; q < AQ; ++q) {
                const int e = threadIdx.x + 256 * q;
                As[e / BM][e % BM] = ra[q];
            }
#pragma unroll
            for (int q = 0; q < BQ; ++q) Bs[kc + 2 * q][cc] = rb[q];
            __syncthreads();
            if (k0 + GBK < ke) gload(k0 + GBK, ke);
#pragma unroll
            for (int ks = 0; ks < GBK; ks += 4) {
                const int kk = ks + (lane >> 4);
                double bf[NT];
#pragma unroll
                for (int b = 0; b < NT; ++b) bf[b] = Bs[kk][wn * WCOLS + b * 16 + (lane & 15)];
#pragma unroll
                for (int a = 0; a < MA; ++a) {
                    const double af = As[kk][wm * 32 + 4 * a + (lane & 3)];
#pragma unroll
                    for (int b = 0; b < NT; ++b)
                        ac[a][b] = __builtin_amdgcn_mfma_f64_4x4x4f64(af, bf[b], ac[a][b], 0, 0, 0);
                }
            }
        }
    };
    product(0, op.KS, acc);
    if constexpr (SQ) product(op.KS, op.KS + op.KA, acca);
    __syncthreads();   // the LDS tiles are reused by the next tile of a persistent loop

    // epilogue: scatter into the contracted matrix (lower triangle only)
#pragma unroll
    for (int a = 0; a < MA; ++a) {
        const int r = r0 + wm * 32 + 4 * a + (lane >> 4);
        if (r >= nrows) continue;
        const int n = ep.rn[r], n2 = ep.rn2[r];
        const double ht = ep.HT[r], ov = ep.O[r];
#pragma unroll
        for (int b = 0; b < NT; ++b) {
            int jj, jp;
            if (SQ) {
                jj = jt + wn * NT + b;
                jp = jp0 + (lane & 15);
                if (jj >= op.j1 || jp > jj) continue;
            } else {
                const int c = c0 + wn * WCOLS + b * 16 + (lane & 15);
                if (c >= op.N) continue;
                jj = c / ep.ncb;
                jp = c - jj * ep.ncb;
            }
            const int J = ep.ja0 + jj, Jp = ep.jb0 + jp;
            const int64_t R = ep.row0a + (int64_t)n * ep.nca + jj;
            const int64_t C = ep.row0b + (int64_t)n2 * ep.ncb + jp;
            if (R >= C) {
                double val = acc[a][b];
                if constexpr (SQ) val += acca[a][b];
                if (J == Jp) val += ht;
                val += ov * ep.h[(size_t)(ep.n_o + J) * ep.n_orb + (ep.n_o + Jp)];
                ep.H[R * ep.ld + C] = val;
            }
            if constexpr (SQ) {
                const int64_t R2 = ep.row0a + (int64_t)n * ep.nca + jp;
                const int64_t C2 = ep.row0b + (int64_t)n2 * ep.ncb + jj;
                if (jp < jj && R2 >= C2) {
                    double val = acc[a][b] - acca[a][b];
                    val += ov * ep.h[(size_t)(ep.n_o + Jp) * ep.n_orb + (ep.n_o + J)];
                    ep.H[R2 * ep.ld + C2] = val;
                }
            }
        }
    }
}

template <int BM, bool SQ>
__global__ __launch_bounds__(256) void k_expand_f64(ExpandOp op, int tiles_m, int tiles)
{
    __shared__ double As[GBK][BM];
    __shared__ double Bs[GBK][GBN];
    const int lb = xcd_remap(blockIdx.x, tiles);
    expand_tile_f64<BM, SQ>(op, lb % tiles_m, lb / tiles_m, As, Bs);
}

// column tiles of a product
int expand_cols(const ExpandOp &op)
{
    if (!op.sq) return (op.N + GBN - 1) / GBN;
    int n = 0;
    for (int jt = op.j0; jt < op.j1; jt += GBJ) n += sq_tiles(jt, op.j1);
    return n;
}

// tile height: 64 rows unless that pads the rows by a quarter more than lower
// tiles would (15 rows of five states take a 16-row tile, 25 a 32-row one) or
// leaves the 256 compute units without two workgroups each. Every height gives
// the same bits (each element is one sum over k in order).
static int expand_height(int nrows, int cols)
{
    if (nrows <= 16) return 16;
    const int p64 = (nrows + 63) / 64 * 64, p32 = (nrows + 31) / 32 * 32;
    return (4 * p64 > 5 * p32 || (p64 / 64) * cols < 512) ? 32 : 64;
}

template <int BM>
static void expand_launch(const ExpandOp &op, int cols, hipStream_t st)
{
    const int tm = (op.nrows + BM - 1) / BM;
    if (op.sq) hipLaunchKernelGGL((k_expand_f64<BM, true>), dim3(tm * cols), dim3(256), 0, st, op, tm, tm * cols);
    else hipLaunchKernelGGL((k_expand_f64<BM, false>), dim3(tm * cols), dim3(256), 0, st, op, tm, tm * cols);
}

hipError_t launch_expand_f64(const ExpandOp &op, hipStream_t st)
{
    if (op.nrows <= 0 || op.N <= 0) return hipSuccess;
    const int cols = expand_cols(op);
    switch (expand_height(op.nrows, cols)) {
    case 16: expand_launch<16>(op, cols, st); break;
    case 32: expand_launch<32>(op, cols, st); break;
    default: expand_launch<64>(op, cols, st); break;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Persistent form over many (instance, symmetry pair) products: a fixed grid
// walks the concatenated tile list (static round-robin); descriptor d owns
// tiles [first[d], first[d] + tiles_m * tiles_n), each of its own height (at most
// BM): with one height for all, fifteen rows of five states took a 32- or 64-row
// tile. Two waves a SIMD at BM = 64, where the compiler's own choice of registers
// left one. Sixteen instances of 500 to 6000 rows: the build 4.56 -> 4.45 ms.
// ---------------------------------------------------------------------------

// height of a task's tiles in the persistent form with tiles of at most bm rows:
// as many workgroups as the whole list has, so only the padding counts
int expand_task_height(int nrows, int bm)
{
    return std::min(bm, expand_height(nrows, 1 << 20));
}

template <int BM>
__global__ __launch_bounds__(256, 2) void k_expand_f64_batched(const GemmTask *__restrict__ tasks, int ntask,
                                                               int64_t total)
{
    __shared__ double As[GBK * BM];
    __shared__ double Bs[GBK][GBN];
    for (int64_t t = blockIdx.x; t < total; t += gridDim.x) {
        int lo = 0, hi = ntask - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (tasks[mid].first <= t) lo = mid;
            else hi = mid - 1;
        }
        const GemmTask &g = tasks[lo];
        const int64_t local = t - g.first;
        const int tm = (int)(local % g.tiles_m), tn = (int)(local / g.tiles_m);
        auto A16 = reinterpret_cast<double (*)[16]>(As);
        auto A32 = reinterpret_cast<double (*)[32]>(As);
        auto A64 = reinterpret_cast<double (*)[64]>(As);
        if (g.height == 16) {
            if (g.op.sq) expand_tile_f64<16, true>(g.op, tm, tn, A16, Bs);
            else expand_tile_f64<16, false>(g.op, tm, tn, A16, Bs);
        } else if (BM == 32 || g.height == 32) {
            if (g.op.sq) expand_tile_f64<32, true>(g.op, tm, tn, A32, Bs);
            else expand_tile_f64<32, false>(g.op, tm, tn, A32, Bs);
        } else {
            if (g.op.sq) expand_tile_f64<64, true>(g.op, tm, tn, A64, Bs);
            else expand_tile_f64<64, false>(g.op, tm, tn, A64, Bs);
        }
    }
}

hipError_t launch_expand_f64_batched(const GemmTask *tasks, int ntask, int64_t total, int bm, int grid,
                                     hipStream_t st)
{
    if (total <= 0) return hipSuccess;
    const unsigned g = (unsigned)std::min<int64_t>(total, grid);
    if (bm == 32)
        hipLaunchKernelGGL((k_expand_f64_batched<32>), dim3(g), dim3(256), 0, st, tasks, ntask, total);
    else
        hipLaunchKernelGGL((k_expand_f64_batched<64>), dim3(g), dim3(256), 0, st, tasks, ntask, total);
    return hipGetLastError();
}

}  // namespace cch
