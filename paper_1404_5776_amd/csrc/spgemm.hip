// Truncated block-sparse products C = P_C(alpha op(A) op(B)) on gfx950.
//
// Every matrix is stored in atom-pair blocks on a spatial cut-off pattern
// (Sec. II.A); a product keeps only the output blocks inside C's cut-off
// (Sec. V.A truncates S^-1 and S^-1 H, and every product of a step is
// truncated the same way).
//
// Symbolic phase (once per pattern triple): for output block (i, j) the k with
// op(A)_ik and op(B)_kj stored are the common entries of row i of A's pattern
// and row j of B's pattern (cut-off patterns are symmetric, so "k in row j"
// is "(k, j) kept").  One thread per output block merges the two ascending
// lists; a count pass sizes the triple list, a fill pass writes
// (block index of op(A)_ik, block index of op(B)_kj), ascending in k.
//
// Numeric phase: one 64-lane wave per output block accumulates its triples
// with the FP64 matrix cores (v_mfma_f64_16x16x4_f64): a b x b block (b <= 16)
// sits in one 16 x 16 tile and the contraction runs in steps of 4.  Complex
// operands are split into real and imaginary planes, so a complex block
// product is four real tile products (re*re, im*im, re*im, im*re) sharing the
// operand loads; a real operand skips the products it does not need.
#include <cstdlib>
#include <type_traits>

#include "internal.h"

namespace rtdm {

typedef double d4 __attribute__((ext_vector_type(4)));

// ----------------------------------------------------------------- symbolic

__global__ void k_sym_count(int64_t nout, const int32_t *__restrict__ c_rowof,
                            const int32_t *__restrict__ c_col, const int64_t *__restrict__ a_ptr,
                            const int32_t *__restrict__ a_col, const int64_t *__restrict__ b_ptr,
                            const int32_t *__restrict__ b_col, int64_t *__restrict__ cnt)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nout) return;
    const int i = c_rowof[c], j = c_col[c];
    int64_t pa = a_ptr[i], ea = a_ptr[i + 1], pb = b_ptr[j], eb = b_ptr[j + 1];
    int64_t n = 0;
    while (pa < ea && pb < eb) {
        const int ka = a_col[pa], kb = b_col[pb];
        n += (ka == kb);
        pa += (ka <= kb);
        pb += (kb <= ka);
    }
    cnt[c] = n;
}

__global__ void k_sym_fill(int64_t nout, const int32_t *__restrict__ c_rowof,
                           const int32_t *__restrict__ c_col, const int64_t *__restrict__ a_ptr,
                           const int32_t *__restrict__ a_col, const int32_t *__restrict__ a_trans,
                           const int64_t *__restrict__ b_ptr, const int32_t *__restrict__ b_col,
                           const int32_t *__restrict__ b_trans, int op_a, int op_b,
                           const int64_t *__restrict__ off, int2 *__restrict__ trip)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nout) return;
    const int i = c_rowof[c], j = c_col[c];
    int64_t pa = a_ptr[i], ea = a_ptr[i + 1], pb = b_ptr[j], eb = b_ptr[j + 1];
    int64_t o = off[c];
    while (pa < ea && pb < eb) {
        const int ka = a_col[pa], kb = b_col[pb];
        if (ka == kb) {
            // op(A)_ik: block (i,k) = pa, or (k,i) = trans[pa] for the conjugate transpose.
            // op(B)_kj: block (k,j) = trans[pb] (pb is (j,k)), or (j,k) = pb for the conjugate transpose.
            const int ia = op_a ? a_trans[pa] : (int)pa;
            const int ib = op_b ? (int)pb : b_trans[pb];
            trip[o++] = make_int2(ia, ib);
        }
        pa += (ka <= kb);
        pb += (kb <= ka);
    }
}

// Row runs (see SpgemmArgs::ch_*): one thread per run of up to nj (<= 16)
// consecutive outputs p0 .. p1-1 of row i of C, op(A) = A.  The thread walks
// row i of A (ascending k) and, in step, the rows j_t of B's pattern (the
// patterns are symmetric, so k in row j_t means block (k, j_t) exists); an
// entry is a k present for at least one output.  Slot of output t in an
// entry: t, or (t % 4) * 4 + t / 4 with `inter4` (the lane order of the b = 4
// kernel, whose lane group g reads outputs g, g + 4, g + 8, g + 12).
constexpr int kMaxRun = 16, kRunThreads = 128;

// Set of outputs (a bit mask) of the u-th group of a segmented run of 2: both, first, second.
constexpr int kRunClasses = 3;
__device__ inline int run_class(int u) { return (0x213 >> (4 * u)) & 15; }

template <bool FILL>
__global__ void k_run_sym(int64_t nch, const int32_t *__restrict__ run_row, const int64_t *__restrict__ run_p0,
                          const int64_t *__restrict__ c_ptr, const int32_t *__restrict__ c_col,
                          const int64_t *__restrict__ a_ptr, const int32_t *__restrict__ a_col,
                          const int64_t *__restrict__ b_ptr, const int32_t *__restrict__ b_col,
                          const int32_t *__restrict__ b_trans, int op_b, int nj, int inter4,
                          int64_t *__restrict__ cnt, const int64_t *__restrict__ off, int32_t *__restrict__ ea,
                          int32_t *__restrict__ eb, int32_t *__restrict__ rout, int32_t *__restrict__ seg)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nch) return;
    const int i = run_row[c];
    const int64_t p0 = run_p0[c];
    const int m = (int)min<int64_t>(nj, c_ptr[i + 1] - p0);
    int64_t pb[kMaxRun], eb_end[kMaxRun];
    for (int t = 0; t < m; ++t) {
        const int j = c_col[p0 + t];
        pb[t] = b_ptr[j];
        eb_end[t] = b_ptr[j + 1];
    }
    if (FILL)
        for (int t = 0; t < nj; ++t) rout[c * nj + t] = t < m ? (int32_t)(p0 + t) : -1;
    // Segmented runs (seg, runs of 2): the entries grouped by the set of outputs
    // they feed (run_class order), each group in ascending k, so that a kernel
    // issues only present products; seg holds the sizes of the first two groups.
    // One walk counts (or places) every group, its counters (or cursors) in LDS.
    __shared__ int32_t cur[kRunThreads][kRunClasses + 1];
    int32_t *my = cur[threadIdx.x];
    if (seg) {
        int32_t at = 0;
        for (int u = 0; u < kRunClasses; ++u) {
            my[run_class(u)] = FILL ? at : 0;
            if (FILL && u < 2) at += seg[2 * c + u];
        }
    }
    int64_t n = 0, o = FILL ? off[c] : 0;
    for (int64_t pa = a_ptr[i]; pa < a_ptr[i + 1]; ++pa) {
        const int k = a_col[pa];
        int mask = 0;
        for (int t = 0; t < m; ++t) {
            while (pb[t] < eb_end[t] && b_col[pb[t]] < k) ++pb[t];
            if (pb[t] < eb_end[t] && b_col[pb[t]] == k) mask |= 1 << t;
        }
        if (!mask) continue;
        if (!FILL) {
            ++n;
            if (seg) ++my[mask];
            continue;
        }
        const int64_t e = seg ? off[c] + my[mask]++ : o++;
        ea[e] = (int32_t)pa;
        for (int t = 0; t < nj; ++t) {
            const int slot = inter4 ? (t & 3) * 4 + (t >> 2) : t;
            int32_t v = -1;
            // op(B)_kj: block (k, j) = trans of (j, k), or (j, k) itself for the conjugate transpose
            if ((mask >> t) & 1) v = op_b ? (int32_t)pb[t] : b_trans[pb[t]];
            eb[e * nj + slot] = v;
        }
    }
    if (!FILL) {
        cnt[c] = n;
        if (seg)
            for (int u = 0; u < 2; ++u) seg[2 * c + u] = my[run_class(u)];
    }
}

void launch_run_count(hipStream_t s, int64_t nch, const int32_t *run_row, const int64_t *run_p0, const int64_t *c_ptr,
                      const int32_t *c_col, const int64_t *a_ptr, const int32_t *a_col, const int64_t *b_ptr,
                      const int32_t *b_col, int nj, int64_t *cnt, int32_t *seg)
{
    if (nch == 0) return;
    RT_CHECK(nj >= 1 && nj <= kMaxRun, RTDM_E_ARG, "row runs hold 1..16 outputs");
    RT_CHECK(!seg || nj == 2, RTDM_E_ARG, "segmented row runs hold 2 outputs");
    hipLaunchKernelGGL(k_run_sym<false>, dim3((unsigned)((nch + kRunThreads - 1) / kRunThreads)), dim3(kRunThreads), 0, s,
                       nch, run_row, run_p0, c_ptr, c_col, a_ptr, a_col, b_ptr, b_col, nullptr, 0, nj, 0, cnt, nullptr,
                       nullptr, nullptr, nullptr, seg);
    RT_HIP(hipGetLastError());
}

void launch_run_fill(hipStream_t s, int64_t nch, const int32_t *run_row, const int64_t *run_p0, const int64_t *c_ptr,
                     const int32_t *c_col, const int64_t *a_ptr, const int32_t *a_col, const int64_t *b_ptr,
                     const int32_t *b_col, const int32_t *b_trans, int op_b, int nj, int inter4, const int64_t *off,
                     int32_t *ea, int32_t *eb, int32_t *rout, int32_t *seg)
{
    if (nch == 0) return;
    RT_CHECK(nj >= 1 && nj <= kMaxRun, RTDM_E_ARG, "row runs hold 1..16 outputs");
    RT_CHECK(!seg || (nj == 2 && !inter4), RTDM_E_ARG, "segmented row runs hold 2 outputs");
    hipLaunchKernelGGL(k_run_sym<true>, dim3((unsigned)((nch + kRunThreads - 1) / kRunThreads)), dim3(kRunThreads), 0, s,
                       nch, run_row, run_p0, c_ptr, c_col, a_ptr, a_col, b_ptr, b_col, b_trans, op_b, nj, inter4, nullptr,
                       off, ea, eb, rout, seg);
    RT_HIP(hipGetLastError());
}

void launch_sym_count(hipStream_t s, int64_t nout, const int32_t *c_rowof, const int32_t *c_col,
                      const int64_t *a_ptr, const int32_t *a_col, const int64_t *b_ptr,
                      const int32_t *b_col, int64_t *cnt)
{
    if (nout == 0) return;
    const int T = 256;
    hipLaunchKernelGGL(k_sym_count, dim3((unsigned)((nout + T - 1) / T)), dim3(T), 0, s, nout,
                       c_rowof, c_col, a_ptr, a_col, b_ptr, b_col, cnt);
    RT_HIP(hipGetLastError());
}

void launch_sym_fill(hipStream_t s, int64_t nout, const int32_t *c_rowof, const int32_t *c_col,
                     const int64_t *a_ptr, const int32_t *a_col, const int32_t *a_trans,
                     const int64_t *b_ptr, const int32_t *b_col, const int32_t *b_trans, int op_a,
                     int op_b, const int64_t *off, int2 *trip)
{
    if (nout == 0) return;
    const int T = 256;
    hipLaunchKernelGGL(k_sym_fill, dim3((unsigned)((nout + T - 1) / T)), dim3(T), 0, s, nout,
                       c_rowof, c_col, a_ptr, a_col, a_trans, b_ptr, b_col, b_trans, op_a, op_b,
                       off, trip);
    RT_HIP(hipGetLastError());
}

// ----------------------------------------------------------------- numeric

// MFMA 16x16x4 f64 operand layout (wave of 64 lanes, lane = 16*q + r), as
// measured on gfx950:
//   A operand: lane supplies A[r][q]   (row r of the 16x4 slice, column q)
//   B operand: lane supplies B[q][r]   (row q of the 4x16 slice, column r)
//   D (4 doubles per lane): element e of lane is D[4*e + q][r]
template <bool AC, bool BC, int OPA, int OPB>
__global__ __launch_bounds__(256) void k_spgemm16(
    int64_t nout, const int64_t *__restrict__ off, const int2 *__restrict__ trip,
    const double *__restrict__ ar, const double *__restrict__ ai, const double *__restrict__ br,
    const double *__restrict__ bi, double *__restrict__ cr, double *__restrict__ ci, int b,
    double alr, double ali)
{
    const int lane = threadIdx.x & 63;
    const int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (c >= nout) return;                     // uniform across the wave
    const int bb = b * b;
    const int r = lane & 15, q = lane >> 4;
    d4 rr = {0, 0, 0, 0}, ii = {0, 0, 0, 0}, ri = {0, 0, 0, 0}, ir = {0, 0, 0, 0};
    const int64_t t0 = off[c], t1 = off[c + 1];
    for (int64_t t = t0; t < t1; ++t) {
        const int2 ab = trip[t];
        const int64_t abase = (int64_t)ab.x * bb, bbase = (int64_t)ab.y * bb;
        for (int k0 = 0; k0 < b; k0 += 4) {
            const int kk = k0 + q;
            const bool ok = (r < b) && (kk < b);
            const int ia = OPA ? (kk * b + r) : (r * b + kk);   // op(A)[r][kk]
            const int ib = OPB ? (r * b + kk) : (kk * b + r);   // op(B)[kk][r]
            double xar = 0.0, xai = 0.0, xbr = 0.0, xbi = 0.0;
            if (ok) {
                xar = ar[abase + ia];
                xbr = br[bbase + ib];
                if (AC) xai = OPA ? -ai[abase + ia] : ai[abase + ia];
                if (BC) xbi = OPB ? -bi[bbase + ib] : bi[bbase + ib];
            }
            rr = __builtin_amdgcn_mfma_f64_16x16x4f64(xar, xbr, rr, 0, 0, 0);
            if (AC && BC) ii = __builtin_amdgcn_mfma_f64_16x16x4f64(xai, xbi, ii, 0, 0, 0);
            if (BC) ri = __builtin_amdgcn_mfma_f64_16x16x4f64(xar, xbi, ri, 0, 0, 0);
            if (AC) ir = __builtin_amdgcn_mfma_f64_16x16x4f64(xai, xbr, ir, 0, 0, 0);
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int row = 4 * e + q, col = r;
        if (row < b && col < b) {
            const double re = rr[e] - ii[e];
            const double im = ri[e] + ir[e];
            const int64_t o = c * bb + row * b + col;
            cr[o] = alr * re - ali * im;
            if (ci) ci[o] = alr * im + ali * re;
        }
    }
}

// Compile-time block size B <= 16 with the contraction concatenated across the
// triples of one output block: the kappa-th contraction index is element m of
// triple tt (kappa = B*tt + m), so the 4-wide MFMA steps run over B*ntrip
// indices instead of padding every triple from B to a multiple of 4.  Lane
// (q, r) supplies index kappa = 4*s + q at step s.  The operands of step s+1
// are loaded before the matrix-core work of step s is issued.

// Workgroups are dealt to the 8 XCDs (each with its own L2) round-robin by
// block index.  xcd_block() with remap = 1 renumbers them so that XCD x runs
// the contiguous range [x*per, (x+1)*per) of logical blocks: neighbouring
// output blocks, which share operand blocks, then meet in the same L2.  The
// grid is launched with 8*per blocks; logical indices >= the real count exit.
//
// remap > 1 deals chunks of `remap` consecutive logical blocks to the XCDs
// round-robin instead (chunk m to XCD m % 8), so that the XCDs work on
// neighbouring chunks at the same time; the grid is then a multiple of
// 8*remap (xcd_grid with the same remap).
constexpr int kXcds = 8;
__device__ inline int64_t xcd_block(int64_t nblocks, int remap = 1)
{
    if (!remap) return blockIdx.x;
    const int64_t x = blockIdx.x % kXcds, i = blockIdx.x / kXcds;
    if (remap > 1) return ((i / remap) * kXcds + x) * remap + i % remap;
    const int64_t per = (nblocks + kXcds - 1) / kXcds;
    return x * per + i;
}
static inline unsigned xcd_grid(int64_t nblocks, int remap = 1)
{
    const int64_t unit = remap > 1 ? (int64_t)kXcds * remap : kXcds;
    return (unsigned)(((nblocks + unit - 1) / unit) * unit);
}

// XCD mapping of the row-run kernels: the chunk size of the round-robin deal
// (128 workgroups: the XCDs then stream neighbouring outputs, whose operand
// blocks meet in the shared last-level cache; contiguous eighths measured
// 11 % slower at b = 13).
static int xcd_chunk() { return 128; }
// Chunks for a launch of nwg workgroups: 128 from 16,384 workgroups on, 32 below,
// where larger ones leave the last round of chunks nearly empty.  U K with chunks
// of 32 / 128, us, at so many workgroups: b = 13 916 / 941 (4,925), 3,515 / 3,654
// (9,683), 1,961 / 2,047 (10,654), 8,519 / 8,588 (21,861), 13,201 / 13,213 (33,490),
// 16,762 / 16,973 (41,440); b = 4 156 / 181 (2,582), 414 / 426 (4,356), 505 / 503
// (9,204), 1,217 / 1,246 (13,658), 2,139 / 2,109 (24,260).  Above the line the two
// are within 1.5 % of each other.  The rule is wrong where rows are long: b = 4,
// 2,744 atoms at R 16 (13 runs a row, 9,064 workgroups) takes 1,965 / 1,854.
static int xcd_chunk_for(int64_t nwg) { return nwg < 16384 ? 32 : xcd_chunk(); }
// The same deal in chunks of about as many output blocks (1,024) for a kernel
// with `per_wg` output blocks per workgroup.
static int xcd_chunk_wg(int per_wg) { return std::max(2, xcd_chunk() * 8 / std::max(per_wg, 1)); }

// Matrix-core step on one 16x16 tile: FP64 (v_mfma_f64_16x16x4_f64) or
// FP32 (v_mfma_f32_16x16x4_f32).  Both take A[r][q] / B[q][r] from lane
// 16*q + r; element e of the result sits in row 4*e + q for FP64 and in row
// 4*q + e for FP32 (measured on gfx950).
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <class T> struct Mfma16;
template <> struct Mfma16<double> {
    typedef double acc_t __attribute__((ext_vector_type(4)));
    static __device__ inline acc_t step(double a, double b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int e, int q) { return 4 * e + q; }
};
template <> struct Mfma16<float> {
    typedef float acc_t __attribute__((ext_vector_type(4)));
    static __device__ inline acc_t step(float a, float b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int e, int q) { return 4 * q + e; }
};

// TA / TB: the stored block is read transposed (op(A)[r][m] at m*B + r, op(B)[m][r]
// at r*B + m); CJA / CJB: conjugate; LC: write the output block column-major.
// A conjugate transpose of a row-major block is TA = CJA = 1; a column-major
// copy of a left operand is TA = 1, CJA = 0, so that the 16 lanes of a row
// group read contiguous doubles.
template <int B, bool AC, bool BC, int TA, int TB, class T = double, int CJA = TA, int CJB = TB,
          int LC = 0>
__global__ __launch_bounds__(256) void k_spgemm_kc(
    int64_t nout, const int64_t *__restrict__ off, const int2 *__restrict__ trip,
    const double *__restrict__ ar, const double *__restrict__ ai, const double *__restrict__ br,
    const double *__restrict__ bi, double *__restrict__ cr, double *__restrict__ ci, double alr,
    double ali)
{
    static_assert(B >= 4 && B <= 16, "k_spgemm_kc needs 4 <= B <= 16");
    constexpr int BB = B * B;
    const int lane = threadIdx.x & 63;
    const int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (c >= nout) return;                     // uniform across the wave
    const int r = lane & 15, q = lane >> 4;
    const bool rv = r < B;
    const int64_t t0 = off[c];
    const int nt = (int)(off[c + 1] - t0);
    const int steps = (B * nt + 3) >> 2;
    // per-lane element offsets inside a block for op(A)[r][m] and op(B)[m][r]
    const int oa_r = TA ? r : r * B;           // + m * (TA ? B : 1)
    const int ob_r = TB ? r * B : r;           // + m * (TB ? 1 : B)
    constexpr int sa = TA ? B : 1, sb = TB ? 1 : B;

    int tt = 0, m = q;                         // B >= 4: the first step stays in triple 0
    int2 ab = nt > 0 ? trip[t0] : make_int2(0, 0);
    T xar = 0, xai = 0, xbr = 0, xbi = 0;
    auto fetch = [&](T &far, T &fai, T &fbr, T &fbi) {
        far = fai = fbr = fbi = 0;
        if (tt < nt && rv) {
            const int64_t pa = (int64_t)ab.x * BB + oa_r + m * sa;
            const int64_t pb = (int64_t)ab.y * BB + ob_r + m * sb;
            far = (T)ar[pa];
            fbr = (T)br[pb];
            if (AC) fai = (T)(CJA ? -ai[pa] : ai[pa]);
            if (BC) fbi = (T)(CJB ? -bi[pb] : bi[pb]);
        }
    };
    auto advance = [&]() {
        m += 4;
        if (m >= B) {
            m -= B;
            ++tt;
            if (tt < nt) ab = trip[t0 + tt];
        }
    };
    typedef typename Mfma16<T>::acc_t acc_t;
    acc_t rr = {0, 0, 0, 0}, ii = {0, 0, 0, 0}, ri = {0, 0, 0, 0}, ir = {0, 0, 0, 0};
    fetch(xar, xai, xbr, xbi);
    for (int s = 0; s < steps; ++s) {
        advance();
        T nar, nai, nbr, nbi;
        fetch(nar, nai, nbr, nbi);
        rr = Mfma16<T>::step(xar, xbr, rr);
        if (AC && BC) ii = Mfma16<T>::step(xai, xbi, ii);
        if (BC) ri = Mfma16<T>::step(xar, xbi, ri);
        if (AC) ir = Mfma16<T>::step(xai, xbr, ir);
        xar = nar;
        xai = nai;
        xbr = nbr;
        xbi = nbi;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int row = Mfma16<T>::row(e, q), col = r;
        if (row < B && col < B) {
            const double re = (double)rr[e] - (double)ii[e];
            const double im = (double)ri[e] + (double)ir[e];
            const int64_t o = c * BB + (LC ? col * B + row : row * B + col);
            cr[o] = alr * re - ali * im;
            if (ci) ci[o] = alr * im + ali * re;
        }
    }
}

// Step products, B = 13 or 16: the contraction of one output block runs over
// groups of four triples.  In each 4-wide MFMA step the lane group q (16
// lanes) supplies element s of the group's q-th triple, so B steps consume
// the four triples exactly (the order of the contraction sum is the only
// difference from a triple-by-triple loop).  The left operand is a
// column-major copy (op(A)[r][s] at s*B + r) and the right operand has
// op(B)[s][r] at s*B + r, so every load is a per-group base pointer plus a
// compile-time offset; lanes without data (rows r >= B, or past the last
// triple) point at a zero block.  Conjugation is a sign applied to the
// accumulated imaginary products at the end.
//
// T = float runs the same dataflow on the FP32 matrix cores (operands rounded
// to FP32 on load, FP32 accumulation).
template <int B, bool AC, bool BC, int CJA, int CJB, int LC, int WPB = 4, class T = double>
__global__ __launch_bounds__(64 * WPB) void k_spgemm_q4(
    int64_t nout, const int64_t *__restrict__ off, const int2 *__restrict__ trip,
    const double *__restrict__ ar, const double *__restrict__ ai, const double *__restrict__ br,
    const double *__restrict__ bi, double *__restrict__ cr, double *__restrict__ ci, double alr,
    double ali, const double *__restrict__ zero, const int32_t *__restrict__ order, int remap)
{
    static_assert(B >= 4 && B <= 16, "k_spgemm_q4 needs 4 <= B <= 16");
    constexpr int BB = B * B;
    const int lane = threadIdx.x & 63;
    const int64_t w = xcd_block((nout + WPB - 1) / WPB, remap) * WPB + (threadIdx.x >> 6);
    if (w >= nout) return;                     // uniform across the wave
    const int64_t c = order ? (int64_t)order[w] : w;
    const int r = lane & 15, q = lane >> 4;
    const bool rv = r < B;
    const int64_t t0 = off[c];
    const int nt = (int)(off[c + 1] - t0);
    typedef typename Mfma16<T>::acc_t acc_t;
    acc_t rr = {0, 0, 0, 0}, ii = {0, 0, 0, 0}, ri = {0, 0, 0, 0}, ir = {0, 0, 0, 0};
    for (int g = 0; g < nt; g += 4) {
        const double *pa = zero, *pai = zero, *pb = zero, *pbi = zero;
        if (rv && g + q < nt) {
            const int2 ab = trip[t0 + g + q];
            const int64_t oa = (int64_t)ab.x * BB + r, ob = (int64_t)ab.y * BB + r;
            pa = ar + oa;
            pb = br + ob;
            if (AC) pai = ai + oa;
            if (BC) pbi = bi + ob;
        }
#pragma unroll
        for (int st = 0; st < B; ++st) {
            const T xa = (T)pa[st * B], xb = (T)pb[st * B];
            rr = Mfma16<T>::step(xa, xb, rr);
            if (AC && BC) ii = Mfma16<T>::step((T)pai[st * B], (T)pbi[st * B], ii);
            if (BC) ri = Mfma16<T>::step(xa, (T)pbi[st * B], ri);
            if (AC) ir = Mfma16<T>::step((T)pai[st * B], xb, ir);
        }
    }
    // op(A)_im = sa * A_im, op(B)_im = sb * B_im
    constexpr double sa = CJA ? -1.0 : 1.0, sb = CJB ? -1.0 : 1.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int row = Mfma16<T>::row(e, q), col = r;
        if (row < B && col < B) {
            const double re = (double)rr[e] - (sa * sb) * (double)ii[e];
            const double im = sb * (double)ri[e] + sa * (double)ir[e];
            const int64_t o = c * BB + (LC ? col * B + row : row * B + col);
            cr[o] = alr * re - ali * im;
            if (ci) ci[o] = alr * im + ali * re;
        }
    }
}

typedef __attribute__((address_space(1))) const double gdouble;

// Row runs of the step products: one wave computes NJ output blocks C_ij of
// the same row i.  The entries of the run are the contraction indices k used
// by any of its outputs; lane group q takes entry g + q, loads op(A)_ik once
// and op(B)_kj of every output (the zero block where that output has no
// triple with this k), and each loaded A element feeds NJ MFMAs.  The operand
// blocks of A beyond L2 are then fetched once per run instead of once per
// output; the price is the absent (zero) products of a run.  Data layout,
// lane mapping, conjugation and output as in k_spgemm_q4.
// seg (runs of 2, optional): per run the number of entries that feed both
// outputs (seg[2c]) and only the first (seg[2c+1]); the entries are stored in
// that order, the rest feed only the second.  Each segment then runs with
// only its outputs' products, so no matrix work goes to absent entries.
template <int B, bool AC, bool BC, int CJB, int LC, int NJ, class T = double, int MINW = 1>
__global__ __launch_bounds__(256, MINW) void k_spgemm_q4j(
    int64_t nch, const int64_t *__restrict__ off, const int32_t *__restrict__ ea,
    const int32_t *__restrict__ eb, const int32_t *__restrict__ cout,
    const double *__restrict__ ar, const double *__restrict__ ai, const double *__restrict__ br,
    const double *__restrict__ bi, double *__restrict__ cr, double *__restrict__ ci, double alr,
    double ali, const double *__restrict__ zero, const int32_t *__restrict__ order, int remap,
    const int32_t *__restrict__ seg)
{
    static_assert(B >= 4 && B <= 16, "k_spgemm_q4j needs 4 <= B <= 16");
    constexpr int BB = B * B;
    const int lane = threadIdx.x & 63;
    const int64_t w = xcd_block((nch + 3) / 4, remap) * 4 + (threadIdx.x >> 6);
    if (w >= nch) return;                      // uniform across the wave
    const int64_t c = order ? (int64_t)order[w] : w;
    const int r = lane & 15, q = lane >> 4;
    const bool rv = r < B;
    const int64_t e0 = off[c];
    const int ne = (int)(off[c + 1] - e0);
    typedef typename Mfma16<T>::acc_t acc_t;
    acc_t rr[NJ], ri[NJ], ir[NJ];
#pragma unroll
    for (int t = 0; t < NJ; ++t) rr[t] = ri[t] = ir[t] = acc_t{0, 0, 0, 0};
    const gdouble *gz = (const gdouble *)zero;
    // entries [gb, ge) of the run; output t's products only where bit t of ACT is set
    auto groups = [&](int gb, int ge, auto act) {
        constexpr int ACT = decltype(act)::value;
        for (int g = gb; g < ge; g += 4) {
            // global-address-space pointers: the loads stay global loads (flat
            // loads would make every wait drain the scalar-memory counter too)
            const gdouble *pa = gz, *pai = gz;
            const gdouble *pb[NJ], *pbi[NJ];
#pragma unroll
            for (int t = 0; t < NJ; ++t) pb[t] = pbi[t] = gz;
            if (rv && g + q < ge) {
                const int64_t e = e0 + g + q;
                const int64_t oa = (int64_t)ea[e] * BB + r;
                pa = (const gdouble *)(ar + oa);
                if (AC) pai = (const gdouble *)(ai + oa);
#pragma unroll
                for (int t = 0; t < NJ; ++t) {
                    if (!((ACT >> t) & 1)) continue;
                    const int kb = eb[e * NJ + t];
                    if (kb >= 0) {
                        const int64_t ob = (int64_t)kb * BB + r;
                        pb[t] = (const gdouble *)(br + ob);
                        if (BC) pbi[t] = (const gdouble *)(bi + ob);
                    }
                }
            }
#pragma unroll
            for (int st = 0; st < B; ++st) {
                const T xa = (T)pa[st * B];
                const T xai = AC ? (T)pai[st * B] : (T)0;
                if constexpr (AC && BC) {
                    // two accumulators per output: re += a_r b_r + (-s a_i) b_i,
                    // im += (s a_r) b_i + a_i b_r with s = -1 for a conjugated B
                    const T nai = CJB ? xai : -xai, sar = CJB ? -xa : xa;
#pragma unroll
                    for (int t = 0; t < NJ; ++t) {
                        if (!((ACT >> t) & 1)) continue;
                        const T xb = (T)pb[t][st * B], xbi = (T)pbi[t][st * B];
                        rr[t] = Mfma16<T>::step(xa, xb, rr[t]);
                        ri[t] = Mfma16<T>::step(sar, xbi, ri[t]);
                        rr[t] = Mfma16<T>::step(nai, xbi, rr[t]);
                        ri[t] = Mfma16<T>::step(xai, xb, ri[t]);
                    }
                } else {
#pragma unroll
                    for (int t = 0; t < NJ; ++t) {
                        if (!((ACT >> t) & 1)) continue;
                        const T xb = (T)pb[t][st * B];
                        const T xbi = BC ? (T)pbi[t][st * B] : (T)0;
                        rr[t] = Mfma16<T>::step(xa, xb, rr[t]);
                        if (BC) ri[t] = Mfma16<T>::step(xa, xbi, ri[t]);
                        if (AC) ir[t] = Mfma16<T>::step(xai, xb, ir[t]);
                    }
                }
            }
        }
    };
    constexpr int ALL = (1 << NJ) - 1;
    if constexpr (NJ == 2) {
        if (seg) {
            const int nf = seg[2 * c], n0 = seg[2 * c + 1];   // uniform across the wave
            groups(0, nf, std::integral_constant<int, 3>());
            groups(nf, nf + n0, std::integral_constant<int, 1>());
            groups(nf + n0, ne, std::integral_constant<int, 2>());
        } else {
            groups(0, ne, std::integral_constant<int, ALL>());
        }
    } else {
        groups(0, ne, std::integral_constant<int, ALL>());
    }
    constexpr double sb = CJB ? -1.0 : 1.0;
#pragma unroll
    for (int t = 0; t < NJ; ++t) {
        const int p = cout[c * NJ + t];
        if (p < 0) continue;                   // uniform: a short run
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = Mfma16<T>::row(e, q), col = r;
            if (row < B && col < B) {
                const double re = (double)rr[t][e];
                const double im = (AC && BC) ? (double)ri[t][e] : sb * (double)ri[t][e] + (double)ir[t][e];
                const int64_t o = (int64_t)p * BB + (LC ? col * B + row : row * B + col);
                cr[o] = alr * re - ali * im;
                if (ci) ci[o] = alr * im + ali * re;
            }
        }
    }
}

// Row runs of 2 (k_spgemm_q4j's dataflow, segments and order of the products)
// on operands in pair layout.  Bound: at b = 13 the row-run products were held
// by the vector-memory address unit, which takes 15 cycles for a wave's
// 8-byte load and the same 15 for a 16-byte one, aligned or not (measured from
// L1 and L2); it was busy 97 % of the real kernel's cycles with the matrix
// cores busy 52 %.  The pair layout brings two contraction steps per load:
// 7 loads per operand block instead of 13.  Lanes 13..15 of a row group read
// row 12 again: they only feed rows and columns of the tile that are not
// stored.  The complex products are then held by the matrix cores (84 % of
// all cycles busy, 13 of 16 rows and columns of a tile useful); the real one,
// with half the operations per byte, by operand blocks from beyond the XCD's L2 (512 atoms:
// its loads alone take 1.10 ms of 1.23, 0.86 if the L2 held them all; its
// matrix instructions alone 0.95).  Fewer outputs sharing an L2 are better
// there: three waves per SIMD beat four by 8 % and five by 18 %, and with the
// next group's loads issued behind this one's matrix instructions two beat
// three by 4 %.  4,096 atoms, R 16, ms per launch, 8-byte loads at four waves
// -> now (four cards): A tau 19.9 -> 15.5 to 15.8, U K 49.7 -> 44.9 to 47.6, W U^dagger
// 48.3 -> 44.5 to 47.4.
// Complex products have no registers to load a group ahead.
// OUT: 0 row-major output, 1 left pairs, 2 right pairs.  u (real products,
// nullable): u = u_sign * output (u_store) or u += u_sign * output, row-major:
// the Taylor sum, whose own pass would read the term again.  ROWS: both operands
// by rows as they are stored, for products recorded into a caller's graph, which
// may use no buffer of the context's: A in the same 16-byte loads, 104 bytes from
// lane to lane, B in two 8-byte ones; the same products in the same order.  SEG =
// false (complex products): entries in ascending k without segments, absent ones
// read from the zero block; more matrix instructions for the order of the sums.
typedef double pd2 __attribute__((ext_vector_type(2), aligned(8)));
typedef __attribute__((address_space(1))) const pd2 gpd2;
template <int B, bool AC, bool BC, int CJB, int OUT, bool ROWS, bool SEG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(AC || BC ? 3 : 2, AC || BC ? 3 : 2))) void k_spgemm_q4p(
    int64_t nch, const int64_t *__restrict__ off, const int32_t *__restrict__ ea,
    const int32_t *__restrict__ eb, const int32_t *__restrict__ cout,
    const double *__restrict__ ar, const double *__restrict__ ai, const double *__restrict__ br,
    const double *__restrict__ bi, double *__restrict__ cr, double *__restrict__ ci, double alr,
    double ali, const double *__restrict__ zero, const int32_t *__restrict__ order, int remap,
    const int32_t *__restrict__ seg, double *__restrict__ u, double u_sign, int u_store)
{
    static_assert(B >= 5 && B <= 15 && (B & 1), "odd block sizes");
    static_assert(!ROWS || !CJB, "a conjugated right operand has its pair layout");
    static_assert(SEG || (AC && BC), "entries without segments: complex operands");
    constexpr int BB = B * B, NJ = 2;
    const int lane = threadIdx.x & 63;
    const int64_t w = xcd_block((nch + 3) / 4, remap) * 4 + (threadIdx.x >> 6);
    if (w >= nch) return;                      // uniform across the wave
    const int64_t c = order ? (int64_t)order[w] : w;
    const int q = lane >> 4, r = min(lane & 15, B - 1);
    const int64_t e0 = off[c];
    const int ne = (int)(off[c + 1] - e0);
    // a lane's first pair in an operand block, its pair h, and its last, unpaired element
    const int fa = ROWS ? r * B : 2 * r, fb = ROWS ? r : 2 * r;
    auto last_left = [&]() { return ROWS ? B - 1 : B * (B - 1) - r; };
    auto last_right = [&]() { return ROWS ? B * (B - 1) : B * (B - 1) - r; };
    auto left_pair = [](const gdouble *p, int h) { return *(const gpd2 *)(p + (ROWS ? 2 : 2 * B) * h); };
    auto right_pair = [](const gdouble *p, int h) {
        return ROWS ? pd2{p[2 * B * h], p[2 * B * h + B]} : *(const gpd2 *)(p + 2 * B * h);
    };
    typedef Mfma16<double>::acc_t acc_t;
    // four sums per complex output (two, with the sign folded into an operand, were
    // no faster at three waves and doubled the roundings of the real part: K of the
    // 512-atom lattice after 4 steps 5.6e-15 -> 2.6e-15 from 64-bit arithmetic)
    acc_t rr[NJ], ri[NJ], ir[NJ], ii[NJ];
#pragma unroll
    for (int t = 0; t < NJ; ++t) rr[t] = ri[t] = ir[t] = ii[t] = acc_t{0, 0, 0, 0};
    const gdouble *gz = (const gdouble *)zero;
    // block indices of the group about to run, loaded one group ahead (the
    // group after a segment's last is the next segment's first)
    int na = 0, nb[NJ] = {0, 0};
    auto fetch = [&](int g) {
        const int64_t e = e0 + min(g + q, ne - 1);
        na = ea[e];
#pragma unroll
        for (int t = 0; t < NJ; ++t) nb[t] = eb[e * NJ + t];
    };
    if (ne > 0) fetch(0);
    auto groups = [&](int gb, int ge, auto act) {
        constexpr int ACT = decltype(act)::value;
        if constexpr (!AC && !BC) {
            // slice h of the next group is loaded into the registers that slice h of
            // this one has just left, so a group's loads have its matrix
            // instructions' time to arrive
            if (gb >= ge) return;
            const gdouble *pa = gz, *pb[NJ] = {gz, gz};
            pd2 xa[B / 2], xb[NJ][B / 2];
            double ya = 0, yb[NJ] = {0, 0};
            auto point = [&](int g) {
                const bool on = g + q < ge;
                pa = on ? (const gdouble *)(ar + (int64_t)na * BB + fa) : gz;
#pragma unroll
                for (int t = 0; t < NJ; ++t)
                    if ((ACT >> t) & 1) pb[t] = on ? (const gdouble *)(br + (int64_t)nb[t] * BB + fb) : gz;
                fetch(min(g + 4, ge));
            };
            auto load = [&](int h) {
                xa[h] = left_pair(pa, h);
#pragma unroll
                for (int t = 0; t < NJ; ++t)
                    if ((ACT >> t) & 1) xb[t][h] = right_pair(pb[t], h);
            };
            auto load_last = [&]() {                   // the unpaired contraction index
                ya = pa[last_left()];
#pragma unroll
                for (int t = 0; t < NJ; ++t)
                    if ((ACT >> t) & 1) yb[t] = pb[t][last_right()];
            };
            auto mma = [&](double va, double v0, double v1) {
                if (ACT & 1) rr[0] = Mfma16<double>::step(va, v0, rr[0]);
                if (ACT & 2) rr[1] = Mfma16<double>::step(va, v1, rr[1]);
            };
            point(gb);
#pragma unroll
            for (int h = 0; h < B / 2; ++h) load(h);
            load_last();
            __builtin_amdgcn_sched_barrier(0);
            for (int g = gb + 4; g < ge; g += 4) {
                point(g);
#pragma unroll
                for (int h = 0; h < B / 2; ++h) {
                    mma(xa[h].x, xb[0][h].x, xb[1][h].x);
                    mma(xa[h].y, xb[0][h].y, xb[1][h].y);
                    load(h);
                    __builtin_amdgcn_sched_barrier(0);
                }
                mma(ya, yb[0], yb[1]);
                load_last();
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int h = 0; h < B / 2; ++h) {
                mma(xa[h].x, xb[0][h].x, xb[1][h].x);
                mma(xa[h].y, xb[0][h].y, xb[1][h].y);
            }
            mma(ya, yb[0], yb[1]);
            return;
        }
        for (int g = gb; g < ge; g += 4) {
            const gdouble *pa = gz, *pai = gz;
            const gdouble *pb[NJ], *pbi[NJ];
#pragma unroll
            for (int t = 0; t < NJ; ++t) pb[t] = pbi[t] = gz;
            if (g + q < ge) {
                const int64_t oa = (int64_t)na * BB + fa;
                pa = (const gdouble *)(ar + oa);
                if (AC) pai = (const gdouble *)(ai + oa);
#pragma unroll
                for (int t = 0; t < NJ; ++t) {
                    if (!((ACT >> t) & 1)) continue;
                    if (!SEG && nb[t] < 0) continue;               // (segmented entries are all present)
                    const int64_t ob = (int64_t)nb[t] * BB + fb;
                    pb[t] = (const gdouble *)(br + ob);
                    if (BC) pbi[t] = (const gdouble *)(bi + ob);
                }
            }
            fetch(min(g + 4, ge));
            auto mma = [&](double xa, double xai, const double (&xb)[NJ], const double (&xbi)[NJ]) {
#pragma unroll
                for (int t = 0; t < NJ; ++t) {
                    if (!((ACT >> t) & 1)) continue;
                    rr[t] = Mfma16<double>::step(xa, xb[t], rr[t]);
                    if (AC && BC) ii[t] = Mfma16<double>::step(xai, xbi[t], ii[t]);
                    if (BC) ri[t] = Mfma16<double>::step(xa, xbi[t], ri[t]);
                    if (AC) ir[t] = Mfma16<double>::step(xai, xb[t], ir[t]);
                }
            };
#pragma unroll
            for (int h = 0; h < B / 2; ++h) {
                const pd2 xa = left_pair(pa, h);
                const pd2 xai = AC ? left_pair(pai, h) : pd2{0, 0};
                pd2 xb[NJ], xbi[NJ];
#pragma unroll
                for (int t = 0; t < NJ; ++t) {
                    xb[t] = xbi[t] = pd2{0, 0};
                    if (!((ACT >> t) & 1)) continue;
                    xb[t] = right_pair(pb[t], h);
                    if (BC) xbi[t] = right_pair(pbi[t], h);
                }
                const double b0[NJ] = {xb[0].x, xb[1].x}, b0i[NJ] = {xbi[0].x, xbi[1].x};
                const double b1[NJ] = {xb[0].y, xb[1].y}, b1i[NJ] = {xbi[0].y, xbi[1].y};
                mma(xa.x, xai.x, b0, b0i);
                mma(xa.y, xai.y, b1, b1i);
            }
            {
                const int oa = last_left(), ob = last_right();
                const double xa = pa[oa], xai = AC ? pai[oa] : 0.0;
                double xb[NJ] = {0, 0}, xbi[NJ] = {0, 0};
#pragma unroll
                for (int t = 0; t < NJ; ++t) {
                    if (!((ACT >> t) & 1)) continue;
                    xb[t] = pb[t][ob];
                    if (BC) xbi[t] = pbi[t][ob];
                }
                mma(xa, xai, xb, xbi);
            }
        }
    };
    if constexpr (SEG) {
        const int nf = seg[2 * c], n0 = seg[2 * c + 1];   // uniform across the wave
        groups(0, nf, std::integral_constant<int, 3>());
        groups(nf, nf + n0, std::integral_constant<int, 1>());
        groups(nf + n0, ne, std::integral_constant<int, 2>());
    } else {
        groups(0, ne, std::integral_constant<int, 3>());
    }
    constexpr double sb = CJB ? -1.0 : 1.0;
    const int col = lane & 15;
#pragma unroll
    for (int t = 0; t < NJ; ++t) {
        const int p = cout[c * NJ + t];
        if (p < 0) continue;                   // uniform: a short run
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 4 * e + q;
            if (row < B && col < B) {
                const double re = rr[t][e] - sb * ii[t][e];
                const double im = sb * ri[t][e] + ir[t][e];
                const int64_t rm = (int64_t)p * BB + row * B + col;
                const int64_t o = OUT == 0   ? rm
                                  : OUT == 1 ? (int64_t)p * BB + pair_at(B, row, col)
                                             : (int64_t)p * BB + pair_at(B, col, row);
                const double vr = alr * re - ali * im;
                if (u) u[rm] = u_store ? u_sign * vr : u[rm] + u_sign * vr;
                if (cr) cr[o] = vr;
                if (ci) ci[o] = alr * im + ali * re;
            }
        }
    }
}

// Blocks into pair layout (kPackLeft, kPackRight) or back (kUnpackLeft).
__global__ __launch_bounds__(256) void k_pack_pairs13(int64_t n, int mode, const double *__restrict__ in,
                                                      double *__restrict__ out)
{
    constexpr int B = 13, BB = B * B;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
        const int64_t p = e / BB;
        const int w = (int)(e - p * BB);
        // (x, m) of element w of the pair layout
        const int x = w >= B * (B - 1) ? w - B * (B - 1) : (w % (2 * B)) >> 1;
        const int m = w >= B * (B - 1) ? B - 1 : 2 * (w / (2 * B)) + (w & 1);
        const int64_t rm = p * BB + (mode == kPackRight ? m * B + x : x * B + m);
        if (mode == kUnpackLeft) out[rm] = in[e];
        else out[e] = in[rm];
    }
}

void launch_pack_pairs(hipStream_t s, int64_t nblocks, int mode, const double *in, double *out)
{
    const int64_t n = nblocks * 169;
    if (n == 0) return;
    const int64_t g = std::min<int64_t>((n + 255) / 256, 65536);
    hipLaunchKernelGGL(k_pack_pairs13, dim3((unsigned)g), dim3(256), 0, s, n, mode, in, out);
    RT_HIP(hipGetLastError());
}

// Start of the Taylor sum from A (row-major blocks), one pass: tau = dt A as
// the right operand of the next product (b = 4: blocks transposed; b = 13:
// right pairs), u_im = -dt A, and at b = 13 the left pairs of A (ap).
template <int B, typename I>
__global__ __launch_bounds__(256) void k_taylor_start(I n, double dt, const double *__restrict__ a,
                                                      double *__restrict__ tau, double *__restrict__ u_im,
                                                      double *__restrict__ ap)
{
    constexpr int BB = B * B;
    for (I e = (I)blockIdx.x * 256 + threadIdx.x; e < n; e += (I)gridDim.x * 256) {
        const I p = e / BB;
        const int w = (int)(e - p * BB), r = w / B, c = w - r * B;
        const double v = a[e], t = dt * v;
        u_im[e] = -t;
        if (B == 4) {
            tau[p * BB + c * B + r] = t;
        } else {
            tau[p * BB + pair_at(B, c, r)] = t;
            ap[p * BB + pair_at(B, r, c)] = v;
        }
    }
}

void launch_taylor_start(hipStream_t s, int64_t nblocks, int b, double dt, const double *a, double *tau, double *u_im,
                         double *ap)
{
    const int64_t n = nblocks * b * b;
    if (n == 0) return;
    RT_CHECK(b == 4 || (b == 13 && ap), RTDM_E_ARG, "the Taylor start needs b = 4 or 13");
    const int64_t g = std::min<int64_t>((n + 255) / 256, 65536);
    const bool small = n + g * 256 < ((int64_t)1 << 32);   // 32-bit index arithmetic
#define RT_TS(B_, I_) \
    hipLaunchKernelGGL((k_taylor_start<B_, I_>), dim3((unsigned)g), dim3(256), 0, s, (I_)n, dt, a, tau, u_im, ap)
    if (b == 4 && small) RT_TS(4, uint32_t);
    else if (b == 4) RT_TS(4, int64_t);
    else if (small) RT_TS(13, uint32_t);
    else RT_TS(13, int64_t);
#undef RT_TS
    RT_HIP(hipGetLastError());
}

template <bool AC, bool BC, int CJB, int OUT, bool ROWS = false, bool SEG = true>
static void launch_q4p(hipStream_t s, const SpgemmArgs &a, const SumInto &u)
{
    const int remap = xcd_chunk_for((a.nch + 3) / 4);
    const unsigned grid = xcd_grid((a.nch + 3) / 4, remap);
    hipLaunchKernelGGL((k_spgemm_q4p<13, AC, BC, CJB, OUT, ROWS, SEG>), dim3(grid), dim3(256), 0, s, a.nch,
                       a.ch_off, a.ch_a, a.ch_b, a.ch_out, a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.alpha_re,
                       a.alpha_im, a.zero, a.ch_order, remap, a.ch_seg, u.p, u.sign, u.store);
}

// Products over row runs of 2 with both operands in pair layout (b = 13, FP64;
// a conjugated right operand U^dagger is the left pairs of U): conj_b, out
// (kOut*; right pairs and the fused sum u for real products only).  rows: both
// operands and the output by rows.  a.ch_seg null: entries without segments.
void launch_spgemm_pairs(hipStream_t s, const SpgemmArgs &a, int conj_b, int out, const SumInto &u, bool rows)
{
    RT_CHECK(a.b == 13 && a.precision == RTDM_PREC_FP64 && a.nj == 2 && a.nch > 0 && a.zero, RTDM_E_ARG,
             "pair-layout products need b = 13, FP64 and runs of 2");
    const bool ac = a.ai != nullptr, bc = a.bi != nullptr;
    if (!a.ch_seg) {
        RT_CHECK(ac && bc && !rows && !conj_b && out == kOutRows && !u.p, RTDM_E_ARG,
                 "runs without segments give a plain complex product by rows");
        launch_q4p<true, true, 0, 0, false, false>(s, a, u);
        RT_HIP(hipGetLastError());
        return;
    }
    const bool real = !ac && !bc && !a.ci;
    RT_CHECK(real || (!u.p && out != kOutRight), RTDM_E_ARG, "right pairs and the fused sum need real operands");
    if (rows) {
        RT_CHECK(!conj_b && out == kOutRows && !u.p, RTDM_E_ARG, "operands by rows give a plain product by rows");
        if (ac && bc) launch_q4p<true, true, 0, 0, true>(s, a, u);
        else if (ac) launch_q4p<true, false, 0, 0, true>(s, a, u);
        else if (bc) launch_q4p<false, true, 0, 0, true>(s, a, u);
        else launch_q4p<false, false, 0, 0, true>(s, a, u);
        RT_HIP(hipGetLastError());
        return;
    }
    if (real && out == kOutRight) {
        launch_q4p<false, false, 0, 2>(s, a, u);
        RT_HIP(hipGetLastError());
        return;
    }
    RT_CHECK(!conj_b || out == kOutRows, RTDM_E_ARG, "a conjugated right operand gives its product by rows");
#define RT_Q4P(AC_, BC_)                                                  \
    do {                                                                  \
        if (conj_b) launch_q4p<AC_, BC_, 1, 0>(s, a, u);                  \
        else if (out == kOutLeft) launch_q4p<AC_, BC_, 0, 1>(s, a, u);    \
        else launch_q4p<AC_, BC_, 0, 0>(s, a, u);                         \
    } while (0)
    if (ac && bc) RT_Q4P(true, true);
    else if (ac) RT_Q4P(true, false);
    else if (bc) RT_Q4P(false, true);
    else RT_Q4P(false, false);
#undef RT_Q4P
    RT_HIP(hipGetLastError());
}

// b = 4: v_mfma_f64_4x4x4_4b_f64 runs four independent 4x4x4 products, one
// per "MFMA block".  Each output block needs SUB real sub-products (1: real x
// real; 2: one operand complex; 4: complex x complex: re*re, im*im, re*im,
// im*re), so a wave serves 4/SUB output blocks, each on SUB MFMA blocks, with
// no padding anywhere: one instruction per step does one block triple of 4/SUB
// outputs.  Lane layout (measured on gfx950), lane = 16*q + 4*g + r:
//   MFMA block g; A operand A_g[r][q]; B operand B_g[q][r]; D: D_g[q][r].
// The wave's outputs advance in lock-step over their triple lists; a finished
// output feeds zeros.

// Split-precision block products (B = 4 or 13, operand layouts as in
// k_spgemm_kc).  Each FP64 operand element x is split into two 16-bit
// parts and the product of two elements is taken as three 16-bit products
// with FP32 accumulation on the matrix cores (v_mfma_f32_16x16x32_*):
//   MODE 0, BF16 x3 (the three-product split of Henry, Tang and Heinecke,
//     2019): hi = bf16(x), lo = bf16(x - hi); a b ~ ah bh + ah bl + al bh.
//   MODE 1, FP16 x2 (the scaled split of Ootomo and Yokota, 2022):
//     y = x s with s = 2^(13 - floor(log2 max|X|)) per operand matrix,
//     hi = fp16(y), lo = fp16((y - hi) 2^11);
//     a b ~ (ah bh + (ah bl + al bh) 2^-11) / (sa sb).
// The contraction of an output block is concatenated over its triples; a
// 32-wide MFMA step takes elements 8q..8q+7 of the step from lane group q.
// The sign of a conjugated operand's imaginary part is applied at the load.
template <int MODE> struct Split16;
template <> struct Split16<0> {
    typedef __bf16 v8 __attribute__((ext_vector_type(8)));
    static __device__ inline void split(double x, float, __bf16 &hi, __bf16 &lo)
    {
        float xf = (float)x;
        asm volatile("" : "+v"(xf));
        hi = (__bf16)xf;
        lo = (__bf16)(xf - (float)hi);
    }
    static __device__ inline f32x4 mfma(v8 a, v8 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    typedef __bf16 e_t;
};
template <> struct Split16<1> {
    typedef _Float16 v8 __attribute__((ext_vector_type(8)));
    static __device__ inline void split(double x, float sc, _Float16 &hi, _Float16 &lo)
    {
        const float y = (float)x * sc;
        hi = (_Float16)y;
        lo = (_Float16)((y - (float)hi) * 2048.0f);
    }
    static __device__ inline f32x4 mfma(v8 a, v8 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
    typedef _Float16 e_t;
};

// Power-of-two operand scale of the FP16 split from max |X| (both planes).
__device__ inline float f16_scale(const double *mx, int k)
{
    const double m = fmax(mx[8 * k + 3], mx[8 * k + 7]);
    return m > 0.0 ? ldexpf(1.0f, 13 - ilogb(m)) : 1.0f;
}

template <int B, bool AC, bool BC, int TA, int TB, int MODE>
__global__ __launch_bounds__(256) void k_spgemm_split(
    int64_t nout, const int64_t *__restrict__ off, const int2 *__restrict__ trip,
    const double *__restrict__ ar, const double *__restrict__ ai, const double *__restrict__ br,
    const double *__restrict__ bi, double *__restrict__ cr, double *__restrict__ ci, double alr,
    double ali, const double *__restrict__ maxabs)
{
    typedef Split16<MODE> SP;
    typedef typename SP::v8 v8;
    constexpr int BB = B * B;
    const int lane = threadIdx.x & 63;
    const int64_t c = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (c >= nout) return;                     // uniform across the wave
    const int r = lane & 15, q = lane >> 4;
    const bool rv = r < B;
    const int64_t t0 = off[c];
    const int nt = (int)(off[c + 1] - t0);
    const int L = nt * B;
    const float sa = MODE ? f16_scale(maxabs, 0) : 1.0f;
    const float sb = MODE ? f16_scale(maxabs, 1) : 1.0f;
    f32x4 h[4] = {}, m[4] = {};                // rr, ii, ri, ir: hi*hi and the mixed terms
    for (int u0 = 0; u0 < L; u0 += 32) {
        v8 ahr, alr8, ahi, ali8, bhr, blr8, bhi, bli8;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const int u = u0 + 8 * q + v;
            double xar = 0.0, xai = 0.0, xbr = 0.0, xbi = 0.0;
            if (rv && u < L) {
                const int tt = u / B, k = u - tt * B;
                const int2 ab = trip[t0 + tt];
                const int64_t pa = (int64_t)ab.x * BB + (TA ? k * B + r : r * B + k);
                const int64_t pb = (int64_t)ab.y * BB + (TB ? r * B + k : k * B + r);
                xar = ar[pa];
                xbr = br[pb];
                if (AC) xai = TA ? -ai[pa] : ai[pa];
                if (BC) xbi = TB ? -bi[pb] : bi[pb];
            }
            typename SP::e_t hi, lo;
            SP::split(xar, sa, hi, lo); ahr[v] = hi; alr8[v] = lo;
            SP::split(xbr, sb, hi, lo); bhr[v] = hi; blr8[v] = lo;
            if (AC) { SP::split(xai, sa, hi, lo); ahi[v] = hi; ali8[v] = lo; }
            if (BC) { SP::split(xbi, sb, hi, lo); bhi[v] = hi; bli8[v] = lo; }
        }
        auto prod3 = [&](int k, const v8 &ah, const v8 &al, const v8 &bh, const v8 &bl) {
            h[k] = SP::mfma(ah, bh, h[k]);
            m[k] = SP::mfma(ah, bl, m[k]);
            m[k] = SP::mfma(al, bh, m[k]);
        };
        prod3(0, ahr, alr8, bhr, blr8);
        if (AC && BC) prod3(1, ahi, ali8, bhi, bli8);
        if (BC) prod3(2, ahr, alr8, bhi, bli8);
        if (AC) prod3(3, ahi, ali8, bhr, blr8);
    }
    const double inv = 1.0 / ((double)sa * (double)sb);
    const double ml = MODE ? 1.0 / 2048.0 : 1.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int row = 4 * q + e, col = r;
        if (row < B && col < B) {
            double v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = ((double)h[k][e] + ml * (double)m[k][e]) * inv;
            const double re = v[0] - v[1];
            const double im = v[2] + v[3];
            const int64_t o = c * BB + row * B + col;
            cr[o] = alr * re - ali * im;
            if (ci) ci[o] = alr * im + ali * re;
        }
    }
}

// Split-precision variant of k_spgemm_q4 for real operands (the Taylor-term
// products A tau of the *_TAYLOR forms), same four-triple grouping, order and
// XCD mapping.  Each 16-bit MFMA (v_mfma_f32_16x16x16_{bf16,f16}) step takes
// four consecutive contraction elements s0..s0+3 of its triple from lane
// group q, so four steps cover B = 13 (elements 13..15 are zero).  Every
// FP64 element is split as in k_spgemm_split (BF16 hi/lo, or FP16 hi/lo of
// the power-of-two scaled value with the low part scaled by 2^11) and each
// product is taken as hi*hi + hi*lo + lo*hi with FP32 accumulation.
template <int MODE> struct Split4;
template <> struct Split4<0> {
    typedef short v4 __attribute__((ext_vector_type(4)));
    static __device__ inline void split(double x, float, short &hi, short &lo)
    {
        float xf = (float)x;                       // 24 bits hold both 8-bit parts
        asm volatile("" : "+v"(xf));               // round to FP32 first: keeps the conversions apart
        const __bf16 h = (__bf16)xf;
        const __bf16 l = (__bf16)(xf - (float)h);
        hi = __builtin_bit_cast(short, h);
        lo = __builtin_bit_cast(short, l);
    }
    static __device__ inline f32x4 mfma(v4 a, v4 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
    }
    typedef short e_t;
};
template <> struct Split4<1> {
    typedef _Float16 v4 __attribute__((ext_vector_type(4)));
    static __device__ inline void split(double x, float sc, _Float16 &hi, _Float16 &lo)
    {
        const float y = (float)x * sc;              // sc a power of two; 24 bits hold both 11-bit parts
        hi = (_Float16)y;
        lo = (_Float16)((y - (float)hi) * 2048.0f);
    }
    static __device__ inline f32x4 mfma(v4 a, v4 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0);
    }
    typedef _Float16 e_t;
};

template <int B, int MODE, int WPB>
__global__ __launch_bounds__(64 * WPB) void k_spgemm_q4s(
    int64_t nout, const int64_t *__restrict__ off, const int2 *__restrict__ trip, const double *__restrict__ ar,
    const double *__restrict__ br, double *__restrict__ cr, double alr, const double *__restrict__ zero,
    const int32_t *__restrict__ order, const double *__restrict__ maxabs, int remap)
{
    typedef Split4<MODE> SP;
    typedef typename SP::v4 v4;
    constexpr int BB = B * B;
    const int lane = threadIdx.x & 63;
    const int64_t w = xcd_block((nout + WPB - 1) / WPB, remap) * WPB + (threadIdx.x >> 6);
    if (w >= nout) return;                     // uniform across the wave
    const int64_t c = order ? (int64_t)order[w] : w;
    const int r = lane & 15, q = lane >> 4;
    const bool rv = r < B;
    const int64_t t0 = off[c];
    const int nt = (int)(off[c + 1] - t0);
    const float sa = MODE ? f16_scale(maxabs, 0) : 1.0f;
    const float sb = MODE ? f16_scale(maxabs, 1) : 1.0f;
    f32x4 h = {0, 0, 0, 0}, m = {0, 0, 0, 0};
    for (int g = 0; g < nt; g += 4) {
        const double *pa = zero, *pb = zero;
        if (rv && g + q < nt) {
            const int2 ab = trip[t0 + g + q];
            pa = ar + (int64_t)ab.x * BB + r;
            pb = br + (int64_t)ab.y * BB + r;
        }
#pragma unroll
        for (int s0 = 0; s0 < B; s0 += 4) {
            v4 ah, al, bh, bl;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int st = s0 + v;
                const double xa = st < B ? pa[st * B] : 0.0, xb = st < B ? pb[st * B] : 0.0;
                typename SP::e_t hi, lo;
                SP::split(xa, sa, hi, lo);
                ah[v] = hi;
                al[v] = lo;
                SP::split(xb, sb, hi, lo);
                bh[v] = hi;
                bl[v] = lo;
            }
            h = SP::mfma(ah, bh, h);
            m = SP::mfma(ah, bl, m);
            m = SP::mfma(al, bh, m);
        }
    }
    const double inv = 1.0 / ((double)sa * (double)sb);
    const double ml = MODE ? 1.0 / 2048.0 : 1.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int row = 4 * q + e, col = r;
        if (row < B && col < B) cr[c * BB + row * B + col] = alr * (((double)h[e] + ml * (double)m[e]) * inv);
    }
}

void launch_spgemm_cm_split(hipStream_t s, const SpgemmArgs &a)
{
    if (a.nout == 0) return;
    RT_CHECK(a.b == 13 && !a.ai && !a.bi && !a.ci &&
                 (a.precision == RTDM_PREC_BF16X3 || a.precision == RTDM_PREC_FP16X2),
             RTDM_E_UNSUPPORTED, "split step products need b = 13, real operands and a split precision");
    RT_CHECK(a.precision != RTDM_PREC_FP16X2 || a.maxabs, RTDM_E_ARG, "FP16 split products need operand maxima");
    const int wpb = a.wpb;
    const int remap = xcd_chunk_wg(wpb);
    const unsigned grid = xcd_grid((a.nout + wpb - 1) / wpb, remap);
#define RT_Q4S(M, W)                                                                                      \
    hipLaunchKernelGGL((k_spgemm_q4s<13, M, W>), dim3(grid), dim3(64 * W), 0, s, a.nout, a.off, a.trip, a.ar, \
                       a.br, a.cr, a.alpha_re, a.zero, a.order, a.maxabs, remap)
    const int mode = a.precision == RTDM_PREC_FP16X2 ? 1 : 0;
    if (mode == 0) {
        if (wpb == 16) RT_Q4S(0, 16);
        else if (wpb == 8) RT_Q4S(0, 8);
        else RT_Q4S(0, 4);
    } else {
        if (wpb == 16) RT_Q4S(1, 16);
        else if (wpb == 8) RT_Q4S(1, 8);
        else RT_Q4S(1, 4);
    }
#undef RT_Q4S
    RT_HIP(hipGetLastError());
}

template <int SUB, bool AC, bool BC, int OPA, int OPB>
__global__ __launch_bounds__(256) void k_spgemm_b4(
    int64_t nout, const int64_t *__restrict__ off, const int2 *__restrict__ trip,
    const double *__restrict__ ar, const double *__restrict__ ai, const double *__restrict__ br,
    const double *__restrict__ bi, double *__restrict__ cr, double *__restrict__ ci, double alr,
    double ali)
{
    constexpr int OUT = 4 / SUB;               // outputs per wave
    const int lane = threadIdx.x & 63;
    const int g = (lane >> 2) & 3, r = lane & 3, q = lane >> 4;
    const int sub = g % SUB;                   // which real sub-product this MFMA block runs
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t c0 = wave * OUT;
    if (c0 >= nout) return;                    // uniform across the wave
    const int64_t c = c0 + g / SUB;            // this lane's output block
    const bool live = c < nout;
    const int64_t t0 = live ? off[c] : 0;
    const int nt = live ? (int)(off[c + 1] - t0) : 0;
    // longest list of the wave (the four MFMA blocks sit 4 lanes apart)
    int ntmax = max(nt, __shfl_xor(nt, 4, 64));
    ntmax = max(ntmax, __shfl_xor(ntmax, 8, 64));
    // operand planes of this sub-product: sub 0 re*re, 1 im*im, 2 re*im, 3 im*re (SUB = 4);
    // SUB = 2: sub 0 re*re, sub 1 the product with the complex operand's imaginary part.
    bool a_im = false, b_im = false;
    if (SUB == 4) { a_im = (sub == 1 || sub == 3); b_im = (sub == 1 || sub == 2); }
    if (SUB == 2) { a_im = AC && sub == 1; b_im = BC && sub == 1; }
    const double *pa = a_im ? ai : ar;
    const double *pb = b_im ? bi : br;
    const double sa = (a_im && OPA) ? -1.0 : 1.0;
    const double sb = (b_im && OPB) ? -1.0 : 1.0;
    const int ia = OPA ? (q * 4 + r) : (r * 4 + q);   // op(A)[r][q]
    const int ib = OPB ? (r * 4 + q) : (q * 4 + r);   // op(B)[q][r]
    double acc = 0.0;
    double xa = 0.0, xb = 0.0;
    if (nt > 0) {
        const int2 ab = trip[t0];
        xa = sa * pa[(int64_t)ab.x * 16 + ia];
        xb = sb * pb[(int64_t)ab.y * 16 + ib];
    }
    for (int t = 0; t < ntmax; ++t) {
        double na = 0.0, nb = 0.0;
        if (t + 1 < nt) {
            const int2 ab = trip[t0 + t + 1];
            na = sa * pa[(int64_t)ab.x * 16 + ia];
            nb = sb * pb[(int64_t)ab.y * 16 + ib];
        }
        acc = __builtin_amdgcn_mfma_f64_4x4x4f64(xa, xb, acc, 0, 0, 0);
        xa = na;
        xb = nb;
    }
    // combine the sub-products of each output (MFMA blocks are 4 lanes apart)
    double re = acc, im = 0.0;
    if (SUB == 4) {
        const double d1 = __shfl_down(acc, 4, 64);    // block g+1
        const double d2 = __shfl_down(acc, 8, 64);    // block g+2
        const double d3 = __shfl_down(acc, 12, 64);   // block g+3
        re = acc - d1;
        im = d2 + d3;
    } else if (SUB == 2) {
        im = __shfl_down(acc, 4, 64);
    }
    if (live && sub == 0) {
        const int64_t o = c * 16 + q * 4 + r;
        cr[o] = alr * re - ali * im;
        if (ci) ci[o] = alr * im + ali * re;
    }
}




// Reduced-precision products for b = 4 on the 16-block 4x4 matrix-core
// instructions (gfx950, measured layout: lane 4 blk + r supplies row r of
// A_blk and column r of B_blk, and holds D_blk[e][r] in its value e).  A wave
// runs 16 output blocks, one per MFMA block, one triple of each per step:
//   MODE 0 FP32   : four v_mfma_f32_4x4x1_16b per block product;
//   MODE 1 BF16x3 : hi/lo split, three v_mfma_f32_4x4x4_16b_bf16;
//   MODE 2 FP16x2 : scaled hi/lo split, three v_mfma_f32_4x4x4_16b_f16.
// Operands are FP64 in memory (op(A) = A; op(B) = B or B^dagger), results
// FP64; accumulation FP32.
template <int MODE> struct Small4;
template <> struct Small4<1> {
    typedef short v4 __attribute__((ext_vector_type(4)));
    static __device__ inline f32x4 mfma(v4 a, v4 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(a, b, c, 0, 0, 0);
    }
    static __device__ inline void split(double x, float, short &hi, short &lo) { Split4<0>::split(x, 1.0f, hi, lo); }
    typedef short e_t;
};
template <> struct Small4<2> {
    typedef _Float16 v4 __attribute__((ext_vector_type(4)));
    static __device__ inline f32x4 mfma(v4 a, v4 b, f32x4 c)
    {
        return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 0, 0, 0);
    }
    static __device__ inline void split(double x, float sc, _Float16 &hi, _Float16 &lo)
    {
        Split4<1>::split(x, sc, hi, lo);
    }
    typedef _Float16 e_t;
};

//
// RUNS: the wave computes a row run of 16 outputs (SpgemmArgs::ch_*, b = 4
// slot order) instead of 16 consecutive outputs: all blocks share the entry's
// op(A)_ik, and block blk takes the op(B)_kj of output blk (zero if absent).
template <bool AC, bool BC, int OPB, int MODE, bool RUNS = false>
__global__ __launch_bounds__(256) void k_spgemm_b4x(
    int64_t nout, const int64_t *__restrict__ off, const int2 *__restrict__ trip,
    const double *__restrict__ ar, const double *__restrict__ ai, const double *__restrict__ br,
    const double *__restrict__ bi, double *__restrict__ cr, double *__restrict__ ci, double alr, double ali,
    const double *__restrict__ maxabs, const int32_t *__restrict__ ea = nullptr,
    const int32_t *__restrict__ eb = nullptr, const int32_t *__restrict__ rout = nullptr)
{
    const int lane = threadIdx.x & 63;
    const int blk = lane >> 2, r = lane & 3;
    // RUNS: nout is the number of runs, off the entry offsets
    const int64_t wv = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t c0 = RUNS ? wv : wv * 16;
    if (c0 >= nout) return;                    // uniform across the wave
    const int64_t c = RUNS ? (int64_t)rout[wv * 16 + blk] : c0 + blk;
    const bool live = RUNS ? c >= 0 : c < nout;
    const int64_t t0 = RUNS ? off[wv] : (live ? off[c] : 0);
    const int nt = RUNS ? (int)(off[wv + 1] - t0) : (live ? (int)(off[c + 1] - t0) : 0);
    int ntmax = nt;
    if (!RUNS) {
#pragma unroll
        for (int o = 4; o < 64; o <<= 1) ntmax = max(ntmax, __shfl_xor(ntmax, o, 64));
    }
    const int slot = (blk & 3) * 4 + (blk >> 2);
    const float sa = MODE == 2 ? f16_scale(maxabs, 0) : 1.0f;
    const float sb = MODE == 2 ? f16_scale(maxabs, 1) : 1.0f;
    f32x4 h[4] = {}, m[4] = {};                // rr, ii, ri, ir
    const double cb = OPB ? -1.0 : 1.0;
    for (int t = 0; t < ntmax; ++t) {
        double xa[4] = {0, 0, 0, 0}, xai[4] = {0, 0, 0, 0}, xb[4] = {0, 0, 0, 0}, xbi[4] = {0, 0, 0, 0};
        int2 ab = make_int2(0, -1);
        if (RUNS) ab = make_int2(ea[t0 + t], eb[(t0 + t) * 16 + slot]);
        else if (t < nt) ab = trip[t0 + t];
        if (ab.y >= 0) {
            const int64_t pa = (int64_t)ab.x * 16 + r * 4, pb = (int64_t)ab.y * 16;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                xa[k] = ar[pa + k];                                    // A[r][k]
                const int64_t e = OPB ? pb + r * 4 + k : pb + k * 4 + r; // op(B)[k][r]
                xb[k] = br[e];
                if (AC) xai[k] = ai[pa + k];
                if (BC) xbi[k] = cb * bi[e];
            }
        }
        if (MODE == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                h[0] = __builtin_amdgcn_mfma_f32_4x4x1f32((float)xa[k], (float)xb[k], h[0], 0, 0, 0);
                if (AC && BC) h[1] = __builtin_amdgcn_mfma_f32_4x4x1f32((float)xai[k], (float)xbi[k], h[1], 0, 0, 0);
                if (BC) h[2] = __builtin_amdgcn_mfma_f32_4x4x1f32((float)xa[k], (float)xbi[k], h[2], 0, 0, 0);
                if (AC) h[3] = __builtin_amdgcn_mfma_f32_4x4x1f32((float)xai[k], (float)xb[k], h[3], 0, 0, 0);
            }
        } else {
            typedef Small4<MODE == 0 ? 1 : MODE> SP;
            typedef typename SP::v4 v4;
            auto prod3 = [&](int u, const double *x, float sx, const double *y, float sy) {
                v4 xh, xl, yh, yl;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    typename SP::e_t hi, lo;
                    SP::split(x[k], sx, hi, lo);
                    xh[k] = hi;
                    xl[k] = lo;
                    SP::split(y[k], sy, hi, lo);
                    yh[k] = hi;
                    yl[k] = lo;
                }
                h[u] = SP::mfma(xh, yh, h[u]);
                m[u] = SP::mfma(xh, yl, m[u]);
                m[u] = SP::mfma(xl, yh, m[u]);
            };
            prod3(0, xa, sa, xb, sb);
            if (AC && BC) prod3(1, xai, sa, xbi, sb);
            if (BC) prod3(2, xa, sa, xbi, sb);
            if (AC) prod3(3, xai, sa, xb, sb);
        }
    }
    if (!live) return;
    const double inv = 1.0 / ((double)sa * (double)sb);
    const double ml = MODE == 2 ? 1.0 / 2048.0 : (MODE == 1 ? 1.0 : 0.0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = ((double)h[u][e] + ml * (double)m[u][e]) * inv;
        const double re = v[0] - v[1], im = v[2] + v[3];
        const int64_t o = c * 16 + e * 4 + r;
        cr[o] = alr * re - ali * im;
        if (ci) ci[o] = alr * im + ali * re;
    }
}

template <bool AC, bool BC, int OB>
static void launch_b4x(hipStream_t s, const SpgemmArgs &a)
{
    if (a.nch > 0) {
        RT_CHECK(a.nj == 16, RTDM_E_ARG, "b = 4 row runs hold 16 outputs");
        const dim3 g((unsigned)((a.nch + 3) / 4)), t(256);
#define RT_B4XJ(M)                                                                                      \
    hipLaunchKernelGGL((k_spgemm_b4x<AC, BC, OB, M, true>), g, t, 0, s, a.nch, a.ch_off, a.trip, a.ar, a.ai, \
                       a.br, a.bi, a.cr, a.ci, a.alpha_re, a.alpha_im, a.maxabs, a.ch_a, a.ch_b, a.ch_out)
        if (a.precision == RTDM_PREC_FP32) RT_B4XJ(0);
        else if (a.precision == RTDM_PREC_BF16X3) RT_B4XJ(1);
        else RT_B4XJ(2);
#undef RT_B4XJ
        return;
    }
    const dim3 g((unsigned)((a.nout + 63) / 64)), t(256);
#define RT_B4X(M)                                                                                     \
    hipLaunchKernelGGL((k_spgemm_b4x<AC, BC, OB, M>), g, t, 0, s, a.nout, a.off, a.trip, a.ar, a.ai, a.br, \
                       a.bi, a.cr, a.ci, a.alpha_re, a.alpha_im, a.maxabs)
    if (a.precision == RTDM_PREC_FP32) RT_B4X(0);
    else if (a.precision == RTDM_PREC_BF16X3) RT_B4X(1);
    else RT_B4X(2);
#undef RT_B4X
}


// FP64 b = 4 product, 16 output blocks per wave: four v_mfma_f64_4x4x4_4b per
// triple step (instruction j runs outputs c0 + 4j + g in its four blocks), so
// every lane has eight (real) operand loads in flight per step instead of
// two.  Same operand bytes per triple as k_spgemm_b4.
template <bool AC, bool BC, int OPB>
__global__ __launch_bounds__(256) void k_spgemm_b4w(
    int64_t nout, const int64_t *__restrict__ off, const int2 *__restrict__ trip,
    const double *__restrict__ ar, const double *__restrict__ ai, const double *__restrict__ br,
    const double *__restrict__ bi, double *__restrict__ cr, double *__restrict__ ci, double alr, double ali)
{
    const int lane = threadIdx.x & 63;
    const int g = (lane >> 2) & 3, r = lane & 3, q = lane >> 4;
    const int64_t c0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16;
    if (c0 >= nout) return;                    // uniform across the wave
    const int ia = r * 4 + q;                          // A[r][q]
    const int ib = OPB ? (r * 4 + q) : (q * 4 + r);    // op(B)[q][r]
    const double cb = OPB ? -1.0 : 1.0;
    int64_t t0[4];
    int nt[4];
    int ntmax = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int64_t c = c0 + 4 * j + g;
        t0[j] = c < nout ? off[c] : 0;
        nt[j] = c < nout ? (int)(off[c + 1] - t0[j]) : 0;
        ntmax = max(ntmax, nt[j]);
    }
    ntmax = max(ntmax, __shfl_xor(ntmax, 4, 64));
    ntmax = max(ntmax, __shfl_xor(ntmax, 8, 64));
    double rr[4] = {0, 0, 0, 0}, ii[4] = {0, 0, 0, 0}, ri[4] = {0, 0, 0, 0}, ir[4] = {0, 0, 0, 0};
    for (int t = 0; t < ntmax; ++t) {
        double xar[4], xai[4], xbr[4], xbi[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            xar[j] = xai[j] = xbr[j] = xbi[j] = 0.0;
            if (t < nt[j]) {
                const int2 ab = trip[t0[j] + t];
                const int64_t pa = (int64_t)ab.x * 16 + ia, pb = (int64_t)ab.y * 16 + ib;
                xar[j] = ar[pa];
                xbr[j] = br[pb];
                if (AC) xai[j] = ai[pa];
                if (BC) xbi[j] = cb * bi[pb];
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            rr[j] = __builtin_amdgcn_mfma_f64_4x4x4f64(xar[j], xbr[j], rr[j], 0, 0, 0);
            if (AC && BC) ii[j] = __builtin_amdgcn_mfma_f64_4x4x4f64(xai[j], xbi[j], ii[j], 0, 0, 0);
            if (BC) ri[j] = __builtin_amdgcn_mfma_f64_4x4x4f64(xar[j], xbi[j], ri[j], 0, 0, 0);
            if (AC) ir[j] = __builtin_amdgcn_mfma_f64_4x4x4f64(xai[j], xbr[j], ir[j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int64_t c = c0 + 4 * j + g;
        if (c < nout) {
            const double re = rr[j] - ii[j], im = ri[j] + ir[j];
            const int64_t o = c * 16 + q * 4 + r;
            cr[o] = alr * re - ali * im;
            if (ci) ci[o] = alr * im + ali * re;
        }
    }
}

// The entries [e0, e1) (every `stride`-th) of one b = 4 row run
// (SpgemmArgs::ch_*) with both operands by rows.  Each entry k of the run is
// one triple step: every lane loads the same op(A)_ik element position (one
// block for the whole wave) and the op(B)_kj elements of its four outputs
// (zero where an output has no triple with this k); instruction jj of the
// four v_mfma_f64_4x4x4_4b runs outputs 4 jj + g in its blocks g.  Software
// pipelined: the indices of entry e + 2 and the operands of entry e + 1 are
// requested before the products of entry e (the loads return in order, so
// waiting for an entry's operands never waits for later requests).
template <bool AC, bool BC>
__device__ inline void b4_run_entries(int64_t e0, int64_t e1, int stride, const int32_t *__restrict__ ea,
                                      const int32_t *__restrict__ eb, const double *__restrict__ ar,
                                      const double *__restrict__ ai, const double *__restrict__ br,
                                      const double *__restrict__ bi, int ia, int ib, int g, double rr[4],
                                      double ii[4], double ri[4], double ir[4])
{
    struct Ops {
        double xar, xai, xbr[4], xbi[4];
    };
    auto load_idx = [&](int64_t e, int &a, int4 &kb) {
        a = ea[e];
        kb = *reinterpret_cast<const int4 *>(eb + e * 16 + g * 4);
    };
    auto load_ops = [&](int a, int4 kb4, Ops &o) {
        const int64_t pa = (int64_t)a * 16 + ia;
        o.xar = ar[pa];
        o.xai = AC ? ai[pa] : 0.0;
        const int kb[4] = {kb4.x, kb4.y, kb4.z, kb4.w};
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            o.xbr[jj] = o.xbi[jj] = 0.0;
            if (kb[jj] >= 0) {
                const int64_t pb = (int64_t)kb[jj] * 16 + ib;
                o.xbr[jj] = br[pb];
                if (BC) o.xbi[jj] = bi[pb];
            }
        }
    };
    if (e0 >= e1) return;
    Ops cur, nxt;
    int a_n = 0;
    int4 kb_n = make_int4(-1, -1, -1, -1);
    {
        int a0;
        int4 k0;
        load_idx(e0, a0, k0);
        if (e0 + stride < e1) load_idx(e0 + stride, a_n, kb_n);
        load_ops(a0, k0, cur);
    }
    for (int64_t e = e0; e < e1; e += stride) {
        int a_nn = 0;
        int4 kb_nn = make_int4(-1, -1, -1, -1);
        if (e + 2 * stride < e1) load_idx(e + 2 * stride, a_nn, kb_nn);
        if (e + stride < e1) load_ops(a_n, kb_n, nxt);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            rr[jj] = __builtin_amdgcn_mfma_f64_4x4x4f64(cur.xar, cur.xbr[jj], rr[jj], 0, 0, 0);
            if (AC && BC) ii[jj] = __builtin_amdgcn_mfma_f64_4x4x4f64(cur.xai, cur.xbi[jj], ii[jj], 0, 0, 0);
            if (BC) ri[jj] = __builtin_amdgcn_mfma_f64_4x4x4f64(cur.xar, cur.xbi[jj], ri[jj], 0, 0, 0);
            if (AC) ir[jj] = __builtin_amdgcn_mfma_f64_4x4x4f64(cur.xai, cur.xbr[jj], ir[jj], 0, 0, 0);
        }
        cur = nxt;
        a_n = a_nn;
        kb_n = kb_nn;
    }
}

// Below this many runs a product takes the split form (one run per
// workgroup): a wave per run would leave most of the 1,024 SIMDs idle.  Below
// kB4Split8Runs the runs are split over 8 waves instead of 4 (16 measured no
// faster on the 64-atom cluster).
constexpr int64_t kB4SplitRuns = 4096, kB4Split8Runs = 1024;

bool b4_split_form(int64_t nch) { return nch < kB4SplitRuns; }

// FP64 b = 4 product over row runs of 16 outputs from operands whose lanes
// take 16 bytes: A row-major, B with every block transposed (bt), so that
// lane 16 q + 4 g + r reads A[r][2h], A[r][2h + 1] and B[2h][r], B[2h + 1][r]
// (h = q & 1) of entry e + (q >> 1) of a pair of entries.  One
// v_mfma_f64_4x4x4_4b then contracts over the even rows of both entries, a
// second one over the odd rows.  A conjugate-transposed right operand in
// row-major blocks is such a B as it is (CJB).
//
// Bound: the loads of k_spgemm_b4j (8 bytes a lane) kept the vector-memory
// address unit busy 99 % of the time at one entry per seven of them; a 16-byte
// load whose lane quads stay inside a block takes the same 15 cycles, and the
// entry's 16 block indices come as one 4-byte load (5 cycles) spread over the
// quad: per pair of entries 7 loads (real) in place of 14.  With the address
// unit relieved the L2 hit rate counts, and the chunked XCD deal pays (hardware
// order: A tau 2.8, U K 6.5 ms).  32,768 atoms, R_K 12, ms per launch, 8-byte
// loads -> now: A tau 4.3 -> 2.6 (0.2 of it the transposition of tau),
// U K 7.5 -> 5.3 (0.3 transposing K), W U^dagger 7.5 -> 5.0.
//
// b4p_entries: the pairs of entries e0, e0 + stride, ... below e1 into the sums
// rr, ii, ri, ir of the wave's 16 outputs; PIPE: the next pair's operands are
// requested before this pair's products (else only its indices).  BROWS: B's
// blocks by rows, two 8-byte loads in place of one of 16, for products without a
// buffer to transpose B into; the same products in the same order.
template <bool AC, bool BC, bool PIPE, bool BROWS = false>
__device__ inline void b4p_entries(int64_t e0, int64_t e1, int stride, const int32_t *__restrict__ ea,
                                   const int32_t *__restrict__ eb, const double *__restrict__ ar,
                                   const double *__restrict__ ai, const double *__restrict__ br,
                                   const double *__restrict__ bi, double (&rr)[4], double (&ii)[4], double (&ri)[4],
                                   double (&ir)[4])
{
    const int lane = threadIdx.x & 63;
    const int g = (lane >> 2) & 3, r = lane & 3, q = lane >> 4;
    const int lo = r * 4 + 2 * (q & 1), eo = q >> 1, slot = g * 4 + r;
    typedef double d2 __attribute__((ext_vector_type(2)));
    const int lob = BROWS ? 8 * (q & 1) + r : lo;
    auto pair_of = [&](const double *m, int64_t p) {
        return BROWS ? d2{m[p], m[p + 4]} : *reinterpret_cast<const d2 *>(m + p);
    };
    struct Ops {
        d2 xar, xai, xbr[4], xbi[4];
    };
    struct Idx {
        int a, b;
    };
    auto load_idx = [&](int64_t e) {
        Idx x{-1, -1};
        if (e + eo < e1) {
            x.a = ea[e + eo];
            x.b = eb[(e + eo) * 16 + slot];
        }
        return x;
    };
    auto load_ops = [&](Idx x, Ops &o) {
        o.xar = o.xai = d2{0, 0};
        if (x.a >= 0) {
            const int64_t pa = (int64_t)x.a * 16 + lo;
            o.xar = *reinterpret_cast<const d2 *>(ar + pa);
            if (AC) o.xai = *reinterpret_cast<const d2 *>(ai + pa);
        }
        // slot g * 4 + jj of the entry sits in lane r = jj of the quad
        const int kb[4] = {__builtin_amdgcn_mov_dpp(x.b, 0x00, 0xf, 0xf, true),
                           __builtin_amdgcn_mov_dpp(x.b, 0x55, 0xf, 0xf, true),
                           __builtin_amdgcn_mov_dpp(x.b, 0xaa, 0xf, 0xf, true),
                           __builtin_amdgcn_mov_dpp(x.b, 0xff, 0xf, 0xf, true)};
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            o.xbr[jj] = o.xbi[jj] = d2{0, 0};
            if (kb[jj] >= 0) {
                const int64_t pb = (int64_t)kb[jj] * 16 + lob;
                o.xbr[jj] = pair_of(br, pb);
                if (BC) o.xbi[jj] = pair_of(bi, pb);
            }
        }
    };
    auto mma1 = [&](double xa, double xi, double yr, double yi, double &srr, double &sri, double &sii, double &sir) {
        srr = __builtin_amdgcn_mfma_f64_4x4x4f64(xa, yr, srr, 0, 0, 0);
        if (AC && BC) sii = __builtin_amdgcn_mfma_f64_4x4x4f64(xi, yi, sii, 0, 0, 0);
        if (BC) sri = __builtin_amdgcn_mfma_f64_4x4x4f64(xa, yi, sri, 0, 0, 0);
        if (AC) sir = __builtin_amdgcn_mfma_f64_4x4x4f64(xi, yr, sir, 0, 0, 0);
    };
    auto products = [&](const Ops &o) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
            mma1(o.xar.x, o.xai.x, o.xbr[jj].x, o.xbi[jj].x, rr[jj], ri[jj], ii[jj], ir[jj]);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
            mma1(o.xar.y, o.xai.y, o.xbr[jj].y, o.xbi[jj].y, rr[jj], ri[jj], ii[jj], ir[jj]);
    };
    if constexpr (PIPE) {
        Ops cur, nxt;
        Idx n1 = load_idx(e0 + stride);
        load_ops(load_idx(e0), cur);
        for (int64_t e = e0; e < e1; e += stride) {
            const Idx n2 = load_idx(e + 2 * stride);
            load_ops(n1, nxt);
            products(cur);
            cur = nxt;
            n1 = n2;
        }
    } else {
        Idx n1 = load_idx(e0);
        for (int64_t e = e0; e < e1; e += stride) {
            Ops o;
            load_ops(n1, o);
            n1 = load_idx(e + stride);
            products(o);
        }
    }
}

// One element of output block p: alpha times the sums, row-major or with the
// block transposed (OUT), and into the fused sum u.
template <int CJB, int OUT>
__device__ inline void b4p_store(int p, double rr, double ii, double ri, double ir, double *__restrict__ cr,
                                 double *__restrict__ ci, double alr, double ali, double *__restrict__ u,
                                 double u_sign, int u_store)
{
    const int lane = threadIdx.x & 63, r = lane & 3, q = lane >> 4;
    const int64_t rm = (int64_t)p * 16 + q * 4 + r, tr = (int64_t)p * 16 + r * 4 + q;
    constexpr double sb = CJB ? -1.0 : 1.0;
    const double vr = rr - sb * ii, vi = sb * ri + ir;
    const double re = alr * vr - ali * vi;
    if (u) u[rm] = u_store ? u_sign * re : u[rm] + u_sign * re;
    if (cr) cr[OUT ? tr : rm] = re;
    if (ci) ci[OUT ? tr : rm] = alr * vi + ali * vr;
}

// One wave per run.  Complex x complex does not pipeline: a second set of
// operands costs waves per SIMD (32,768 atoms, R 12: U K 5.0 -> 5.5 ms).  Four
// sums per complex output: adding the imaginary products to the real ones' sum
// as they come doubled its roundings (error of a product against 64-bit
// arithmetic 6.0e-16 -> 8.5e-16) for 0 - 4 % of the time.
template <bool AC, bool BC, int CJB, int OUT, bool BROWS = false>
__global__ __launch_bounds__(256) void k_spgemm_b4p(
    int64_t nch, const int64_t *__restrict__ off, const int32_t *__restrict__ ea,
    const int32_t *__restrict__ eb, const int32_t *__restrict__ cout, const double *__restrict__ ar,
    const double *__restrict__ ai, const double *__restrict__ br, const double *__restrict__ bi,
    double *__restrict__ cr, double *__restrict__ ci, double alr, double ali, double *__restrict__ u,
    double u_sign, int u_store, int remap)
{
    const int64_t c = xcd_block((nch + 3) / 4, remap) * 4 + (threadIdx.x >> 6);
    if (c >= nch) return;                      // uniform across the wave
    const int g = (threadIdx.x >> 2) & 3;
    double rr[4] = {0, 0, 0, 0}, ii[4] = {0, 0, 0, 0}, ri[4] = {0, 0, 0, 0}, ir[4] = {0, 0, 0, 0};
    b4p_entries<AC, BC, !(AC && BC), BROWS>(off[c], off[c + 1], 2, ea, eb, ar, ai, br, bi, rr, ii, ri, ir);
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        const int p = cout[c * 16 + 4 * jj + g];
        if (p >= 0) b4p_store<CJB, OUT>(p, rr[jj], ii[jj], ri[jj], ir[jj], cr, ci, alr, ali, u, u_sign, u_store);
    }
}

// The same for products with few runs (small systems): one workgroup of W
// waves per run, wave w taking the pairs of entries w, w + W, ..., the waves'
// partial sums added in LDS, wave jj those of outputs 4 jj .. 4 jj + 3, in the
// fixed order w = 0, 1, ...  Bound: with a run per compute unit still the
// address unit (62 entries of 170 cycles at 8 bytes a lane, 80 at 16), then
// the launch and its chain of loads.  64-atom cluster, us per launch, 8-byte
// loads of one entry after the other -> now: U K 11.8 -> 8.8, W U^dagger
// 13.7 -> 8.5.
template <bool AC, bool BC, int CJB, int OUT, int W>
__global__ __launch_bounds__(64 * W) void k_spgemm_b4ps(
    int64_t nch, const int64_t *__restrict__ off, const int32_t *__restrict__ ea,
    const int32_t *__restrict__ eb, const int32_t *__restrict__ cout, const double *__restrict__ ar,
    const double *__restrict__ ai, const double *__restrict__ br, const double *__restrict__ bi,
    double *__restrict__ cr, double *__restrict__ ci, double alr, double ali, double *__restrict__ u,
    double u_sign, int u_store)
{
    static_assert(W >= 4, "one wave per four outputs adds the partial sums");
    constexpr int NACC = 1 + (AC && BC) + BC + AC;   // sums per output: rr, ii, ri, ir
    __shared__ double part[W][4][NACC][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t c = blockIdx.x;              // grid = nch: uniform across the workgroup
    const int p = cout[c * 16 + 4 * (wv & 3) + ((lane >> 2) & 3)];   // output of the sums below
    double rr[4] = {0, 0, 0, 0}, ii[4] = {0, 0, 0, 0}, ri[4] = {0, 0, 0, 0}, ir[4] = {0, 0, 0, 0};
    b4p_entries<AC, BC, true>(off[c] + 2 * wv, off[c + 1], 2 * W, ea, eb, ar, ai, br, bi, rr, ii, ri, ir);
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        int k = 0;
        part[wv][jj][k++][lane] = rr[jj];
        if (AC && BC) part[wv][jj][k++][lane] = ii[jj];
        if (BC) part[wv][jj][k++][lane] = ri[jj];
        if (AC) part[wv][jj][k++][lane] = ir[jj];
    }
    __syncthreads();
    if (wv >= 4 || p < 0) return;
    double sum[NACC];
#pragma unroll
    for (int k = 0; k < NACC; ++k) {
        sum[k] = part[0][wv][k][lane];
#pragma unroll
        for (int w = 1; w < W; ++w) sum[k] += part[w][wv][k][lane];
    }
    constexpr bool CC = AC && BC;
    b4p_store<CJB, OUT>(p, sum[0], CC ? sum[CC ? 1 : 0] : 0.0, BC ? sum[CC ? 2 : BC ? 1 : 0] : 0.0,
                        AC ? sum[NACC - 1] : 0.0, cr, ci, alr, ali, u, u_sign, u_store);
}

template <bool AC, bool BC, int CJB, int OUT, bool BROWS = false>
static void launch_b4p_runs(hipStream_t s, const SpgemmArgs &a, const SumInto &u)
{
    const int remap = xcd_chunk_for((a.nch + 3) / 4);
    hipLaunchKernelGGL((k_spgemm_b4p<AC, BC, CJB, OUT, BROWS>), dim3(xcd_grid((a.nch + 3) / 4, remap)), dim3(256), 0, s,
                       a.nch, a.ch_off, a.ch_a, a.ch_b, a.ch_out, a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.alpha_re,
                       a.alpha_im, u.p, u.sign, u.store, remap);
}

template <bool AC, bool BC, int CJB, int OUT>
static void launch_b4p_as(hipStream_t s, const SpgemmArgs &a, const SumInto &u)
{
#define RT_B4PS(W)                                                                                                  \
    hipLaunchKernelGGL((k_spgemm_b4ps<AC, BC, CJB, OUT, W>), dim3((unsigned)a.nch), dim3(64 * W), 0, s, a.nch, a.ch_off, \
                       a.ch_a, a.ch_b, a.ch_out, a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.alpha_re, a.alpha_im, u.p,   \
                       u.sign, u.store)
    if (a.nch < kB4Split8Runs) {
        RT_B4PS(8);
        return;
    }
    if (a.nch < kB4SplitRuns) {
        RT_B4PS(4);
        return;
    }
#undef RT_B4PS
    launch_b4p_runs<AC, BC, CJB, OUT>(s, a, u);
}

// b = 4 FP64 product over runs of 16 from a row-major left operand and a right
// operand with transposed blocks (conj_b: the row-major blocks of the matrix
// whose conjugate transpose it is); out_t: the output with transposed blocks
// (real left operands; real right ones too below kB4SplitRuns runs); u: the
// output's fused sum (real products).
void launch_spgemm_b4t(hipStream_t s, const SpgemmArgs &a, int conj_b, int out_t, const SumInto &u)
{
    RT_CHECK(a.b == 4 && a.precision == RTDM_PREC_FP64 && a.nj == 16 && a.nch > 0 && a.op_a == 0, RTDM_E_ARG,
             "transposed-block products need b = 4, FP64 and runs of 16");
    const bool ac = a.ai != nullptr, bc = a.bi != nullptr;
    RT_CHECK(!u.p || (!ac && !bc && !a.ci), RTDM_E_ARG, "the fused sum needs real operands");
    RT_CHECK(!out_t || (!ac && !conj_b && (!bc || a.nch >= kB4SplitRuns)), RTDM_E_ARG,
             "no transposed output of these operands");
#define RT_B4P(AC_, BC_)                                                      \
    do {                                                                      \
        if (conj_b) launch_b4p_as<AC_, BC_, 1, 0>(s, a, u);                   \
        else launch_b4p_as<AC_, BC_, 0, 0>(s, a, u);                          \
    } while (0)
    if (out_t && bc) launch_b4p_runs<false, true, 0, 1>(s, a, u);
    else if (out_t) launch_b4p_as<false, false, 0, 1>(s, a, u);
    else if (ac && bc) RT_B4P(true, true);
    else if (ac) RT_B4P(true, false);
    else if (bc) RT_B4P(false, true);
    else RT_B4P(false, false);
#undef RT_B4P
    RT_HIP(hipGetLastError());
}

// FP64 b = 4 product over row runs with few runs (small systems) whose right
// operand is by rows: one workgroup of W waves per run, wave w taking the entries w, w + W, ..., so
// that a run's chain of dependent loads is 1/W as long and W times as many
// waves share the chip.  The waves' partial sums are added in LDS in the
// fixed order w = 0, 1, ..., W - 1.
template <bool AC, bool BC, int W>
__global__ __launch_bounds__(64 * W) void k_spgemm_b4js(
    int64_t nch, const int64_t *__restrict__ off, const int32_t *__restrict__ ea,
    const int32_t *__restrict__ eb, const int32_t *__restrict__ cout, const double *__restrict__ ar,
    const double *__restrict__ ai, const double *__restrict__ br, const double *__restrict__ bi,
    double *__restrict__ cr, double *__restrict__ ci, double alr, double ali)
{
    constexpr int NACC = 1 + (AC && BC) + BC + AC;   // accumulators per output: rr, ii, ri, ir
    __shared__ double part[W - 1][NACC * 4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int g = (lane >> 2) & 3, r = lane & 3, q = lane >> 4;
    const int64_t c = blockIdx.x;              // grid = nch: uniform across the workgroup
    const int ia = r * 4 + q, ib = q * 4 + r;
    double rr[4] = {0, 0, 0, 0}, ii[4] = {0, 0, 0, 0}, ri[4] = {0, 0, 0, 0}, ir[4] = {0, 0, 0, 0};
    b4_run_entries<AC, BC>(off[c] + wv, off[c + 1], W, ea, eb, ar, ai, br, bi, ia, ib, g, rr, ii, ri, ir);
    auto pack = [&](double (*dst)[64]) {
        int k = 0;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            dst[k++][lane] = rr[jj];
            if (AC && BC) dst[k++][lane] = ii[jj];
            if (BC) dst[k++][lane] = ri[jj];
            if (AC) dst[k++][lane] = ir[jj];
        }
    };
    if (wv > 0) pack(part[wv - 1]);
    __syncthreads();
    if (wv != 0) return;
#pragma unroll 1
    for (int w = 0; w < W - 1; ++w) {          // one wave's partials at a time (registers)
        int k = 0;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            rr[jj] += part[w][k++][lane];
            if (AC && BC) ii[jj] += part[w][k++][lane];
            if (BC) ri[jj] += part[w][k++][lane];
            if (AC) ir[jj] += part[w][k++][lane];
        }
    }
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        const int p = cout[c * 16 + 4 * jj + g];
        if (p >= 0) {
            const double re = rr[jj] - ii[jj], im = ri[jj] + ir[jj];
            const int64_t o = (int64_t)p * 16 + q * 4 + r;
            cr[o] = alr * re - ali * im;
            if (ci) ci[o] = alr * im + ali * re;
        }
    }
}

template <bool AC, bool BC>
static void launch_b4j(hipStream_t s, const SpgemmArgs &a)
{
    RT_CHECK(a.nj == 16, RTDM_E_ARG, "b = 4 row runs hold 16 outputs");
    if (a.nch < kB4Split8Runs) {
        hipLaunchKernelGGL((k_spgemm_b4js<AC, BC, 8>), dim3((unsigned)a.nch), dim3(512), 0, s, a.nch,
                           a.ch_off, a.ch_a, a.ch_b, a.ch_out, a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.alpha_re,
                           a.alpha_im);
        return;
    }
    if (a.nch >= kB4SplitRuns) {
        launch_b4p_runs<AC, BC, 0, 0, true>(s, a, SumInto());
        return;
    }
    hipLaunchKernelGGL((k_spgemm_b4js<AC, BC, 4>), dim3((unsigned)a.nch), dim3(256), 0, s, a.nch, a.ch_off, a.ch_a,
                       a.ch_b, a.ch_out, a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.alpha_re, a.alpha_im);
}

template <bool AC, bool BC, int OB>
static void launch_b4w(hipStream_t s, const SpgemmArgs &a)
{
    hipLaunchKernelGGL((k_spgemm_b4w<AC, BC, OB>), dim3((unsigned)((a.nout + 63) / 64)), dim3(256), 0, s, a.nout,
                       a.off, a.trip, a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.alpha_re, a.alpha_im);
}

template <int SUB, bool AC, bool BC, int OA, int OB>
static void launch_b4(hipStream_t s, const SpgemmArgs &a)
{
    constexpr int OUT = 4 / SUB;
    const int64_t waves = (a.nout + OUT - 1) / OUT;
    hipLaunchKernelGGL((k_spgemm_b4<SUB, AC, BC, OA, OB>), dim3((unsigned)((waves + 3) / 4)), dim3(256),
                       0, s, a.nout, a.off, a.trip, a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.alpha_re,
                       a.alpha_im);
}

template <bool AC, bool BC, int OA, int OB>
static void launch_split(hipStream_t s, const SpgemmArgs &a, dim3 g, dim3 t)
{
#define RT_SPLIT(B_, M_)                                                                         \
    hipLaunchKernelGGL((k_spgemm_split<B_, AC, BC, OA, OB, M_>), g, t, 0, s, a.nout, a.off, a.trip, \
                       a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.alpha_re, a.alpha_im, a.maxabs)
    const int mode = a.precision == RTDM_PREC_FP16X2 ? 1 : 0;
    if (a.b == 13 && mode == 0) RT_SPLIT(13, 0);
    else if (a.b == 13) RT_SPLIT(13, 1);
    else if (mode == 0) RT_SPLIT(4, 0);
    else RT_SPLIT(4, 1);
#undef RT_SPLIT
}

template <bool AC, bool BC>
static void dispatch_ops(hipStream_t s, const SpgemmArgs &a, dim3 g, dim3 t)
{
#define RT_LAUNCH(OA, OB)                                                                        \
    do {                                                                                         \
        if (a.precision != RTDM_PREC_FP64 && a.b == 4 && OA == 0)                                \
            launch_b4x<AC, BC, OB>(s, a);                                                        \
        else if (a.precision == RTDM_PREC_BF16X3 || a.precision == RTDM_PREC_FP16X2)             \
            launch_split<AC, BC, OA, OB>(s, a, g, t);                                            \
        else if (a.precision == RTDM_PREC_FP32 && a.b == 13)                                     \
            hipLaunchKernelGGL((k_spgemm_kc<13, AC, BC, OA, OB, float>), g, t, 0, s, a.nout,     \
                               a.off, a.trip, a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.alpha_re,    \
                               a.alpha_im);                                                      \
        else if (a.precision == RTDM_PREC_FP32 && a.b >= 4)                                      \
            hipLaunchKernelGGL((k_spgemm_kc<4, AC, BC, OA, OB, float>), g, t, 0, s, a.nout,      \
                               a.off, a.trip, a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.alpha_re,    \
                               a.alpha_im);                                                      \
        else if (a.b == 4 && OA == 0 && OB == 0 && a.nch > 0)                                    \
            launch_b4j<AC, BC>(s, a);                                                            \
        else if (a.b == 4 && OA == 0)                                                            \
            launch_b4w<AC, BC, OB>(s, a);                                                        \
        else if (a.b == 4)                                                                       \
            launch_b4<(AC && BC) ? 4 : ((AC || BC) ? 2 : 1), AC, BC, OA, OB>(s, a);              \
        else if (a.b == 13)                                                                      \
            hipLaunchKernelGGL((k_spgemm_kc<13, AC, BC, OA, OB>), g, t, 0, s, a.nout, a.off,     \
                               a.trip, a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.alpha_re,           \
                               a.alpha_im);                                                      \
        else if (a.b == 16)                                                                      \
            hipLaunchKernelGGL((k_spgemm_kc<16, AC, BC, OA, OB>), g, t, 0, s, a.nout, a.off,     \
                               a.trip, a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.alpha_re,           \
                               a.alpha_im);                                                      \
        else                                                                                     \
            hipLaunchKernelGGL((k_spgemm16<AC, BC, OA, OB>), g, t, 0, s, a.nout, a.off, a.trip,  \
                               a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.b, a.alpha_re, a.alpha_im); \
    } while (0)
    if (!a.op_a && !a.op_b) RT_LAUNCH(0, 0);
    else if (a.op_a && !a.op_b) RT_LAUNCH(1, 0);
    else if (!a.op_a && a.op_b) RT_LAUNCH(0, 1);
    else RT_LAUNCH(1, 1);
#undef RT_LAUNCH
}

// Step products with a column-major copy of the left operand (op(A)[r][m] at
// m*B + r) and a right operand whose op(B)[m][r] sits at m*B + r (row-major
// B, or the column-major copy of a matrix used conjugate-transposed).
template <bool AC, bool BC, int CJB, int LC>
static void launch_cm(hipStream_t s, const SpgemmArgs &a, dim3 g, dim3 t)
{
    {
        const int wpb = a.wpb;
        const int remap = xcd_chunk_wg(wpb);
        const unsigned grid = xcd_grid((a.nout + wpb - 1) / wpb, remap);
#define RT_Q4(W, T)                                                                               \
    hipLaunchKernelGGL((k_spgemm_q4<13, AC, BC, 0, CJB, LC, W, T>), dim3(grid), dim3(64 * W), 0, s, \
                       a.nout, a.off, a.trip, a.ar, a.ai, a.br, a.bi, a.cr, a.ci, a.alpha_re,       \
                       a.alpha_im, a.zero, a.order, remap)
        if (a.precision == RTDM_PREC_FP32) {
            if (wpb == 16) RT_Q4(16, float);
            else if (wpb == 8) RT_Q4(8, float);
            else RT_Q4(4, float);
        } else {
            if (wpb == 16) RT_Q4(16, double);
            else if (wpb == 8) RT_Q4(8, double);
            else RT_Q4(4, double);
        }
#undef RT_Q4
    }
}

// Row-run kernel (k_spgemm_q4j): runs of 2, 3 or 4 outputs, or 8 for real operands.
template <bool AC, bool BC, int CJB, int LC>
static void launch_cmj(hipStream_t s, const SpgemmArgs &a)
{
    const int remap = xcd_chunk();
    const unsigned grid = xcd_grid((a.nch + 3) / 4, remap);
    const bool f32 = a.precision == RTDM_PREC_FP32;
#define RT_Q4J_W(NJ, T, W)                                                                       \
    hipLaunchKernelGGL((k_spgemm_q4j<13, AC, BC, CJB, LC, NJ, T, W>), dim3(grid), dim3(256), 0, s,   \
                       a.nch,                                                                         \
                       a.ch_off, a.ch_a, a.ch_b, a.ch_out, a.ar, a.ai, a.br, a.bi, a.cr, a.ci,        \
                       a.alpha_re, a.alpha_im, a.zero, a.ch_order, remap, a.ch_seg)
#define RT_Q4J(NJ, T) RT_Q4J_W(NJ, T, 1)
    if (a.nj == 2) {
        // complex runs of 2 compiled for at least 4 waves per SIMD (at most 128
        // registers): 4 % faster than the compiler's 3; real runs lose 12 % so
        if (f32) RT_Q4J(2, float);
        else RT_Q4J_W(2, double, (AC && BC) ? 4 : 1);
    } else if (a.nj == 3) {
        if (f32) RT_Q4J(3, float);
        else RT_Q4J_W(3, double, (AC && BC) ? 4 : 1);
    } else if (a.nj == 4) {
        if (f32) RT_Q4J(4, float);
        else RT_Q4J(4, double);
    } else {
        if constexpr (!AC && !BC) {
            RT_CHECK(a.nj == 8, RTDM_E_ARG, "row runs of 2, 3, 4 or 8 outputs");
            if (f32) RT_Q4J(8, float);
            else RT_Q4J(8, double);
        } else {
            RT_CHECK(false, RTDM_E_ARG, "row runs of complex products hold 2, 3 or 4 outputs");
        }
    }
#undef RT_Q4J
#undef RT_Q4J_W
}

void launch_spgemm_cm(hipStream_t s, const SpgemmArgs &a, int conj_b, int out_col_major)
{
    if (a.nout == 0) return;
    RT_CHECK(a.b == 13 && (a.precision == RTDM_PREC_FP64 || a.precision == RTDM_PREC_FP32), RTDM_E_UNSUPPORTED,
             "column-major step products need b = 13 and FP64 or FP32");
    const dim3 g((unsigned)((a.nout + 3) / 4)), t(256);
    const bool ac = a.ai != nullptr, bc = a.bi != nullptr;
#define RT_CM(AC_, BC_)                                                            \
    do {                                                                           \
        if (a.nch > 0) {                                                           \
            if (conj_b && out_col_major) launch_cmj<AC_, BC_, 1, 1>(s, a);         \
            else if (conj_b) launch_cmj<AC_, BC_, 1, 0>(s, a);                     \
            else if (out_col_major) launch_cmj<AC_, BC_, 0, 1>(s, a);              \
            else launch_cmj<AC_, BC_, 0, 0>(s, a);                                 \
        } else if (conj_b && out_col_major) launch_cm<AC_, BC_, 1, 1>(s, a, g, t); \
        else if (conj_b) launch_cm<AC_, BC_, 1, 0>(s, a, g, t);                    \
        else if (out_col_major) launch_cm<AC_, BC_, 0, 1>(s, a, g, t);             \
        else launch_cm<AC_, BC_, 0, 0>(s, a, g, t);                                \
    } while (0)
    if (ac && bc) RT_CM(true, true);
    else if (ac) RT_CM(true, false);
    else if (bc) RT_CM(false, true);
    else RT_CM(false, false);
#undef RT_CM
    RT_HIP(hipGetLastError());
}


// FP32 variant of k_spgemm_q4 for real operands (the Taylor-term products of
// the reduced-precision form): column-major FP32 left operand, row-major FP32
// right operand, v_mfma_f32_16x16x4_f32 with FP32 accumulation, FP32 output
// scaled by alpha.  Same four-triple grouping, order and XCD mapping.
template <int B, int WPB>
__global__ __launch_bounds__(64 * WPB) void k_spgemm_q4r32(
    int64_t nout, const int64_t *__restrict__ off, const int2 *__restrict__ trip,
    const float *__restrict__ a, const float *__restrict__ b, float *__restrict__ cout, float alpha,
    const float *__restrict__ zero, const int32_t *__restrict__ order)
{
    constexpr int BB = B * B;
    const int lane = threadIdx.x & 63;
    const int64_t w = xcd_block((nout + WPB - 1) / WPB) * WPB + (threadIdx.x >> 6);
    if (w >= nout) return;                     // uniform across the wave
    const int64_t c = order ? (int64_t)order[w] : w;
    const int r = lane & 15, q = lane >> 4;
    const bool rv = r < B;
    const int64_t t0 = off[c];
    const int nt = (int)(off[c + 1] - t0);
    typedef Mfma16<float>::acc_t acc_t;
    acc_t acc = {0, 0, 0, 0};
    for (int g = 0; g < nt; g += 4) {
        const float *pa = zero, *pb = zero;
        if (rv && g + q < nt) {
            const int2 ab = trip[t0 + g + q];
            pa = a + (int64_t)ab.x * BB + r;
            pb = b + (int64_t)ab.y * BB + r;
        }
#pragma unroll
        for (int st = 0; st < B; ++st) acc = Mfma16<float>::step(pa[st * B], pb[st * B], acc);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int row = Mfma16<float>::row(e, q), col = r;
        if (row < B && col < B) cout[c * BB + row * B + col] = alpha * acc[e];
    }
}

// Row-run form of k_spgemm_q4r32 (the dataflow of k_spgemm_q4j on FP32
// storage): NJ outputs of one row per wave, each loaded left-operand element
// feeding NJ FP32 MFMAs.
typedef __attribute__((address_space(1))) const float gfloat;
template <int B, int NJ>
__global__ __launch_bounds__(256) void k_spgemm_q4jr32(
    int64_t nch, const int64_t *__restrict__ off, const int32_t *__restrict__ ea,
    const int32_t *__restrict__ eb, const int32_t *__restrict__ cidx, const float *__restrict__ a,
    const float *__restrict__ b, float *__restrict__ cout, float alpha, const float *__restrict__ zero,
    const int32_t *__restrict__ order, int remap, const int32_t *__restrict__ seg)
{
    constexpr int BB = B * B;
    const int lane = threadIdx.x & 63;
    const int64_t w = xcd_block((nch + 3) / 4, remap) * 4 + (threadIdx.x >> 6);
    if (w >= nch) return;                      // uniform across the wave
    const int64_t c = order ? (int64_t)order[w] : w;
    const int r = lane & 15, q = lane >> 4;
    const bool rv = r < B;
    const int64_t e0 = off[c];
    const int ne = (int)(off[c + 1] - e0);
    typedef Mfma16<float>::acc_t acc_t;
    acc_t acc[NJ];
#pragma unroll
    for (int t = 0; t < NJ; ++t) acc[t] = acc_t{0, 0, 0, 0};
    const gfloat *gz = (const gfloat *)zero;
    // entries [gb, ge); output t's products only where bit t of ACT is set (segments as in k_spgemm_q4j)
    auto groups = [&](int gb, int ge, auto act) {
        constexpr int ACT = decltype(act)::value;
        for (int g = gb; g < ge; g += 4) {
            const gfloat *pa = gz;
            const gfloat *pb[NJ];
#pragma unroll
            for (int t = 0; t < NJ; ++t) pb[t] = gz;
            if (rv && g + q < ge) {
                const int64_t e = e0 + g + q;
                pa = (const gfloat *)(a + (int64_t)ea[e] * BB + r);
#pragma unroll
                for (int t = 0; t < NJ; ++t) {
                    if (!((ACT >> t) & 1)) continue;
                    const int kb = eb[e * NJ + t];
                    if (kb >= 0) pb[t] = (const gfloat *)(b + (int64_t)kb * BB + r);
                }
            }
#pragma unroll
            for (int st = 0; st < B; ++st) {
                const float xa = pa[st * B];
#pragma unroll
                for (int t = 0; t < NJ; ++t)
                    if ((ACT >> t) & 1) acc[t] = Mfma16<float>::step(xa, pb[t][st * B], acc[t]);
            }
        }
    };
    constexpr int ALL = (1 << NJ) - 1;
    if constexpr (NJ == 2) {
        if (seg) {
            const int nf = seg[2 * c], n0 = seg[2 * c + 1];   // uniform across the wave
            groups(0, nf, std::integral_constant<int, 3>());
            groups(nf, nf + n0, std::integral_constant<int, 1>());
            groups(nf + n0, ne, std::integral_constant<int, 2>());
        } else {
            groups(0, ne, std::integral_constant<int, ALL>());
        }
    } else {
        groups(0, ne, std::integral_constant<int, ALL>());
    }
#pragma unroll
    for (int t = 0; t < NJ; ++t) {
        const int p = cidx[c * NJ + t];
        if (p < 0) continue;                   // uniform: a short run
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = Mfma16<float>::row(e, q), col = r;
            if (row < B && col < B) cout[(int64_t)p * BB + row * B + col] = alpha * acc[t][e];
        }
    }
}

// Real FP32-storage b = 4 product (the late Taylor terms of the fp32_taylor
// form): A in FP32 row-major blocks, B in FP32 transposed blocks, so that a
// lane's row of A and column of B are one 16-byte load each;
// v_mfma_f32_4x4x1_16b with FP32 accumulation, lane 4 blk + r holding row r
// of A_blk and column r of B_blk.  The term alpha * sum is added into the FP64
// plane u (u += u_sign * term: the propagator's sum) and, when c32 is set,
// stored in FP32 transposed blocks as the next term's right operand.  RUNS:
// one row run of 16 outputs per wave (entries shared by all blocks, b = 4
// slot order); otherwise 16 consecutive outputs per wave, each with its own
// triple list.  Bound: the vector-memory address unit (15 cycles per 16-byte
// load, 5 per 4-byte one): 22 cycles an entry over runs, where one load of A
// an entry and four 4-byte loads of B took 45.  2,744 atoms, R 16, per term
// with its sum: 0.78 -> 0.49 ms.
struct F32Idx8 {
    int a, b[8];
};
// h += A_s B_s over entries s = E .. 7, A_s broadcast from MFMA block s
template <int E>
__device__ inline void mfma_f32_8(const f32x4 &xa, const f32x4 (&xb)[8], f32x4 &h)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) h = __builtin_amdgcn_mfma_f32_4x4x1f32(xa[k], xb[E][k], h, 4, E, 0);
    if constexpr (E < 7) mfma_f32_8<E + 1>(xa, xb, h);
}

template <bool RUNS>
__global__ __launch_bounds__(256) void k_spgemm_b4r32(
    int64_t n, const int64_t *__restrict__ off, const int2 *__restrict__ trip, const int32_t *__restrict__ ea,
    const int32_t *__restrict__ eb, const int32_t *__restrict__ rout, const float *__restrict__ a,
    const float *__restrict__ b, float *__restrict__ c32, float alpha, double *__restrict__ u, double u_sign,
    int remap)
{
    const int lane = threadIdx.x & 63;
    const int blk = lane >> 2, r = lane & 3;
    const int64_t nwv = RUNS ? n : (n + 15) / 16;
    const int64_t wv = xcd_block((nwv + 3) / 4, remap) * 4 + (threadIdx.x >> 6);
    if (wv >= nwv) return;                     // uniform across the wave
    const int64_t c = RUNS ? (int64_t)rout[wv * 16 + blk] : wv * 16 + blk;
    const bool live = RUNS ? c >= 0 : c < n;
    const int64_t t0 = RUNS ? off[wv] : (live ? off[c] : 0);
    const int nt = RUNS ? (int)(off[wv + 1] - t0) : (live ? (int)(off[c + 1] - t0) : 0);
    int ntmax = nt;
    if (!RUNS) {
#pragma unroll
        for (int o = 4; o < 64; o <<= 1) ntmax = max(ntmax, __shfl_xor(ntmax, o, 64));
    }
    const int slot = (blk & 3) * 4 + (blk >> 2);
    f32x4 h = {0, 0, 0, 0};
    auto load_ops = [&](int2 ab, f32x4 &xa, f32x4 &xb) {
        xa = xb = f32x4{0, 0, 0, 0};
        if (ab.y >= 0) {
            xa = *reinterpret_cast<const f32x4 *>(a + (int64_t)ab.x * 16 + r * 4);   // A[r][0..3]
            xb = *reinterpret_cast<const f32x4 *>(b + (int64_t)ab.y * 16 + r * 4);   // B[0..3][r]
        }
    };
    auto products = [&](const f32x4 &xa, const f32x4 &xb) {
#pragma unroll
        for (int k = 0; k < 4; ++k) h = __builtin_amdgcn_mfma_f32_4x4x1f32(xa[k], xb[k], h, 0, 0, 0);
    };
    if constexpr (RUNS) {
        // Eight entries at a time: lane 4 blk + r loads row r of the A block of
        // entry blk % 8, and the MFMAs of entry s broadcast block s's rows to all
        // sixteen blocks (cbsz 4, abid s), so one load serves the A of eight
        // entries.  The next eight entries' indices are loaded ahead.
        auto load_idx = [&](int t) {
            F32Idx8 x{-1, {-1, -1, -1, -1, -1, -1, -1, -1}};
            if (t + (blk & 7) < nt) x.a = ea[t0 + t + (blk & 7)];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (t + e < nt) x.b[e] = eb[(t0 + t + e) * 16 + slot];
            return x;
        };
        F32Idx8 cur = load_idx(0);
        for (int t = 0; t < nt; t += 8) {
            f32x4 xa = {0, 0, 0, 0}, xb[8];
            if (cur.a >= 0) xa = *reinterpret_cast<const f32x4 *>(a + (int64_t)cur.a * 16 + r * 4);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                xb[e] = f32x4{0, 0, 0, 0};
                if (cur.b[e] >= 0) xb[e] = *reinterpret_cast<const f32x4 *>(b + (int64_t)cur.b[e] * 16 + r * 4);
            }
            cur = load_idx(t + 8);
            mfma_f32_8<0>(xa, xb, h);
        }
    } else {
        for (int t = 0; t < ntmax; ++t) {
            const int2 ab = t < nt ? trip[t0 + t] : make_int2(0, -1);
            f32x4 xa, xb;
            load_ops(ab, xa, xb);
            products(xa, xb);
        }
    }
    if (!live) return;
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = alpha * h[e];
        const int64_t o = c * 16 + e * 4 + r;
        u[o] += u_sign * (double)v[e];
    }
    if (c32) *reinterpret_cast<f32x4 *>(c32 + c * 16 + r * 4) = v;   // column r of the block
}

// The b = 4 FP32 Taylor term: b32 and c32 (nullable) with transposed blocks, u += u_sign * term.
void launch_spgemm_b4_r32(hipStream_t s, const SpgemmArgs &a, const float *a32, const float *b32, float *c32, double *u,
                          double u_sign)
{
    RT_CHECK(a.b == 4 && u, RTDM_E_ARG, "b = 4 FP32 Taylor terms are summed as they are written");
    const bool runs = a.nch > 0;
    RT_CHECK(!runs || a.nj == 16, RTDM_E_ARG, "b = 4 row runs hold 16 outputs");
    if (!runs && a.nout == 0) return;
    const int64_t nwg = ((runs ? a.nch : (a.nout + 15) / 16) + 3) / 4;
    const int remap = xcd_chunk_for(nwg);
    const dim3 g(xcd_grid(nwg, remap)), t(256);
    if (runs)
        hipLaunchKernelGGL(k_spgemm_b4r32<true>, g, t, 0, s, a.nch, a.ch_off, nullptr, a.ch_a, a.ch_b, a.ch_out, a32,
                           b32, c32, (float)a.alpha_re, u, u_sign, remap);
    else
        hipLaunchKernelGGL(k_spgemm_b4r32<false>, g, t, 0, s, a.nout, a.off, a.trip, nullptr, nullptr, nullptr, a32,
                           b32, c32, (float)a.alpha_re, u, u_sign, remap);
    RT_HIP(hipGetLastError());
}

// BF16 x 2 storage of b = 4 blocks for the BF16x3 late Taylor terms: x =
// hi + lo with the split of the register-split kernels (Split4<0>: round to
// FP32, hi its BF16 rounding, lo that of the remainder).  Block p takes 32
// values (64 bytes, one memory sector like an FP32 block): per row its four hi
// parts, then its four lo parts, one 16-byte load of a lane; `transpose`
// stores each block transposed (the columns of a right operand).
__global__ void k_to_bf16x2(int64_t n, int transpose, const double *__restrict__ in, short *__restrict__ out)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int w = (int)(e & 15);
        const int row = transpose ? w & 3 : w >> 2, k = transpose ? w >> 2 : w & 3;
        const int64_t o = (e >> 4) * 32 + row * 8 + k;
        short h, l;
        Split4<0>::split(in[e], 1.0f, h, l);
        out[o] = h;
        out[o + 4] = l;
    }
}

void launch_to_bf16x2(hipStream_t s, int64_t nblocks, int transpose, const double *in, short *out)
{
    const int64_t n = nblocks * 16;
    if (n == 0) return;
    int64_t g = (n + 255) / 256;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_to_bf16x2, dim3((unsigned)g), dim3(256), 0, s, n, transpose, in, out);
    RT_HIP(hipGetLastError());
}

// BF16x3 late Taylor term at b = 4 over row runs of 16 outputs, operands
// stored split (launch_to_bf16x2: A by rows, tau by columns): one wave per
// run, lane 4 blk + r holding row r of A and column r of output blk's B as
// four BF16 values per part, both parts one 16-byte load; three
// v_mfma_f32_4x4x4_16b_bf16 per entry (hi hi, then hi lo and lo hi into a
// second accumulator), eight entries at a time with A broadcast from one
// MFMA block per entry as in k_spgemm_b4r32.  The result tau = alpha (h + m)
// is added into the FP64 plane u (u += u_sign tau: the propagator's sum) and,
// when c16 is set, stored split and transposed as the next term's right
// operand.  The split, the products and their order per output are those of
// the register-split kernel (k_spgemm_b4x<..., 1, true>).  Per entry 22
// cycles of the vector-memory address unit (70 with 8-byte loads of each part).
typedef short bf16q __attribute__((ext_vector_type(4)));
typedef short bf16o __attribute__((ext_vector_type(8)));
template <int E>
__device__ inline void mfma_bf16_8(bf16o xa, const bf16o (&xb)[8], f32x4 &h, f32x4 &m)
{
    const bf16q ah = __builtin_shufflevector(xa, xa, 0, 1, 2, 3), al = __builtin_shufflevector(xa, xa, 4, 5, 6, 7);
    const bf16q bh = __builtin_shufflevector(xb[E], xb[E], 0, 1, 2, 3),
                bl = __builtin_shufflevector(xb[E], xb[E], 4, 5, 6, 7);
    h = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ah, bh, h, 4, E, 0);
    m = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ah, bl, m, 4, E, 0);
    m = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(al, bh, m, 4, E, 0);
    if constexpr (E < 7) mfma_bf16_8<E + 1>(xa, xb, h, m);
}

__global__ __launch_bounds__(256) void k_spgemm_b4r16(
    int64_t nch, const int64_t *__restrict__ off, const int32_t *__restrict__ ea, const int32_t *__restrict__ eb,
    const int32_t *__restrict__ rout, const short *__restrict__ a16, const short *__restrict__ b16,
    short *__restrict__ c16, double alpha, double *__restrict__ u, double u_sign, int remap)
{
    const int lane = threadIdx.x & 63;
    const int blk = lane >> 2, r = lane & 3;
    const int64_t wv = xcd_block((nch + 3) / 4, remap) * 4 + (threadIdx.x >> 6);
    if (wv >= nch) return;                     // uniform across the wave
    const int64_t c = rout[wv * 16 + blk];
    const int64_t t0 = off[wv];
    const int nt = (int)(off[wv + 1] - t0);
    const int slot = (blk & 3) * 4 + (blk >> 2);
    f32x4 h = {0, 0, 0, 0}, m = {0, 0, 0, 0};
    auto load_idx = [&](int t) {
        F32Idx8 x{-1, {-1, -1, -1, -1, -1, -1, -1, -1}};
        if (t + (blk & 7) < nt) x.a = ea[t0 + t + (blk & 7)];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (t + e < nt) x.b[e] = eb[(t0 + t + e) * 16 + slot];
        return x;
    };
    F32Idx8 cur = load_idx(0);
    for (int t = 0; t < nt; t += 8) {
        bf16o xa = {}, xb[8];
        if (cur.a >= 0) xa = *reinterpret_cast<const bf16o *>(a16 + (int64_t)cur.a * 32 + r * 8);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            xb[e] = bf16o{};
            if (cur.b[e] >= 0) xb[e] = *reinterpret_cast<const bf16o *>(b16 + (int64_t)cur.b[e] * 32 + r * 8);
        }
        cur = load_idx(t + 8);
        mfma_bf16_8<0>(xa, xb, h, m);
    }
    if (c < 0) return;
    bf16o st;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const double v = alpha * ((double)h[e] + 1.0 * (double)m[e]);
        const int64_t o = c * 16 + e * 4 + r;
        u[o] = u[o] + u_sign * v;
        short hh, ll;
        Split4<0>::split(v, 1.0f, hh, ll);
        st[e] = hh;
        st[e + 4] = ll;
    }
    if (c16) *reinterpret_cast<bf16o *>(c16 + c * 32 + r * 8) = st;   // column r of the block
}

void launch_spgemm_r16(hipStream_t s, const SpgemmArgs &a, const short *a16, const short *b16, short *c16,
                       double *u, double u_sign)
{
    RT_CHECK(a.b == 4 && a.nch > 0 && a.nj == 16, RTDM_E_ARG, "split BF16 Taylor terms need b = 4 row runs of 16");
    const int remap = xcd_chunk_for((a.nch + 3) / 4);
    hipLaunchKernelGGL(k_spgemm_b4r16, dim3(xcd_grid((a.nch + 3) / 4, remap)), dim3(256), 0, s, a.nch, a.ch_off, a.ch_a,
                       a.ch_b, a.ch_out, a16, b16, c16, a.alpha_re, u, u_sign, remap);
    RT_HIP(hipGetLastError());
}

void launch_spgemm_r32(hipStream_t s, const SpgemmArgs &a, const float *a32, const float *b32, float *c32,
                       const float *zero32)
{
    if (a.nout == 0) return;
    RT_CHECK(a.b == 13, RTDM_E_UNSUPPORTED, "FP32 step products of this form need b = 13");
    if (a.nch > 0) {
        const int remap = xcd_chunk();
        const unsigned grid = xcd_grid((a.nch + 3) / 4, remap);
#define RT_R32J(NJ)                                                                                     \
    hipLaunchKernelGGL((k_spgemm_q4jr32<13, NJ>), dim3(grid), dim3(256), 0, s, a.nch, a.ch_off, a.ch_a, \
                       a.ch_b, a.ch_out, a32, b32, c32, (float)a.alpha_re, zero32, a.ch_order, remap, a.ch_seg)
        if (a.nj == 2) RT_R32J(2);
        else if (a.nj == 3) RT_R32J(3);
        else if (a.nj == 4) RT_R32J(4);
        else {
            RT_CHECK(a.nj == 8, RTDM_E_ARG, "row runs of 2, 4 or 8 outputs");
            RT_R32J(8);
        }
#undef RT_R32J
        RT_HIP(hipGetLastError());
        return;
    }
    const int wpb = a.wpb;
    const unsigned grid = xcd_grid((a.nout + wpb - 1) / wpb);
#define RT_R32(W)                                                                                  \
    hipLaunchKernelGGL((k_spgemm_q4r32<13, W>), dim3(grid), dim3(64 * W), 0, s, a.nout, a.off, a.trip, \
                       a32, b32, c32, (float)a.alpha_re, zero32, a.order)
    if (wpb == 16) RT_R32(16);
    else if (wpb == 8) RT_R32(8);
    else RT_R32(4);
#undef RT_R32
    RT_HIP(hipGetLastError());
}

void launch_spgemm(hipStream_t s, const SpgemmArgs &a)
{
    if (a.nout == 0) return;
    RT_CHECK(a.b >= 1 && a.b <= 16, RTDM_E_UNSUPPORTED, "block size must be 1..16");
    RT_CHECK(a.precision == RTDM_PREC_FP64 || (a.b == 4 || a.b == 13), RTDM_E_UNSUPPORTED,
             "reduced-precision products need b = 4 or 13");
    RT_CHECK(a.precision != RTDM_PREC_FP16X2 || a.maxabs, RTDM_E_ARG, "FP16 split products need operand maxima");
    const dim3 g((unsigned)((a.nout + 3) / 4)), t(256);
    const bool ac = a.ai != nullptr, bc = a.bi != nullptr;
    if (ac && bc) dispatch_ops<true, true>(s, a, g, t);
    else if (ac) dispatch_ops<true, false>(s, a, g, t);
    else if (bc) dispatch_ops<false, true>(s, a, g, t);
    else dispatch_ops<false, false>(s, a, g, t);
    RT_HIP(hipGetLastError());
}

}  // namespace rtdm
