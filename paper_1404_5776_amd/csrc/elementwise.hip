// Block-wise and reduction kernels around the truncated products: Taylor-sum
// updates, Hermitisation, the kick, Mulliken charges, the on-site H model,
// observables and the block-Jacobi start of the inverse iteration.
//
// Every reduction is deterministic: a fixed grid of kRedBlocks workgroups,
// each thread summing a fixed strided subset in a fixed order, a fixed LDS
// tree per workgroup, then one workgroup summing the partials in a fixed
// tree.  Results are therefore bit-identical from run to run.
#include <cmath>

#include "internal.h"

namespace rtdm {

constexpr int kT = 256;

// ----------------------------------------------------------------- helpers

__device__ inline double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Reduction of 4 slots (0..2 sums, 3 max) over a workgroup of kT threads, in a
// fixed order: a shuffle tree per wave, then the waves' values in wave order.
// The result on every thread; sh holds 4 kT / 64 doubles and may be used again
// after the next workgroup barrier.
__device__ inline void block_reduce4(double v[4], double *sh)
{
    const int wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 3; ++k) v[k] = wave_sum(v[k]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v[3] = fmax(v[3], __shfl_xor(v[3], o, 64));
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) sh[4 * wv + k] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = sh[k];
#pragma unroll
        for (int w = 1; w < kT / 64; ++w) v[k] = k < 3 ? v[k] + sh[4 * w + k] : fmax(v[k], sh[4 * w + k]);
    }
}

__device__ inline void write_partials(double v[4], double *partials)
{
    __shared__ double sh[4 * (kT / 64)];
    block_reduce4(v, sh);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) partials[blockIdx.x * 4 + k] = v[k];
    }
}

// ----------------------------------------------------------------- elementwise

__global__ void k_axpby(int64_t n, double a, const double *__restrict__ x, double c,
                        const double *__restrict__ y, double *__restrict__ out)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x)
        out[e] = y ? a * x[e] + c * y[e] : a * x[e];
}

void launch_axpby(hipStream_t s, int64_t n, double a, const double *x, double c, const double *y,
                  double *out)
{
    if (n == 0) return;
    int64_t g = (n + kT - 1) / kT;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_axpby, dim3((unsigned)g), dim3(kT), 0, s, n, a, x, c, y, out);
    RT_HIP(hipGetLastError());
}

__global__ void k_add_identity(int64_t n_atoms, int b, const int32_t *__restrict__ diag, double val,
                               double *__restrict__ m)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_atoms * b) return;
    const int64_t i = e / b;
    const int a = (int)(e % b);
    m[(int64_t)diag[i] * b * b + a * b + a] += val;
}

void launch_add_identity(hipStream_t s, int64_t n_atoms, int b, const int32_t *diag, double val,
                         double *m)
{
    const int64_t n = n_atoms * b;
    if (n == 0) return;
    hipLaunchKernelGGL(k_add_identity, dim3((unsigned)((n + kT - 1) / kT)), dim3(kT), 0, s, n_atoms,
                       b, diag, val, m);
    RT_HIP(hipGetLastError());
}

// K_ij *= exp(i kappa . (r_i - r_j)), kappa that of atom i's group where `group`
// is set (pairs never cross groups in a block-diagonal batch: kappa[3 g ..]).
// kr_t, ki_t (nullable, b = 4 or 13): K as a right operand as well (see
// k_hermitize).  Bound: HBM (two planes read and written); a phase per block
// shared by 32 lanes instead of one per element was slower (4,096 atoms b = 13
// 1.0 -> 1.9 ms).
template <int B, typename I>
__global__ __launch_bounds__(kT) void k_kick(I n, int b, const int32_t *__restrict__ rowof,
                                             const int32_t *__restrict__ col, const double *__restrict__ xyz,
                                             const int32_t *__restrict__ group, const double *__restrict__ kappa,
                                             double kx, double ky, double kz, double *__restrict__ kr,
                                             double *__restrict__ ki, double *__restrict__ kr_t,
                                             double *__restrict__ ki_t)
{
    const I bs = B ? B : b, bb = bs * bs;
    for (I e = (I)blockIdx.x * kT + threadIdx.x; e < n; e += (I)gridDim.x * kT) {
        const I p = e / bb, w = e - p * bb;
        const int64_t i = rowof[p], j = col[p];
        if (group) {
            const int64_t g = group[i];
            kx = kappa[3 * g];
            ky = kappa[3 * g + 1];
            kz = kappa[3 * g + 2];
        }
        const double ph = kx * (xyz[3 * i] - xyz[3 * j]) + ky * (xyz[3 * i + 1] - xyz[3 * j + 1]) +
                          kz * (xyz[3 * i + 2] - xyz[3 * j + 2]);
        double sn, cs;
        sincos(ph, &sn, &cs);
        const double xr = kr[e], xi = ki[e];
        const double vr = cs * xr - sn * xi, vi = cs * xi + sn * xr;
        kr[e] = vr;
        ki[e] = vi;
        if (B && kr_t) {
            const I a = w / bs, c = w - a * bs;
            const int64_t o = (int64_t)p * bb + (B == 4 ? (int)(c * 4 + a) : pair_at(B, (int)c, (int)a));
            kr_t[o] = vr;
            ki_t[o] = vi;
        }
    }
}

void launch_kick(hipStream_t s, int64_t nnzb, int b, const int32_t *rowof, const int32_t *col, const double *xyz,
                 const int32_t *group, const double *kappa_g, const double kappa[3], double *kr, double *ki,
                 double *kr_t, double *ki_t)
{
    const int64_t n = nnzb * b * b;
    if (n == 0) return;
    RT_CHECK(!kr_t || b == 4 || b == 13, RTDM_E_ARG, "right-operand copies need b = 4 or 13");
    const double kx = kappa ? kappa[0] : 0.0, ky = kappa ? kappa[1] : 0.0, kz = kappa ? kappa[2] : 0.0;
    const int64_t g = std::min<int64_t>((n + kT - 1) / kT, 65536);
    const bool small = n + g * kT < ((int64_t)1 << 32);   // 32-bit index arithmetic
#define RT_KICK(B_, I_)                                                                                          \
    hipLaunchKernelGGL((k_kick<B_, I_>), dim3((unsigned)g), dim3(kT), 0, s, (I_)n, b, rowof, col, xyz, group,    \
                       kappa_g, kx, ky, kz, kr, ki, kr_t, ki_t)
    if (b == 4 && small) RT_KICK(4, uint32_t);
    else if (b == 4) RT_KICK(4, int64_t);
    else if (b == 13 && small) RT_KICK(13, uint32_t);
    else if (b == 13) RT_KICK(13, int64_t);
    else if (small) RT_KICK(0, uint32_t);
    else RT_KICK(0, int64_t);
#undef RT_KICK
    RT_HIP(hipGetLastError());
}

// K_ij[a][c] = (Kn_ij[a][c] + conj(Kn_ji[c][a])) / 2.  B: the block size when
// fixed at compile time (4, 13: the index divisions by constants), else 0.
// kr_t, ki_t (nullable, B = 4 or 13): K as the right operand of the next U K
// (transposed blocks, right pairs), written here instead of by a pass of its
// own over K before the product.
template <int B, typename I>
__device__ __forceinline__ void hermitize_block(I n, int b, const int32_t *__restrict__ trans,
                                                const double *__restrict__ knr,
                                                const double *__restrict__ kni,
                                                double *__restrict__ kr, double *__restrict__ ki,
                                                double *__restrict__ kr_t, double *__restrict__ ki_t,
                                                double *__restrict__ partials)
{
    const I bs = B ? B : b, bb = bs * bs;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (I e = (I)blockIdx.x * kT + threadIdx.x; e < n; e += (I)kRedBlocks * kT) {
        const I p = e / bb, w = e - p * bb;
        const I a = w / bs, c = w - a * bs;
        const int64_t pe = (int64_t)trans[p] * bb + c * bs + a;
        const double xr = knr[e], xi = kni[e], yr = knr[pe], yi = -kni[pe];
        const double hr = 0.5 * (xr + yr), hi = 0.5 * (xi + yi);
        kr[e] = hr;
        ki[e] = hi;
        if (B && kr_t) {
            const int64_t o = (int64_t)p * bb + (B == 4 ? (int)(c * 4 + a) : pair_at(B, (int)c, (int)a));
            kr_t[o] = hr;
            ki_t[o] = hi;
        }
        const double dr = xr - yr, di = xi - yi;
        v[0] += dr * dr + di * di;
        v[1] += xr * xr + xi * xi;
    }
    write_partials(v, partials);
}

template <int B, typename I>
__global__ __launch_bounds__(kT) void k_hermitize(I n, int b, const int32_t *__restrict__ trans,
                                                  const double *__restrict__ knr,
                                                  const double *__restrict__ kni,
                                                  double *__restrict__ kr, double *__restrict__ ki,
                                                  double *__restrict__ kr_t, double *__restrict__ ki_t,
                                                  double *__restrict__ partials)
{
    hermitize_block<B, I>(n, b, trans, knr, kni, kr, ki, kr_t, ki_t, partials);
}

void launch_hermitize(hipStream_t s, int64_t nnzb, int b, const int32_t *trans, const double *knr,
                      const double *kni, double *kr, double *ki, double *partials, double *kr_t, double *ki_t)
{
    RT_CHECK(!kr_t || b == 4 || b == 13, RTDM_E_ARG, "right-operand copies need b = 4 or 13");
    const int64_t n = nnzb * b * b;
    const bool small = n + (int64_t)kRedBlocks * kT < ((int64_t)1 << 32);   // 32-bit index arithmetic
#define RT_HERM(B_, I_)                                                                                       \
    hipLaunchKernelGGL((k_hermitize<B_, I_>), dim3(kRedBlocks), dim3(kT), 0, s, (I_)n, b, trans, knr, kni, kr, ki, \
                       kr_t, ki_t, partials)
    if (b == 4 && small) RT_HERM(4, uint32_t);
    else if (b == 4) RT_HERM(4, int64_t);
    else if (b == 13 && small) RT_HERM(13, uint32_t);
    else if (b == 13) RT_HERM(13, int64_t);
    else if (small) RT_HERM(0, uint32_t);
    else RT_HERM(0, int64_t);
#undef RT_HERM
    RT_HIP(hipGetLastError());
}

// q_i = Re sum_{j in S row i, (i,j) in K} sum_{a,c} K_ij[a][c] S_ji[c][a], W waves
// per atom, every K of a kick set in one launch.  The row's (block, element)
// pairs are flattened, 64 W per pass, so every lane works and a pass has
// 64 W independent loads.  Bound: the chain of dependent loads of a wave (the
// block maps, then K and S) and, before the block size was a constant, the
// 64-bit divisions of every pass.  Four waves per atom where the atoms alone
// leave the chip idle or an atom is long (b > 4): 64 atoms b = 4 9.7 -> 4.5
// us; three kicks of 380 atoms in clusters b = 13, three launches of 80 -> one
// of 50 us.
// prev (nullable) receives the old q_i (keep_old) or the new one, ref
// (nullable) the new one of the first K.
// The charges of a workgroup's atoms; block_at(kk, kb, w, a, c) gives element w = (a, c)
// of block kb of the real part of kick set kk's K.
template <int B, int W, typename F>
__device__ __forceinline__ void mulliken_block(int blk, int n_atoms, int n_k, int b, const int64_t *__restrict__ s_ptr,
                                               const int32_t *__restrict__ s_trans,
                                               const int32_t *__restrict__ s_to_k, const double *__restrict__ sv,
                                               double *__restrict__ q, double *__restrict__ prev, int keep_old,
                                               double *__restrict__ ref, F block_at)
{
    __shared__ double part[kT / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    constexpr int PER = kT / 64 / W;           // atoms per workgroup
    const int x0 = blk * PER + wv / W;         // (kick, atom) of this wave
    const bool live = x0 < n_atoms * n_k;
    const int kk = live ? x0 / n_atoms : 0, i = live ? x0 - kk * n_atoms : 0;
    const int bs = B ? B : b, bb = bs * bs;
    const int64_t p0 = s_ptr[i];
    const int nel = live ? (int)(s_ptr[i + 1] - p0) * bb : 0;
    double acc = 0.0;
#pragma unroll 4
    for (int x = (wv % W) * 64 + lane; x < nel; x += 64 * W) {
        const int pp = x / bb, w = x - pp * bb;
        const int64_t p = p0 + pp;
        const int kb = s_to_k[p];
        const int a = w / bs, c = w - a * bs;
        const double sval = sv[(int64_t)s_trans[p] * bb + c * bs + a];
        if (kb >= 0) acc += block_at(kk, kb, w, a, c) * sval;
    }
    acc = wave_sum(acc);
    if (W > 1) {
        if (lane == 0) part[wv] = acc;
        __syncthreads();
        if (wv % W == 0) {
            acc = part[wv];
#pragma unroll
            for (int k = 1; k < W; ++k) acc += part[wv + k];
        }
    }
    if (live && lane == 0 && wv % W == 0) {
        if (prev) prev[x0] = keep_old ? q[x0] : acc;
        if (ref && kk == 0) ref[i] = acc;
        q[x0] = acc;
    }
}

template <int B, int W>
__global__ __launch_bounds__(kT) void k_mulliken(int n_atoms, int n_k, int b, const int64_t *__restrict__ s_ptr,
                                                 const int32_t *__restrict__ s_trans,
                                                 const int32_t *__restrict__ s_to_k, const double *__restrict__ sv,
                                                 KPlanes kp, double *__restrict__ q, double *__restrict__ prev,
                                                 int keep_old, double *__restrict__ ref)
{
    const int bb = B ? B * B : b * b;
    mulliken_block<B, W>(blockIdx.x, n_atoms, n_k, b, s_ptr, s_trans, s_to_k, sv, q, prev, keep_old, ref,
                         [&](int kk, int kb, int w, int, int) { return kp.re[kk][(int64_t)kb * bb + w]; });
}

// Hermitise and the charges of the new K in one launch, for small systems: the
// first kRedBlocks workgroups hermitise, the others take the charges of one
// atom each from the same sums 0.5 (Kn_ij + Kn_ji^*) instead of waiting for K:
// two elements of Kn for one of K, against a launch.  A step of 64 atoms b = 4,
// all launches: 31.0 -> 26.9 us.
template <int B>
__global__ __launch_bounds__(kT) void k_hermitize_charges(uint32_t n, int b, const int32_t *__restrict__ trans,
                                                          const double *__restrict__ knr,
                                                          const double *__restrict__ kni, double *__restrict__ kr,
                                                          double *__restrict__ ki, double *__restrict__ kr_t,
                                                          double *__restrict__ ki_t, double *__restrict__ partials,
                                                          int n_atoms, const int64_t *__restrict__ s_ptr,
                                                          const int32_t *__restrict__ s_trans,
                                                          const int32_t *__restrict__ s_to_k,
                                                          const double *__restrict__ sv, double *__restrict__ q,
                                                          double *__restrict__ prev)
{
    if (blockIdx.x < kRedBlocks) {             // uniform across the workgroup
        hermitize_block<B, uint32_t>(n, b, trans, knr, kni, kr, ki, kr_t, ki_t, partials);
        return;
    }
    const int bs = B ? B : b, bb = bs * bs;
    mulliken_block<B, 4>(blockIdx.x - kRedBlocks, n_atoms, 1, b, s_ptr, s_trans, s_to_k, sv, q, prev, 1, nullptr,
                         [&](int, int kb, int w, int a, int c) {
                             const double x = knr[(int64_t)kb * bb + w];
                             const double y = knr[(int64_t)trans[kb] * bb + c * bs + a];
                             return 0.5 * (x + y);
                         });
}

// one wave per atom only for b <= 4 with enough atoms to fill the 1,024 SIMDs four times
// (by the atoms alone: a kick set's sums are those of a run with that kick only)
static bool mulliken_wide(int64_t n_atoms, int b) { return b > 4 || n_atoms < 4096; }

// Up to 2^20 elements of K.  Whole steps, two launches -> one, us: b = 4 31.0 -> 26.9 at
// 64 atoms (0.05 2^20 elements), 161 -> 156 at 400 (0.6), 315 -> 309 at 700 (1.1), 1,402 ->
// 1,381 at 2,500 (5.0); b = 13 63.6 -> 60.7 at 20 atoms (0.06), 354 -> 348 at 100 (0.95),
// 1,237 -> 1,222 at 250 (3.3).  One launch is 1 to 2 % faster beyond the line too, as far
// as measured; the line keeps the form to the systems whose step is a chain of launches.
// Four waves per atom as in launch_mulliken, so the sums are the same.
bool hermitize_charges_form(int64_t n_atoms, int64_t nnzb, int b)
{
    return nnzb * b * b <= ((int64_t)1 << 20) && mulliken_wide(n_atoms, b) && n_atoms > 0;
}

void launch_hermitize_charges(hipStream_t s, int64_t nnzb, int b, const int32_t *trans, const double *knr,
                              const double *kni, double *kr, double *ki, double *partials, double *kr_t,
                              double *ki_t, int64_t n_atoms, const int64_t *s_ptr, const int32_t *s_trans,
                              const int32_t *s_to_k, const double *sv, double *q, double *prev)
{
    RT_CHECK(hermitize_charges_form(n_atoms, nnzb, b), RTDM_E_ARG, "too large for one launch");
    RT_CHECK(!kr_t || b == 4 || b == 13, RTDM_E_ARG, "right-operand copies need b = 4 or 13");
#define RT_HC(B_)                                                                                                  \
    hipLaunchKernelGGL(k_hermitize_charges<B_>, dim3((unsigned)(kRedBlocks + n_atoms)), dim3(kT), 0, s,            \
                       (uint32_t)(nnzb * b * b), b, trans, knr, kni, kr, ki, kr_t, ki_t, partials, (int)n_atoms, s_ptr, \
                       s_trans, s_to_k, sv, q, prev)
    if (b == 4) RT_HC(4);
    else if (b == 13) RT_HC(13);
    else RT_HC(0);
#undef RT_HC
    RT_HIP(hipGetLastError());
}

void launch_mulliken(hipStream_t s, int64_t n_atoms, int n_k, int b, const int64_t *s_ptr, const int32_t *s_trans,
                     const int32_t *s_to_k, const double *sv, const KPlanes &k, double *q, double *prev, int keep_old,
                     double *ref)
{
    if (n_atoms == 0) return;
    RT_CHECK(n_k >= 1 && n_k <= kMaxKicks && n_atoms * n_k < INT32_MAX, RTDM_E_UNSUPPORTED, "too many charges");
    const bool wide = mulliken_wide(n_atoms, b);
    const int per = wide ? 1 : kT / 64;
    const dim3 g((unsigned)((n_atoms * n_k + per - 1) / per)), t(kT);
#define RT_MULL(B_, W_)                                                                                             \
    hipLaunchKernelGGL((k_mulliken<B_, W_>), g, t, 0, s, (int)n_atoms, n_k, b, s_ptr, s_trans, s_to_k, sv, k, q, prev, \
                       keep_old, ref)
    if (b == 4 && wide) RT_MULL(4, 4);
    else if (b == 4) RT_MULL(4, 1);
    else if (b == 13) RT_MULL(13, 4);
    else if (wide) RT_MULL(0, 4);
    else RT_MULL(0, 1);
#undef RT_MULL
    RT_HIP(hipGetLastError());
}

// H_ii += g (q_eff,i - q_ref,i) on the diagonal of atom i's block, with the
// charges at the step's time point q_eff = q_a + theta (q_x - q_y):
// extrapolation (q_x, q_y) = (q(t), q(t - dt)) or interpolation
// (q(t + dt), q(t)), q_a = q(t).
__global__ void k_onsite_shift(int64_t n_atoms, int b, const int32_t *__restrict__ diag,
                               const int32_t *__restrict__ nbf, double gain, const double *__restrict__ q_a,
                               double theta, const double *__restrict__ q_x, const double *__restrict__ q_y,
                               const double *__restrict__ q_ref, double *__restrict__ h)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_atoms * b) return;
    const int64_t i = e / b;
    const int a = (int)(e % b);
    if (nbf && a >= nbf[i]) return;            // a padded function of a smaller atom
    const double q = q_a[i] + theta * (q_x[i] - q_y[i]);
    h[(int64_t)diag[i] * b * b + a * b + a] += gain * (q - q_ref[i]);
}

// A = A0 + X D on the range of X and A, with A0 = P(X H0) and D the on-site
// term of the Mulliken model: D_jj = g (q_a + theta (q_x - q_y) - q_ref)_j on
// each of atom j's own functions.  Since D only scales block columns of X,
// P(X (H0 + D)) = P(X H0) + X D exactly in arithmetic; the sums are rounded
// differently from the product of X with H0 + D.
template <typename I>
__global__ void k_a_onsite(I n, int b, const int32_t *__restrict__ col, const int32_t *__restrict__ nbf,
                           double gain, const double *__restrict__ q_a, double theta,
                           const double *__restrict__ q_x, const double *__restrict__ q_y,
                           const double *__restrict__ q_ref, const double *__restrict__ a0,
                           const double *__restrict__ x, double *__restrict__ a)
{
    const I bb = (I)b * b;
    for (I e = (I)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (I)gridDim.x * blockDim.x) {
        const I p = e / bb;
        const int cc = (int)((e - p * bb) % (I)b);
        const int j = col[p];
        double v = a0[e];
        if (!nbf || cc < nbf[j]) {
            const double q = q_a[j] + theta * (q_x[j] - q_y[j]);
            v += x[e] * (gain * (q - q_ref[j]));
        }
        a[e] = v;
    }
}

void launch_a_onsite(hipStream_t s, int64_t nnzb, int b, const int32_t *col, const int32_t *nbf, double gain,
                     const double *q_a, double theta, const double *q_x, const double *q_y, const double *q_ref,
                     const double *a0, const double *x, double *a)
{
    const int64_t n = nnzb * b * b;
    if (n == 0) return;
    int64_t g = (n + kT - 1) / kT;
    if (g > 65536) g = 65536;
    // 32-bit index arithmetic (the divisions by b^2 and b) whenever it fits
    if (n + (int64_t)g * kT < ((int64_t)1 << 32))
        hipLaunchKernelGGL(k_a_onsite<uint32_t>, dim3((unsigned)g), dim3(kT), 0, s, (uint32_t)n, b, col, nbf, gain,
                           q_a, theta, q_x, q_y, q_ref, a0, x, a);
    else
        hipLaunchKernelGGL(k_a_onsite<int64_t>, dim3((unsigned)g), dim3(kT), 0, s, n, b, col, nbf, gain, q_a, theta,
                           q_x, q_y, q_ref, a0, x, a);
    RT_HIP(hipGetLastError());
}

void launch_onsite_shift(hipStream_t s, int64_t n_atoms, int b, const int32_t *diag, const int32_t *nbf, double gain,
                         const double *q_a, double theta, const double *q_x, const double *q_y,
                         const double *q_ref, double *h)
{
    const int64_t n = n_atoms * b;
    if (n == 0) return;
    hipLaunchKernelGGL(k_onsite_shift, dim3((unsigned)((n + kT - 1) / kT)), dim3(kT), 0, s, n_atoms,
                       b, diag, nbf, gain, q_a, theta, q_x, q_y, q_ref, h);
    RT_HIP(hipGetLastError());
}

// H_ij += (E(t) . ((r_i + r_j)/2 - r_c)) S_ij on the pattern of S, with the
// Gaussian profile E(t) = E0 exp(-(t - t0)^2 / (2 sigma^2)) at the device
// step time t = tt[0] + (st[1] + theta) tt[1] and r_c the centre of the
// group of atom i (centre[3 g..3 g+2]).
__global__ void k_field(int64_t nnzb, int b, const int32_t *__restrict__ rowof,
                        const int32_t *__restrict__ col, const double *__restrict__ xyz,
                        const int32_t *__restrict__ group, const double *__restrict__ centre,
                        const double *__restrict__ sv, double ex, double ey, double ez, double t0,
                        double sigma, const int64_t *__restrict__ st, const double *__restrict__ tt,
                        double theta, double *__restrict__ h)
{
    const int64_t bb = (int64_t)b * b;
    const double t = tt[0] + ((double)st[1] + theta) * tt[1];
    const double d = t - t0;
    const double f = exp(-(d * d) / (2.0 * sigma * sigma));
    const double E[3] = {ex * f, ey * f, ez * f};
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnzb * bb;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = e / bb;
        const int64_t i = rowof[p], j = col[p];
        const double *c = centre + 3 * (group ? group[i] : 0);
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) v += 0.5 * ((xyz[3 * i + k] - c[k]) + (xyz[3 * j + k] - c[k])) * E[k];
        h[e] += v * sv[e];
    }
}

void launch_field(hipStream_t s, int64_t nnzb, int b, const int32_t *rowof, const int32_t *col,
                  const double *xyz, const int32_t *group, const double *centre, const double *sv,
                  const double E0[3], double t0, double sigma, const int64_t *st, const double *tt,
                  double theta, double *h)
{
    const int64_t n = nnzb * (int64_t)b * b;
    if (n == 0) return;
    const int64_t g = std::min<int64_t>((n + kT - 1) / kT, 65536);
    hipLaunchKernelGGL(k_field, dim3((unsigned)g), dim3(kT), 0, s, nnzb, b, rowof, col, xyz, group, centre,
                       sv, E0[0], E0[1], E0[2], t0, sigma, st, tt, theta, h);
    RT_HIP(hipGetLastError());
}

// Damped transform of a dipole trace, one thread per frequency, the sum over
// time points in order: F[f](w) = sum_{k=0}^{n} f(t_k) exp((i w - gamma) t_k) dt,
// t_k = k dt, f = P - P0 (zero at k = 0; P(t_k) = trace[(k-1) * stride + off
// + 0..2] for k >= 1).  The field transform is -kappa (kick) or the sum over
// the Gaussian field sampled at t_k.  alpha[w][j] = F[P_j - P0_j] / F[E_j]
// (NaN where F[E_j] = 0), strength[w] = (2 w / pi) Im(sum_j alpha_jj / 3).
__global__ void k_spectrum(int64_t n_omega, const double *__restrict__ omega, double gamma, double dt,
                           int64_t n, const double *__restrict__ trace, int64_t stride, int64_t off,
                           double p0x, double p0y, double p0z, int kick, double kx, double ky, double kz,
                           double t0, double sigma, double *__restrict__ alpha, double *__restrict__ strength)
{
    const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= n_omega) return;
    const double om = omega[w];
    const double P0[3] = {p0x, p0y, p0z};
    const double E0[3] = {kx, ky, kz};
    double fr[3] = {0.0, 0.0, 0.0}, fi[3] = {0.0, 0.0, 0.0};
    double er[3] = {0.0, 0.0, 0.0}, ei[3] = {0.0, 0.0, 0.0};
    for (int64_t k = 0; k <= n; ++k) {
        const double t = (double)k * dt;
        const double m = exp(-gamma * t) * dt;
        double sn, cs;
        sincos(om * t, &sn, &cs);
        const double pr = m * cs, pi = m * sn;
        if (k > 0) {
            const double *row = trace + (k - 1) * stride + off;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const double f = row[j] - P0[j];
                fr[j] += pr * f;
                fi[j] += pi * f;
            }
        }
        if (!kick) {
            const double d = t - t0;
            const double g = exp(-(d * d) / (2.0 * sigma * sigma));
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                er[j] += pr * (E0[j] * g);
                ei[j] += pi * (E0[j] * g);
            }
        }
    }
    double tr_im = 0.0;
    for (int j = 0; j < 3; ++j) {
        double ar, ai;
        if (kick) {
            er[j] = -E0[j];
            ei[j] = 0.0;
        }
        if (er[j] == 0.0 && ei[j] == 0.0) {
            ar = ai = __builtin_nan("");
        } else {
            const double den = er[j] * er[j] + ei[j] * ei[j];
            ar = (fr[j] * er[j] + fi[j] * ei[j]) / den;
            ai = (fi[j] * er[j] - fr[j] * ei[j]) / den;
            tr_im += ai;
        }
        alpha[(w * 3 + j) * 2] = ar;
        alpha[(w * 3 + j) * 2 + 1] = ai;
    }
    if (strength) strength[w] = 2.0 * om / M_PI * (tr_im / 3.0);
}

void launch_spectrum(hipStream_t s, int64_t n_omega, const double *omega, double gamma, double dt, int64_t n,
                     const double *trace, int64_t stride, int64_t off, const double P0[3], int kick,
                     const double E0[3], double t0, double sigma, double *alpha, double *strength)
{
    if (n_omega == 0) return;
    hipLaunchKernelGGL(k_spectrum, dim3((unsigned)((n_omega + 63) / 64)), dim3(64), 0, s, n_omega, omega, gamma,
                       dt, n, trace, stride, off, P0[0], P0[1], P0[2], kick, E0[0], E0[1], E0[2], t0, sigma,
                       alpha, strength);
    RT_HIP(hipGetLastError());
}

// Dipole -sum (r_i - r_c) q_i and sum q_i of atoms a0 .. a1-1 about (cx, cy, cz),
// by one workgroup of kT threads: d[0..2] and d[3] on every thread.
__device__ inline void dipole_sums(int64_t a0, int64_t a1, const double *__restrict__ xyz,
                                   const double *__restrict__ centre, const double *__restrict__ q, double *sh,
                                   double d[4])
{
    const double cx = centre[0], cy = centre[1], cz = centre[2];
    double w[4] = {0.0, 0.0, 0.0, 0.0};
    double tr = 0.0;
    for (int64_t i = a0 + threadIdx.x; i < a1; i += kT) {
        const double qi = q[i];
        w[0] -= (xyz[3 * i] - cx) * qi;
        w[1] -= (xyz[3 * i + 1] - cy) * qi;
        w[2] -= (xyz[3 * i + 2] - cz) * qi;
        tr += qi;
    }
    block_reduce4(w, sh);
    __syncthreads();
    double u[4] = {tr, 0.0, 0.0, 0.0};
    block_reduce4(u, sh);
    __syncthreads();
    d[0] = w[0];
    d[1] = w[1];
    d[2] = w[2];
    d[3] = u[0];
}

// The kRedBlocks partials of a reduction summed by one workgroup (k_red_finish's
// order): v[0..2] sums, v[3] max, on every thread.
__device__ inline void finish_sums(const double *__restrict__ partials, double *sh, double v[4])
{
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < 3; ++k) v[k] = partials[t * 4 + k] + partials[(t + kT) * 4 + k];
    v[3] = fmax(partials[t * 4 + 3], partials[(t + kT) * 4 + 3]);
    block_reduce4(v, sh);
    __syncthreads();
}

__device__ inline double herm_error(double d2, double k2) { return k2 > 0.0 ? sqrt(d2 / k2) : 0.0; }

// Observables of the current K into `row` at time t (a single workgroup).
__global__ __launch_bounds__(kT) void k_observables(int64_t n, const double *__restrict__ xyz,
                                                    const double *__restrict__ centre,
                                                    const double *__restrict__ q,
                                                    const double *__restrict__ herm_sums, double t,
                                                    double *__restrict__ row)
{
    __shared__ double sh[4 * (kT / 64)];
    double d[4];
    dipole_sums(0, n, xyz, centre, q, sh, d);
    if (threadIdx.x == 0) {
        row[0] = t;
        row[1] = d[0];
        row[2] = d[1];
        row[3] = d[2];
        row[4] = d[3];
        row[5] = herm_sums ? herm_error(herm_sums[0], herm_sums[1]) : 0.0;
        row[6] = __builtin_nan("");
        row[7] = 0.0;
    }
}

void launch_observables(hipStream_t s, int64_t n_atoms, const double *xyz, const double *centre, const double *q,
                        const double *herm_sums, double t, double *row)
{
    hipLaunchKernelGGL(k_observables, dim3(1), dim3(kT), 0, s, n_atoms, xyz, centre, q, herm_sums, t, row);
    RT_HIP(hipGetLastError());
}

// End of a step, one launch: workgroup (k, 0) finishes kick k's Hermiticity sums
// and writes its trace row obs + k obs_stride + 8 st[0] at time tt[0] + (st[1] +
// 1) tt[1]; workgroup (k, 1 + g) writes group g's row; the last workgroup to
// finish (counted in st[2]) advances st[0] and st[1].  In small systems, where a
// step is a chain of launches, this stands for a launch each of the sums, the
// rows and the counters.
__global__ __launch_bounds__(kT) void k_step_tail(StepTail a)
{
    __shared__ double sh[4 * (kT / 64)];
    const int per = 1 + (int)a.n_groups, kk = blockIdx.x / per, j = blockIdx.x - kk * per;
    const double *q = a.q + (int64_t)kk * a.n;
    const int64_t row_at = a.st[0];
    double d[4];
    if (j == 0) {
        double v[4];
        finish_sums(a.partials + (int64_t)kk * kRedBlocks * 4, sh, v);
        dipole_sums(0, a.n, a.xyz, a.centre, q, sh, d);
        if (threadIdx.x == 0) {
            for (int k = 0; k < 4; ++k) a.herm[4 * kk + k] = v[k];
            double *row = a.obs + kk * a.obs_stride + 8 * row_at;
            row[0] = a.tt[0] + (double)(a.st[1] + 1) * a.tt[1];
            row[1] = d[0];
            row[2] = d[1];
            row[3] = d[2];
            row[4] = d[3];
            row[5] = herm_error(v[0], v[1]);
            row[6] = __builtin_nan("");
            row[7] = 0.0;
        }
    } else {
        const int64_t g = j - 1;
        dipole_sums(a.gptr[g], a.gptr[g + 1], a.xyz, a.centre_g + 3 * g, q, sh, d);
        if (threadIdx.x == 0) {
            double *o = a.obs_g + kk * a.obs_g_stride + (row_at * a.n_groups + g) * 4;
            for (int k = 0; k < 4; ++k) o[k] = d[k];
        }
    }
    // every thread of this workgroup has read st by now (the reductions above synchronise)
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd((unsigned long long *)&a.st[2], 1ull) == (unsigned long long)gridDim.x - 1) {
            a.st[0] = row_at + 1;
            a.st[1] += 1;
            a.st[2] = 0;
        }
    }
}

void launch_step_tail(hipStream_t s, int n_kicks, const StepTail &a)
{
    hipLaunchKernelGGL(k_step_tail, dim3((unsigned)(n_kicks * (1 + a.n_groups))), dim3(kT), 0, s, a);
    RT_HIP(hipGetLastError());
}

// One thread per atom: Gauss-Jordan with partial pivoting on [S_ii | I] in scratch.
__global__ void k_block_inverse(int64_t n_atoms, int b, const int32_t *__restrict__ s_diag,
                                const double *__restrict__ sv, const int32_t *__restrict__ x_diag,
                                double *__restrict__ xv, double *__restrict__ scratch)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_atoms) return;
    const int w = 2 * b;
    double *m = scratch + i * (int64_t)b * w;
    const double *src = sv + (int64_t)s_diag[i] * b * b;
    for (int r = 0; r < b; ++r)
        for (int c = 0; c < w; ++c) m[r * w + c] = c < b ? src[r * b + c] : (c - b == r ? 1.0 : 0.0);
    for (int col = 0; col < b; ++col) {
        int piv = col;
        double best = fabs(m[col * w + col]);
        for (int r = col + 1; r < b; ++r)
            if (fabs(m[r * w + col]) > best) { best = fabs(m[r * w + col]); piv = r; }
        if (piv != col)
            for (int c = 0; c < w; ++c) {
                const double tmp = m[col * w + c];
                m[col * w + c] = m[piv * w + c];
                m[piv * w + c] = tmp;
            }
        const double inv = 1.0 / m[col * w + col];
        for (int c = 0; c < w; ++c) m[col * w + c] *= inv;
        for (int r = 0; r < b; ++r) {
            if (r == col) continue;
            const double f = m[r * w + col];
            if (f != 0.0)
                for (int c = 0; c < w; ++c) m[r * w + c] -= f * m[col * w + c];
        }
    }
    double *dst = xv + (int64_t)x_diag[i] * b * b;
    for (int r = 0; r < b; ++r)
        for (int c = 0; c < b; ++c) dst[r * b + c] = m[r * w + b + c];
}

void launch_block_inverse(hipStream_t s, int64_t n_atoms, int b, const int32_t *s_diag,
                          const double *sv, const int32_t *x_diag, double *xv, double *scratch)
{
    if (n_atoms == 0) return;
    hipLaunchKernelGGL(k_block_inverse, dim3((unsigned)((n_atoms + 63) / 64)), dim3(64), 0, s,
                       n_atoms, b, s_diag, sv, x_diag, xv, scratch);
    RT_HIP(hipGetLastError());
}

__global__ void k_row_abs_max(int64_t n_atoms, int b, const int64_t *__restrict__ s_ptr,
                              const double *__restrict__ sv, double *__restrict__ atom_max)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_atoms) return;
    double best = 0.0;
    for (int a = 0; a < b; ++a) {
        double sum = 0.0;
        for (int64_t p = s_ptr[i]; p < s_ptr[i + 1]; ++p)
            for (int c = 0; c < b; ++c) sum += fabs(sv[p * b * b + a * b + c]);
        best = fmax(best, sum);
    }
    atom_max[i] = best;
}

void launch_row_abs_max(hipStream_t s, int64_t n_atoms, int b, const int64_t *s_ptr,
                        const double *sv, double *atom_max)
{
    if (n_atoms == 0) return;
    hipLaunchKernelGGL(k_row_abs_max, dim3((unsigned)((n_atoms + kT - 1) / kT)), dim3(kT), 0, s,
                       n_atoms, b, s_ptr, sv, atom_max);
    RT_HIP(hipGetLastError());
}

__global__ void k_transpose_blocks(int64_t nblocks, int b, const double *__restrict__ in,
                                   double *__restrict__ out)
{
    const int bb = b * b;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nblocks * bb;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = e / bb;
        const int w = (int)(e - p * bb);
        const int r = w / b, c = w - r * b;
        out[p * bb + c * b + r] = in[e];
    }
}

void launch_transpose_blocks(hipStream_t s, int64_t nblocks, int b, const double *in, double *out)
{
    const int64_t n = nblocks * b * b;
    if (n == 0) return;
    int64_t g = (n + kT - 1) / kT;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_transpose_blocks, dim3((unsigned)g), dim3(kT), 0, s, nblocks, b, in, out);
    RT_HIP(hipGetLastError());
}

// out_ji = in_ij^dagger for every block p = (i, j) of a pattern (trans[p] =
// the block (j, i)): out[trans[p]][c][r] = conj(in[p][r][c]).  B is the block
// size when fixed at compile time (4), else 0 and b is read at run time.
template <int B>
__global__ void k_conj_transpose(int64_t nnzb, int b, const int32_t *__restrict__ trans,
                                 const double *__restrict__ in_re, const double *__restrict__ in_im,
                                 double *__restrict__ out_re, double *__restrict__ out_im)
{
    const int bs = B ? B : b, bb = bs * bs;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnzb * bb;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = e / bb;
        const int w = (int)(e - p * bb);
        const int r = w / bs, c = w - r * bs;
        const int64_t o = (int64_t)trans[p] * bb + c * bs + r;
        out_re[o] = in_re[e];
        out_im[o] = -in_im[e];
    }
}

void launch_conj_transpose(hipStream_t s, int64_t nnzb, int b, const int32_t *trans, const double *in_re,
                           const double *in_im, double *out_re, double *out_im)
{
    const int64_t n = nnzb * b * b;
    if (n == 0) return;
    int64_t g = (n + kT - 1) / kT;
    if (g > 65536) g = 65536;
    if (b == 4)
        hipLaunchKernelGGL(k_conj_transpose<4>, dim3((unsigned)g), dim3(kT), 0, s, nnzb, b, trans, in_re, in_im,
                           out_re, out_im);
    else
        hipLaunchKernelGGL(k_conj_transpose<0>, dim3((unsigned)g), dim3(kT), 0, s, nnzb, b, trans, in_re, in_im,
                           out_re, out_im);
    RT_HIP(hipGetLastError());
}

// U^dagger with every block transposed: block trans[p] = conj(block p), element
// by element, b = 4.  Eight lanes move one 128-byte block as 16-byte pairs.
__global__ __launch_bounds__(kT) void k_conj_move4(int64_t n2, const int32_t *__restrict__ trans,
                                                   const double2 *__restrict__ in_re,
                                                   const double2 *__restrict__ in_im, double2 *__restrict__ out_re,
                                                   double2 *__restrict__ out_im)
{
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < n2; e += (int64_t)gridDim.x * kT) {
        const int64_t o = (int64_t)trans[e >> 3] * 8 + (e & 7);
        const double2 v = in_im[e];
        out_re[o] = in_re[e];
        out_im[o] = make_double2(-v.x, -v.y);
    }
}

void launch_conj_move(hipStream_t s, int64_t nnzb, int b, const int32_t *trans, const double *in_re,
                      const double *in_im, double *out_re, double *out_im)
{
    if (nnzb == 0) return;
    RT_CHECK(b == 4, RTDM_E_UNSUPPORTED, "conjugate moves need b = 4");
    const int64_t n2 = nnzb * 8, g = std::min<int64_t>((n2 + kT - 1) / kT, 65536);
    hipLaunchKernelGGL(k_conj_move4, dim3((unsigned)g), dim3(kT), 0, s, n2, trans, (const double2 *)in_re,
                       (const double2 *)in_im, (double2 *)out_re, (double2 *)out_im);
    RT_HIP(hipGetLastError());
}

__global__ void k_to_f32(int64_t nblocks, int b, int transpose, const double *__restrict__ in,
                         float *__restrict__ out)
{
    const int bb = b * b;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nblocks * bb;
         e += (int64_t)gridDim.x * blockDim.x) {
        int64_t o = e;
        if (transpose) {
            const int64_t p = e / bb;
            const int w = (int)(e - p * bb);
            const int r = w / b, c = w - r * b;
            o = p * bb + c * b + r;
        }
        out[o] = (float)in[e];
    }
}

void launch_to_f32(hipStream_t s, int64_t nblocks, int b, int transpose, const double *in, float *out)
{
    const int64_t n = nblocks * b * b;
    if (n == 0) return;
    int64_t g = (n + kT - 1) / kT;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_to_f32, dim3((unsigned)g), dim3(kT), 0, s, nblocks, b, transpose, in, out);
    RT_HIP(hipGetLastError());
}

__global__ void k_axpy_f32(int64_t n, double a, const float *__restrict__ x, double *__restrict__ y)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x)
        y[e] += a * (double)x[e];
}

void launch_axpy_f32(hipStream_t s, int64_t n, double a, const float *x, double *y)
{
    if (n == 0) return;
    int64_t g = (n + kT - 1) / kT;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_axpy_f32, dim3((unsigned)g), dim3(kT), 0, s, n, a, x, y);
    RT_HIP(hipGetLastError());
}

__global__ void k_fill(int64_t n, double v, double *__restrict__ out)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x)
        out[e] = v;
}

void launch_fill(hipStream_t s, int64_t n, double v, double *out)
{
    if (n == 0) return;
    int64_t g = (n + kT - 1) / kT;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)g), dim3(kT), 0, s, n, v, out);
    RT_HIP(hipGetLastError());
}

// Step state kept on the device so that one captured step can be replayed:
// st[0] = next trace row (0 with `reset`), st[1] = steps done in this call,
// st[2] = workgroups of k_step_tail done, and tt[0] = time at the start of the
// call, tt[1] = dt.
__global__ void k_step_begin(int64_t *st, double *tt, double t0, double dt, int reset)
{
    if (threadIdx.x == 0) {
        if (reset) st[0] = 0;
        st[1] = 0;
        st[2] = 0;
        tt[0] = t0;
        tt[1] = dt;
    }
}

void launch_step_begin(hipStream_t s, int64_t *st, double *tt, double t0, double dt, int reset)
{
    hipLaunchKernelGGL(k_step_begin, dim3(1), dim3(64), 0, s, st, tt, t0, dt, reset);
    RT_HIP(hipGetLastError());
}

// ----------------------------------------------------------------- reductions

// End of an inverse iteration: X' = 2 X - X W (into xw), the sums of ||X' - X||^2,
// ||X'||^2 and the largest change, and X' as an operand of the next products: B = 13
// left and right pairs, B = 4 transposed blocks (right), B = 0 neither.  Bound:
// memory; two matrices read and up to three written, where the update, the
// sums and the re-layouts in passes of their own moved nine and W was laid out
// in two more.  Inverse of 1,000 atoms b = 13, R_K 16: 22.8 -> 21.8 ms; of
// 32,768 atoms b = 4, R_K 12: 28.6 -> 25.9 ms.
template <int B>
__global__ __launch_bounds__(kT) void k_newton_update(int64_t n, const double *__restrict__ x,
                                                      double *__restrict__ xw, double *__restrict__ left,
                                                      double *__restrict__ right, double *__restrict__ partials)
{
    constexpr int BB = B * B;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < n; e += (int64_t)kRedBlocks * kT) {
        const double old = x[e], now = 2.0 * old - xw[e];
        xw[e] = now;
        if (B) {
            const int64_t p = e / (B ? BB : 1);
            const int w = (int)(e - p * BB), r = w / (B ? B : 1), c = w - r * B;
            if (B == 13) left[p * BB + pair_at(B, r, c)] = now;
            right[p * BB + (B == 4 ? c * 4 + r : pair_at(B, c, r))] = now;
        }
        const double d = now - old;
        v[0] += d * d;
        v[1] += now * now;
        v[3] = fmax(v[3], fabs(d));
    }
    write_partials(v, partials);
}

void launch_newton_update(hipStream_t s, int64_t n, int b, const double *x, double *xw, double *left, double *right,
                          double *partials)
{
    RT_CHECK(!right || (b == 13 && left) || (b == 4 && !left), RTDM_E_ARG, "operand forms of b = 4 or 13");
#define RT_NEWTON(B_) \
    hipLaunchKernelGGL(k_newton_update<B_>, dim3(kRedBlocks), dim3(kT), 0, s, n, x, xw, left, right, partials)
    if (right && b == 13) RT_NEWTON(13);
    else if (right) RT_NEWTON(4);
    else RT_NEWTON(0);
#undef RT_NEWTON
    RT_HIP(hipGetLastError());
}

__global__ __launch_bounds__(kT) void k_red_unitarity(int64_t nnzb_p, int b,
                                                      const int32_t *__restrict__ p_to_hs,
                                                      const double *__restrict__ sv,
                                                      const double *__restrict__ zr,
                                                      const double *__restrict__ zi,
                                                      double *__restrict__ partials)
{
    const int bb = b * b;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < nnzb_p * bb;
         e += (int64_t)kRedBlocks * kT) {
        const int64_t p = e / bb;
        const int w = (int)(e - p * bb);
        const int hs = p_to_hs[p];
        const double sval = hs >= 0 ? sv[(int64_t)hs * bb + w] : 0.0;
        const double dr = zr[e] - sval, di = zi[e];
        const double m2 = dr * dr + di * di;
        const double m = sqrt(m2);
        v[0] += m2;
        v[1] += m;
        v[3] = fmax(v[3], m);
    }
    write_partials(v, partials);
}

void launch_red_unitarity(hipStream_t s, int64_t nnzb_p, int b, const int32_t *p_to_hs,
                          const double *sv, const double *zr, const double *zi, double *partials)
{
    hipLaunchKernelGGL(k_red_unitarity, dim3(kRedBlocks), dim3(kT), 0, s, nnzb_p, b, p_to_hs, sv, zr,
                       zi, partials);
    RT_HIP(hipGetLastError());
}

__global__ __launch_bounds__(kT) void k_red_minus_identity(int64_t nnzb, int b,
                                                           const int32_t *__restrict__ rowof,
                                                           const int32_t *__restrict__ col,
                                                           const double *__restrict__ v,
                                                           double *__restrict__ partials)
{
    const int bb = b * b;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < nnzb * bb;
         e += (int64_t)kRedBlocks * kT) {
        const int64_t p = e / bb;
        const int w = (int)(e - p * bb);
        const double id = (rowof[p] == col[p] && w % (b + 1) == 0) ? 1.0 : 0.0;
        const double d = v[e] - id;
        acc[0] += d * d;
        acc[1] += fabs(d);
        acc[3] = fmax(acc[3], fabs(d));
    }
    write_partials(acc, partials);
}

void launch_red_minus_identity(hipStream_t s, int64_t nnzb, int b, const int32_t *rowof,
                               const int32_t *col, const double *v, double *partials)
{
    hipLaunchKernelGGL(k_red_minus_identity, dim3(kRedBlocks), dim3(kT), 0, s, nnzb, b, rowof, col, v,
                       partials);
    RT_HIP(hipGetLastError());
}

__global__ __launch_bounds__(kT) void k_red_sumsq(int64_t n, const double *__restrict__ x,
                                                  double *__restrict__ partials)
{
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < n; e += (int64_t)kRedBlocks * kT) {
        v[0] += x[e] * x[e];
        v[3] = fmax(v[3], fabs(x[e]));
    }
    write_partials(v, partials);
}

// Sum of the diagonal elements of the diagonal blocks (slot 0).
__global__ __launch_bounds__(kT) void k_red_trace(int64_t n_atoms, int b, const int32_t *__restrict__ diag,
                                                  const double *__restrict__ v, double *__restrict__ partials)
{
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x; e < n_atoms * b; e += (int64_t)kRedBlocks * kT) {
        const int64_t i = e / b;
        const int a = (int)(e - i * b);
        acc[0] += v[(int64_t)diag[i] * b * b + a * (b + 1)];
    }
    write_partials(acc, partials);
}

void launch_red_trace(hipStream_t s, int64_t n_atoms, int b, const int32_t *diag, const double *v,
                      double *partials)
{
    hipLaunchKernelGGL(k_red_trace, dim3(kRedBlocks), dim3(kT), 0, s, n_atoms, b, diag, v, partials);
    RT_HIP(hipGetLastError());
}

// Gershgorin row discs of a block-sparse matrix: for element row (i, a),
// lohi = (c - r, c + r) with c = a_(ia,ia) and r = sum over the row's other
// elements of |a| (blocks of the row in order, each block's row summed first).
__global__ void k_gershgorin(int64_t n_atoms, int b, const int64_t *__restrict__ rowptr,
                             const int32_t *__restrict__ diag, const double *__restrict__ v,
                             double *__restrict__ lohi)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_atoms * b) return;
    const int64_t i = e / b;
    const int a = (int)(e - i * b);
    const int64_t bb = (int64_t)b * b;
    double rs = 0.0;
    for (int64_t p = rowptr[i]; p < rowptr[i + 1]; ++p) {
        double t = 0.0;
        for (int c = 0; c < b; ++c) t += fabs(v[p * bb + a * b + c]);
        rs += t;
    }
    const double cen = v[(int64_t)diag[i] * bb + a * (b + 1)];
    const double rad = rs - fabs(cen);
    lohi[2 * e] = cen - rad;
    lohi[2 * e + 1] = cen + rad;
}

void launch_gershgorin(hipStream_t s, int64_t n_atoms, int b, const int64_t *rowptr, const int32_t *diag,
                       const double *v, double *lohi)
{
    const int64_t n = n_atoms * b;
    if (n == 0) return;
    hipLaunchKernelGGL(k_gershgorin, dim3((unsigned)((n + kT - 1) / kT)), dim3(kT), 0, s, n_atoms, b, rowptr, diag,
                       v, lohi);
    RT_HIP(hipGetLastError());
}

void launch_red_sumsq(hipStream_t s, int64_t n, const double *x, double *partials)
{
    hipLaunchKernelGGL(k_red_sumsq, dim3(kRedBlocks), dim3(kT), 0, s, n, x, partials);
    RT_HIP(hipGetLastError());
}

void launch_red_max(hipStream_t s, int64_t n, const double *x, double *partials)
{
    launch_red_sumsq(s, n, x, partials);
}

// One workgroup of kT threads sums kRedBlocks partials (kRedBlocks = 2 kT).
__global__ __launch_bounds__(kT) void k_red_finish(const double *__restrict__ partials,
                                                   double *__restrict__ out)
{
    __shared__ double sh[4 * (kT / 64)];
    double v[4];
    finish_sums(partials, sh, v);
    if (threadIdx.x == 0)
        for (int k = 0; k < 4; ++k) out[k] = v[k];
}

void launch_red_finish(hipStream_t s, const double *partials, double *out)
{
    static_assert(kRedBlocks == 2 * kT, "finish kernel assumes two partials per thread");
    hipLaunchKernelGGL(k_red_finish, dim3(1), dim3(kT), 0, s, partials, out);
    RT_HIP(hipGetLastError());
}

__global__ void k_unit_to_row(const double *__restrict__ unit_sums,
                              const double *__restrict__ s_norm2, double *__restrict__ row)
{
    if (threadIdx.x == 0) row[6] = sqrt(unit_sums[0] / s_norm2[0]);
}

void launch_unit_to_row(hipStream_t s, const double *unit_sums, const double *s_norm2, double *row)
{
    hipLaunchKernelGGL(k_unit_to_row, dim3(1), dim3(64), 0, s, unit_sums, s_norm2, row);
    RT_HIP(hipGetLastError());
}

// ----------------------------------------------------------------- layout

// re = in, im = 0: a real upload into a complex slot (the caller's data may sit
// on any 8-byte boundary, so 8 bytes a lane).
__global__ void k_copy_real(int64_t n, const double *__restrict__ in, double *__restrict__ re,
                            double *__restrict__ im)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        re[e] = in[e];
        im[e] = 0.0;
    }
}

void launch_copy_real(hipStream_t s, int64_t n, const double *in, double *re, double *im)
{
    if (n == 0) return;
    const int64_t g = std::min<int64_t>((n + kT - 1) / kT, 65536);
    hipLaunchKernelGGL(k_copy_real, dim3((unsigned)g), dim3(kT), 0, s, n, in, re, im);
    RT_HIP(hipGetLastError());
}

__global__ void k_split(int64_t n, const double *__restrict__ inter, double *__restrict__ re,
                        double *__restrict__ im)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x) {
        re[e] = inter[2 * e];
        if (im) im[e] = inter[2 * e + 1];
    }
}

void launch_split(hipStream_t s, int64_t n, const double *inter, double *re, double *im)
{
    if (n == 0) return;
    int64_t g = (n + kT - 1) / kT;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_split, dim3((unsigned)g), dim3(kT), 0, s, n, inter, re, im);
    RT_HIP(hipGetLastError());
}

__global__ void k_interleave(int64_t n, const double *__restrict__ re, const double *__restrict__ im,
                             double *__restrict__ inter)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x) {
        inter[2 * e] = re[e];
        inter[2 * e + 1] = im ? im[e] : 0.0;
    }
}

void launch_interleave(hipStream_t s, int64_t n, const double *re, const double *im, double *inter)
{
    if (n == 0) return;
    int64_t g = (n + kT - 1) / kT;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_interleave, dim3((unsigned)g), dim3(kT), 0, s, n, re, im, inter);
    RT_HIP(hipGetLastError());
}

// x[0] += v (one thread): a device scalar corrected in stream order.
__global__ void k_add_scalar(double *x, double v)
{
    if (threadIdx.x == 0) x[0] += v;
}

void launch_add_scalar(hipStream_t s, double *x, double v)
{
    hipLaunchKernelGGL(k_add_scalar, dim3(1), dim3(64), 0, s, x, v);
    RT_HIP(hipGetLastError());
}

}  // namespace rtdm

