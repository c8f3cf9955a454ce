// Stroboscopic-resampling baseline: nearest-neighbour reading of an
// oversampled segment on a uniform grid in the resampled time of
// Eq. (new_t), folded for an FFT at the requested bin spacing.  The grid
// times and nearest indices are computed in FP64 with the operations in a
// fixed order (no fused multiply-adds), so the integer decisions are those
// of the plain evaluation.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <string>

#include "../../include/nr_strobo.h"
#include "nr_params.hpp"

namespace {

thread_local std::string g_strobo_error;

nr_status fail(const std::string& m, nr_status st)
{
    g_strobo_error = m;
    return st;
}

// Value of a double in lane k (k the same in every lane).
__device__ __forceinline__ double lane_value(double v, int k)
{
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(b & 0xffffffffLL), k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), k);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// One thread per fold slot r of segment blockIdx.y: the grid points r,
// r + fold, ... < M, in that order.
template <bool CPLX>
__global__ __launch_bounds__(256) void plain_fold_kernel(const float* __restrict__ x, int64_t n, double fs_o, double a,
                                                         double tscale, int identity, int64_t M, int64_t fold,
                                                         float2* __restrict__ out)
{
#pragma clang fp contract(off)
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= fold) return;
    x += (int64_t)blockIdx.y * n * (CPLX ? 2 : 1);
    out += (int64_t)blockIdx.y * fold;
    float re = 0.0f, im = 0.0f;
    for (int64_t m = r; m < M; m += fold) {
        const double tau = (double)m / fs_o;
        const double t = identity ? tau : -expm1(1.6 * log1p(-tau / a)) * tscale;
        const double q = rint(t * fs_o);
        if (q >= 0.0 && q < (double)n) {
            const int64_t s = (int64_t)q;
            if (CPLX) {
                re += x[2 * s];
                im += x[2 * s + 1];
            } else {
                re += x[s];
            }
        }
    }
    out[r] = make_float2(re, im);
}

// The same for kSlots fold slots a thread, r = r0 + p 256 + threadIdx.x.
//
// The sample nearest to a grid point is rint of the inverse time map, whose
// log1p and expm1 in FP64 bound the kernel above (8 segments of 2^20 samples, a
// million grid points each: 52 us; 21 so).  The points of one workgroup and one
// multiple of the fold lie close together, so one evaluation in their middle
// (lane k does that for multiple k) serves them all: with z = d / (fs a y),
// d the distance in points and y = 1 - tau / a in the middle, the map is
// Q + G (1 - (1 - z)^1.6), G = fs tscale y^1.6, and the binomial series to z^4
// is off by less than 0.02 G z^5.  That integer is the plain evaluation's
// wherever the value lies further than both errors from a half-integer:
// 1e-6 samples for the series (the middle is taken only if its bound is ten
// times smaller) and 1e-14 of the value for roundings (the plain one takes
// about ten operations of 2^-53 each).  Elsewhere, about two points in a
// million, and where the series is not short enough, the plain evaluation
// decides.
constexpr int kSlots = 8;
template <bool CPLX>
__global__ __launch_bounds__(256) void fold_kernel(const float* __restrict__ x, int64_t n, double fs_o, double a,
                                                   double tscale, int64_t M, int64_t fold, float2* __restrict__ out)
{
#pragma clang fp contract(off)
    const int64_t r0 = (int64_t)blockIdx.x * (256 * kSlots);
    x += (int64_t)blockIdx.y * n * (CPLX ? 2 : 1);
    out += (int64_t)blockIdx.y * fold;
    constexpr double kHalf = 128.0 * kSlots;
    const int lane = threadIdx.x & 63;
    const double A = tscale * fs_o;
    float re[kSlots], im[kSlots];
#pragma unroll
    for (int p = 0; p < kSlots; ++p) re[p] = im[p] = 0.0f;
    for (int64_t m0 = r0; m0 < M; m0 += 64 * fold) {
        const double xm = ((double)(m0 + lane * fold) + kHalf) / fs_o / a;
        const double E = expm1(1.6 * log1p(-xm));        // y^1.6 - 1
        const double G = A * (1.0 + E), z1 = 1.0 / (fs_o * a * (1.0 - xm)), zm = kHalf * z1;
        const bool near = zm > 0.0 && zm < 0.1 && 0.02 * G * zm * zm * zm * zm * zm < 1e-7;
        const double mine = near ? z1 : NAN, Qm = -E * A;   // NAN: no comparison below holds
        for (int k = 0; k < 64 && m0 + k * fold < M; ++k) {
            const double zs = lane_value(mine, k), Q = lane_value(Qm, k), g = lane_value(G, k);
#pragma unroll
            for (int p = 0; p < kSlots; ++p) {
                const int at = p * 256 + threadIdx.x;
                const int64_t m = m0 + k * fold + at;
                if (r0 + at >= fold || m >= M) continue;
                const double z = ((double)at - kHalf) * zs;
                const double v = fma(g, z * fma(z, -fma(z, fma(z, 0.0224, 0.064), 0.48), 1.6), Q);
                double q = rint(v);
                if (!(fabs(v - q) < 0.5 - 1e-6 - 1e-14 * fabs(v)))
                    q = rint(-expm1(1.6 * log1p(-((double)m / fs_o) / a)) * tscale * fs_o);
                if (q >= 0.0 && q < (double)n) {
                    const int64_t s = (int64_t)q;
                    if (CPLX) {
                        re[p] += x[2 * s];
                        im[p] += x[2 * s + 1];
                    } else {
                        re[p] += x[s];
                    }
                }
            }
        }
    }
#pragma unroll
    for (int p = 0; p < kSlots; ++p) {
        const int64_t r = r0 + p * 256 + threadIdx.x;
        if (r < fold) out[r] = make_float2(re[p], im[p]);
    }
}

// Shared evaluations where eight slots a thread leave two workgroups a compute
// unit; below that, with one slot a thread, the series' one load at a time takes
// longer than the evaluations that it spares (1 x 2^20 samples on 2^18 slots 9.6
// us plain, 12.3 with the series; 8 x 2^18 on 2^16 16.9 and 22.3).  The identity
// has none to spare (8 x 2^20 samples: 14.8 us, 25.0).
constexpr int64_t kManyBlocks = 512;

template <bool CPLX>
void launch_fold(const float* x, int64_t n, int32_t n_seg, double fs_o, double a, double tscale, int identity,
                 int64_t M, int64_t fold, float2* out, hipStream_t st)
{
    const int64_t many = (fold + 256 * kSlots - 1) / (256 * kSlots);
    if (!identity && many * n_seg >= kManyBlocks)
        fold_kernel<CPLX><<<dim3((unsigned)many, (unsigned)n_seg), 256, 0, st>>>(x, n, fs_o, a, tscale, M, fold, out);
    else
        plain_fold_kernel<CPLX><<<dim3((unsigned)((fold + 255) / 256), (unsigned)n_seg), 256, 0, st>>>(
            x, n, fs_o, a, tscale, identity, M, fold, out);
}

// The grid of the segment: M and the constants of the inverse time map.
struct Grid {
    int64_t M;
    double a, tscale;
    int identity;
};

nr_status make_grid(double fs_o, int64_t n, double mc, double f0, Grid& g)
{
    if (!(std::isfinite(fs_o) && fs_o > 0.0) || n < 1 || !(std::isfinite(mc) && mc >= 0.0) ||
        !(std::isfinite(f0) && f0 > 0.0))
        return fail("fs_o, f0 must be positive, mc >= 0 and n_samples >= 1", NR_ERR_INVALID_ARG);
    const double b = mc > 0.0 ? nr::chirp_beta(mc, f0) : 0.0;
    const double t_last = (double)(n - 1) / fs_o;
    g.identity = b == 0.0;
    if (g.identity) {
        g.M = n;
        g.a = 0.0;
        g.tscale = 0.0;
        return NR_OK;
    }
    if (!(1.0 - (8.0 / 3.0) * b * t_last > 0.0)) return fail("the segment reaches coalescence", NR_ERR_INVALID_ARG);
    g.a = 3.0 / (5.0 * b);
    g.tscale = 3.0 / (8.0 * b);
    const double dtau_max = g.a * (-std::expm1(0.625 * std::log1p(-(8.0 / 3.0) * b * t_last)));
    g.M = (int64_t)std::floor(dtau_max * fs_o) + 1;
    return NR_OK;
}

}  // namespace

extern "C" {

nr_status nr_strobo_points(double fs_o, int64_t n_samples, double mc_msun, double f0, int64_t* m_out)
{
    if (!m_out) return fail("m_out is NULL", NR_ERR_INVALID_ARG);
    Grid g{};
    const nr_status st = make_grid(fs_o, n_samples, mc_msun, f0, g);
    if (st == NR_OK) *m_out = g.M;
    return st;
}

nr_status nr_strobo_fold(const void* x, int32_t x_complex, int64_t n_samples, int32_t n_seg, double fs_o,
                         double mc_msun, double f0, int64_t fold, void* out, void* stream)
{
    if (!x || !out) return fail("x and out must not be NULL", NR_ERR_INVALID_ARG);
    if (n_seg < 1 || n_seg > 65535) return fail("n_seg must be in [1, 65535]", NR_ERR_INVALID_ARG);
    if (fold < 1 || fold > (int64_t(1) << 34)) return fail("fold must be in [1, 2^34]", NR_ERR_INVALID_ARG);
    Grid g{};
    const nr_status st = make_grid(fs_o, n_samples, mc_msun, f0, g);
    if (st != NR_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    if (x_complex)
        launch_fold<true>((const float*)x, n_samples, n_seg, fs_o, g.a, g.tscale, g.identity, g.M, fold, (float2*)out, s);
    else
        launch_fold<false>((const float*)x, n_samples, n_seg, fs_o, g.a, g.tscale, g.identity, g.M, fold, (float2*)out, s);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(std::string("fold: ") + hipGetErrorString(e), NR_ERR_DEVICE);
    return NR_OK;
}

const char* nr_strobo_last_error(void) { return g_strobo_error.c_str(); }

}  // extern "C"
