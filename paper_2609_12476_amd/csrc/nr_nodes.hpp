// Band-limited nodes: the resampling sum over a segment's samples replaced by
// the same sum over far fewer points.
//
// The sum of an instance is X_m = sum_j x_j E_m(j), E_m(j) = exp(-2 pi i f_m
// dtau_j).  As a function of the sample index every E_m is a slow function
// times the carrier exp(-2 pi i f_ref j / fs): its local frequency f_m dtau'
// stays within a few hertz of f_ref.  A function of band half-width P is
// fixed by its values at nodes j_b = D b taken at a rate fs / D above 2 P,
//   E_m(j) exp(+2 pi i f_ref j / fs) = sum_b E_m(j_b) exp(+2 pi i f_ref j_b / fs) h((j - j_b) / D)
// with the interpolation kernel h (a Kaiser-windowed sinc of half-width H
// nodes: band-limited interpolation, the polyphase form of Crochiere and
// Rabiner), so that
//   X_m = sum_b z_b E_m(j_b),   z_b = sum_s x_{j_b + s} h(s / D) exp(-2 pi i f_ref s / fs).
// The z_b depend on the segment and on f_ref only: every template of a
// sub-band shares them, and an instance is a resampling sum over its nodes
// (about 120 for a 30 s segment and a 1 Hz sub-band instead of 7680 samples),
// the same type-I NUFFT (Sec. III.B, App. A) at the same tau.
//
//   node_filter    z of every (segment, f_ref, node), a short-time Fourier
//                  transform of the segment on the matrix cores.
//   node_spread    tau, heterodyne and ES spreading of an instance's nodes
//                  onto its grid in LDS, then the transform of the grid to
//                  the instance's modes (a small DFT on the matrix cores, or
//                  the Stockham FFT for large grids), deconvolution, power.
#pragma once

#include <algorithm>

#include "nr_fft.hpp"
#include "nr_internal.hpp"

namespace nr {

// ------------------------------------------------------- matrix products --

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// 16 x 16 tile of C += A B over four values of the contraction index: lane l
// gives A[m = l % 16][k = l / 16] and B[k = l / 16][n = l % 16]; accumulator
// i of lane l is C[mfma_row<T>(l / 16, i)][n = l % 16].
template <typename T>
struct Mfma;
template <>
struct Mfma<float> {
    using acc = f32x4;
    static __device__ __forceinline__ acc step(float a, float b, acc c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
};
template <>
struct Mfma<double> {
    using acc = f64x4;
    static __device__ __forceinline__ acc step(double a, double b, acc c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
};

// ---------------------------------------------------------------- filter --

// Reference frequencies are multiples of fs / Q, Q = kNodeRefs D, so the
// carrier repeats every Q samples and z is a short-time Fourier transform:
// the windowed samples around a node, folded modulo Q, times Q-point carriers
// (the weighted overlap-add filter bank of Crochiere and Rabiner).  With the
// window's symmetry and y(k) = sum_i h(k + Q i) x_{j_b + k + Q i},
//   Re z_b = sum_{k <= Q/2} cos(2 pi r k / Q) (y(k) + y(-k))   (k = 0, Q/2 halved)
//   Im z_b = -sum_{k <= Q/2} sin(2 pi r k / Q) (y(k) - y(-k)),
// two matrix products A B over Q / 2 + 1 values: A = carriers [16 references
// r of a tile][k], B = folded samples [k][16 nodes].
//
// One workgroup: 64 consecutive nodes (16 per wave) of one segment, MT tiles.
// Node windows overlap, so the samples are staged in LDS once and each lane
// folds the B values of its (k, node) itself, for all MT tiles: 2 I reads and
// 4 I operations beside 2 MT matrix steps.  A group of lanes whose read the
// 32 banks serve together (32 lanes in FP32: 16 nodes, two k; 16 in FP64)
// finds distinct banks for D = 2 (mod 4) in FP32 and odd D in FP64.  In FP32 two
// or four chains per product, from the window's small ends (k = kp - 1) to its
// centre, keep the rounding of the FP32 sums below that of the spreading:
// spectra of 20 sub-bands err by 2.0e-7 (relative l2) with the chains of the
// DFT below, 3.2e-7 from the centre outwards, 2.6e-7 on the sample path.
// Measured on the 1 h workload (120 segments of 7680 samples; 45 carriers at
// 128 nodes, 26 at 250): 106 us for a product of the unfolded taps (1260
// instead of 235 contraction steps per product), 44 us folded with two tiles a
// workgroup and node spacings of 4 (mod 8), whose reads met on half the banks,
// 35 us with up to four tiles, 29 us free of bank conflicts (the latency of
// 11 us of matrix steps at two waves a SIMD); beta bank 31 -> 20 us.
template <typename T, int MT, int I>
__device__ __forceinline__ void node_filter_block(const FilterItem& it, const T* __restrict__ strain,
                                                  const T* __restrict__ carriers, const T* __restrict__ window,
                                                  cpx<T>* __restrict__ z, T* __restrict__ lds)
{
    constexpr int IS = (I + 3) / 4 * 4;       // stride of the window's images of one k
    constexpr int R = I / 2;                  // images i = -R .. R
    const int D = it.D, Q = it.Q, kp = 16 * it.ksteps, reach = R * Q + kp;
    T* ws = lds;
    T* xs = lds + kp * IS;
    // window of the workgroup's nodes: sample w0 is xs[0]
    const int64_t w0 = (int64_t)it.j0 + (int64_t)it.node0 * D - reach;
    const int len = (kNodeTile - 1) * D + 2 * reach + 1;
    const T* __restrict__ src = strain + it.src_off;
    // 16 loads in flight per thread
    for (int q0 = threadIdx.x; q0 < len; q0 += 16 * kBlock) {
        T v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int64_t j = w0 + q0 + u * kBlock;
            v[u] = q0 + u * kBlock < len && j >= 0 && j < it.L ? src[j] : T(0);
        }
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (q0 + u * kBlock < len) xs[q0 + u * kBlock] = v[u];
    }
    for (int q0 = threadIdx.x; q0 < kp * IS; q0 += 8 * kBlock) {
        T v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = q0 + u * kBlock < kp * IS ? window[it.win_off + q0 + u * kBlock] : T(0);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (q0 + u * kBlock < kp * IS) ws[q0 + u * kBlock] = v[u];
    }
    __syncthreads();
    const int wave = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nn = lane & 15, kq = lane >> 4;
    const int node = 16 * wave + nn;
    // x at +k, -k of the node's centre, k = kp - 1 downwards
    const T* __restrict__ xp = xs + node * D + reach + (kp - 1 - kq);
    const T* __restrict__ xm = xs + node * D + reach - (kp - 1 - kq);
    const T* __restrict__ wk = ws + kq * IS;
    using V2 = cpx<T>;                                       // (cosine, -sine) of a lane
    const V2* __restrict__ tp = reinterpret_cast<const V2*>(carriers) + it.tap_off + lane;
    const int64_t tile = (int64_t)it.ksteps * 4 * 64;
    constexpr int CH = sizeof(T) == 8 ? 1 : MT <= 2 ? 4 : 2;  // chains
    typename Mfma<T>::acc re[MT][CH], im[MT][CH];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int c = 0; c < CH; ++c) re[t][c] = im[t][c] = typename Mfma<T>::acc{};
    V2 a[MT][4];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) a[t][c] = tp[t * tile + c * 64];
    for (int ks = 0; ks < it.ksteps; ++ks) {
        // the next step's carriers, in flight behind this step's products
        V2 an[MT][4];
        tp += ks + 1 < it.ksteps ? 256 : 0;
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c) an[t][c] = tp[t * tile + c * 64];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            T e = T(0), o = T(0);
#pragma unroll
            for (int i = -R; i <= R; ++i) {
                const T w = wk[4 * c * IS + i + R], p = xp[i * Q - 4 * c], m = xm[4 * c - i * Q];
                e = fma(w, p + m, e);
                o = fma(w, p - m, o);
            }
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                re[t][c % CH] = Mfma<T>::step(a[t][c].x, e, re[t][c % CH]);
                im[t][c % CH] = Mfma<T>::step(a[t][c].y, o, im[t][c % CH]);
            }
        }
        xp -= 16;
        xm += 16;
        wk += 16 * IS;
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c) a[t][c] = an[t][c];
    }
    const int b = it.node0 + node;
    if (b >= it.nodes) return;
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int f = kFilterRows * t + mfma_row(sizeof(T) == 8, kq, i);
            T r = re[t][0][i], q = im[t][0][i];
            if constexpr (CH == 2) {
                r += re[t][1][i];
                q += im[t][1][i];
            }
            if constexpr (CH == 4) {
                r = (r + re[t][1][i]) + (re[t][2][i] + re[t][3][i]);
                q = (q + im[t][1][i]) + (im[t][2][i] + im[t][3][i]);
            }
            z[it.z_off + (int64_t)f * it.nodes + b] = cpx<T>{r, q};
        }
}

// MAXT: the most tiles of any item of the launch (its registers set the
// kernel's occupancy: 16 accumulators a tile in FP32).
template <typename T, int I, int MAXT>
__global__ __launch_bounds__(kBlock) void node_filter_kernel(const FilterItem* __restrict__ items,
                                                             const T* __restrict__ strain,
                                                             const T* __restrict__ carriers,
                                                             const T* __restrict__ window, cpx<T>* __restrict__ z)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T* lds = reinterpret_cast<T*>(smem_raw);
    const FilterItem it = items[blockIdx.x];
    const int tiles = uniform(it.tiles);
    if (MAXT == 1 || tiles == 1)
        node_filter_block<T, 1, I>(it, strain, carriers, window, z, lds);
    else if (MAXT == 2 || tiles == 2)
        node_filter_block<T, 2, I>(it, strain, carriers, window, z, lds);
    else if (tiles == 3)
        node_filter_block<T, 3, I>(it, strain, carriers, window, z, lds);
    else
        node_filter_block<T, 4, I>(it, strain, carriers, window, z, lds);
}

// ---------------------------------------------------------------- spread --

// Instance records and series are the same for a whole wave: read through the
// constant address space they come over the scalar cache into scalar
// registers (after an LDS fence the compiler would otherwise load them per
// lane).
#define NR_CONST __attribute__((address_space(4)))
template <typename X>
__device__ __forceinline__ const NR_CONST X* as_const(const X* p)
{
    return (const NR_CONST X*)(uintptr_t)p;
}

// A record of whole 64-bit words at a wave-uniform address.
template <typename X>
__device__ __forceinline__ X load_const(const NR_CONST void* p)
{
    static_assert(sizeof(X) % 8 == 0 && alignof(X) <= 8, "whole words");
    const NR_CONST uint64_t* q = (const NR_CONST uint64_t*)p;
    uint64_t w[sizeof(X) / 8];
#pragma unroll
    for (size_t i = 0; i < sizeof(X) / 8; ++i) w[i] = q[i];
    X x;
    __builtin_memcpy(&x, w, sizeof x);
    return x;
}

// dtau at NP sample positions (series of dtau_of, uniform degree).
template <int NP, int N>
__device__ __forceinline__ void node_horner(const NR_CONST double* b, const double* x, double* out)
{
#pragma unroll
    for (int e = 0; e < NP; ++e) out[e] = b[N - 1];
#pragma unroll
    for (int k = N - 2; k >= 0; --k) {
#pragma unroll
        for (int e = 0; e < NP; ++e) out[e] = fma(out[e], x[e], b[k]);
    }
#pragma unroll
    for (int e = 0; e < NP; ++e) out[e] *= x[e];
}

template <int NP>
__device__ __forceinline__ void node_dtau(int ndeg, double c, const NR_CONST double* b, const double* x,
                                          double* out)
{
    switch (ndeg) {
    case 0:
#pragma unroll
        for (int e = 0; e < NP; ++e) out[e] = x[e] * c;
        return;
#define NR_N(N) \
    case N: node_horner<NP, N>(b, x, out); return;
        NR_N(1) NR_N(2) NR_N(3) NR_N(4) NR_N(5) NR_N(6) NR_N(7) NR_N(8) NR_N(9) NR_N(10) NR_N(11) NR_N(12)
#undef NR_N
    default:
        break;
    }
#pragma unroll
    for (int e = 0; e < NP; ++e) out[e] = b[ndeg - 1];
    for (int k = ndeg - 2; k >= 0; --k) {
#pragma unroll
        for (int e = 0; e < NP; ++e) out[e] = fma(out[e], x[e], b[k]);
    }
#pragma unroll
    for (int e = 0; e < NP; ++e) out[e] *= x[e];
}

// exp(-2 pi i ph) applied to z, ph in cycles.
__device__ __forceinline__ cpx<float> node_heterodyne(double ph, cpx<float> z)
{
    const float f = (float)(ph - rint(ph));
    const float cs = __builtin_amdgcn_cosf(f), sn = __builtin_amdgcn_sinf(f);
    return cpx<float>{z.x * cs + z.y * sn, z.y * cs - z.x * sn};
}
__device__ __forceinline__ cpx<double> node_heterodyne(double ph, cpx<double> z)
{
    double sn, cs;
    sincospi(2.0 * (ph - rint(ph)), &sn, &cs);
    return cpx<double>{z.x * cs + z.y * sn, z.y * cs - z.x * sn};
}

// Orders the LDS accesses of one wave's lanes among themselves (the hardware
// runs them in program order; no instruction is emitted).
__device__ __forceinline__ void lane_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Cells of a strip, real and imaginary part in one aligned word pair.
template <typename T>
struct Cell;
template <>
struct Cell<float> {
    typedef float v __attribute__((ext_vector_type(2)));
};
template <>
struct Cell<double> {
    typedef double v __attribute__((ext_vector_type(2)));
};

// Coefficients of the kernel pieces: per pair t < W / 2 the NE even, then the
// NE odd ones, read over the scalar cache; in FP32 the leading ones stay in
// vector registers (an fma reads one scalar operand only).
template <typename T, int W, int NE>
struct NodePoly;
template <int W, int NE>
struct NodePoly<float, W, NE> {
    const NR_CONST float* q;
    float lead[W];
    __device__ __forceinline__ void load(const void* p)
    {
        q = as_const(reinterpret_cast<const float*>(p));
#pragma unroll
        for (int k = 0; k < W; ++k) {
            lead[k] = q[k * NE + NE - 1];
            asm volatile("" : "+v"(lead[k]));
        }
    }
    __device__ __forceinline__ float top(int h) const { return lead[h]; }
    __device__ __forceinline__ float at(int h, int k) const { return q[h * NE + k]; }
    static __device__ __forceinline__ void fence() {}
};
template <int W, int NE>
struct NodePoly<double, W, NE> {
    const NR_CONST double* q;
    __device__ __forceinline__ void load(const void* p) { q = as_const(reinterpret_cast<const double*>(p)); }
    __device__ __forceinline__ double top(int h) const { return q[h * NE + NE - 1]; }
    __device__ __forceinline__ double at(int h, int k) const { return q[h * NE + k]; }
    // a pair's coefficients are not fetched before the last pair's are used up
    static __device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }
};

// The W tap values of NP nodes.  u = 1 - 2 frac(S) in (-1, 1]; tap t is
// E_t(u^2) + u O_t(u^2) and, the kernel being even, tap W - 1 - t is E_t(u^2)
// - u O_t(u^2): half the polynomial work (W even).
template <typename T, int W, int NE, int NP>
__device__ __forceinline__ void node_taps(const NodePoly<T, W, NE>& poly, const T* u, T (*a)[W])
{
    T u2[NP];
#pragma unroll
    for (int e = 0; e < NP; ++e) u2[e] = u[e] * u[e];
#pragma unroll
    for (int t = 0; t < W / 2; ++t) {
        T ev[NP], od[NP];
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            ev[e] = fma(poly.top(2 * t), u2[e], poly.at(2 * t, NE - 2));
            od[e] = fma(poly.top(2 * t + 1), u2[e], poly.at(2 * t + 1, NE - 2));
        }
#pragma unroll
        for (int k = NE - 3; k >= 0; --k)
#pragma unroll
            for (int e = 0; e < NP; ++e) {
                ev[e] = fma(ev[e], u2[e], poly.at(2 * t, k));
                od[e] = fma(od[e], u2[e], poly.at(2 * t + 1, k));
            }
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            a[e][t] = fma(u[e], od[e], ev[e]);
            a[e][W - 1 - t] = fma(-u[e], od[e], ev[e]);
        }
        poly.fence();
    }
}

// Two consecutive node values (a row's values are aligned to one value only).
template <typename T>
struct alignas(sizeof(T) * 2) NodePairHalf {
    T x, y;
};
template <typename T>
struct NodeValues {
    NodePairHalf<T> v[2];
};

// The nodes [first, first + count) of an instance onto the wave's strip of
// unwrapped cells; lane v takes nodes v * stride + r of them, r < stride.
// Returns the unwrapped cell of the strip's first position.
//
// The lanes' nodes lie at least one cell apart, so within one tap no two
// lanes meet and a plain read, add and write of the cell serves (an LDS
// addition ds_add_f32 of 64 lanes took about 240 cycles here, four a lane);
// the taps follow each other in program order.  Where consecutive nodes are
// less than a cell apart (pair), a lane's two nodes share W + 1 cells and
// their taps are summed in registers: 9 instead of 16 cell updates (W = 8).
// 1 h workload, 122,501 instances of about 121 nodes: 1430 us per step with
// LDS additions, 123 us with updates tap by tap, 94 us with the pairs, 88 us
// with node pairs loaded and placed together (273 VALU instructions an
// instance, 0.7 of their issue at the clock it runs at; the rest is the chain
// of updates and the scalar loads before it); its sample spreader, the
// cell-run kernel, takes 1240 us.
template <typename T, int W, int NE>
__device__ __forceinline__ int node_strip(const InstDev& d, const NodeArgs& a, const NodePoly<T, W, NE>& poly,
                                          int first, int count, int lane, typename Cell<T>::v* strip)
{
    using V = typename Cell<T>::v;
    const NR_CONST double* coef = as_const(a.coef + d.coef_off);
    const cpx<T>* __restrict__ z = reinterpret_cast<const cpx<T>*>(a.z) + d.strain_off + first;
    const double dfn = d.df * (double)a.n, hnn = 0.5 * (double)W;
    const double j0 = (double)(uniform((int)d.pt_off) + first * d.C), Cd = (double)d.C;
    const int hi = uniform((int)(d.pt_off >> 32));
    const int apart = (hi & 0xffff) + 1;            // lanes' nodes at least a cell apart
    const bool pair = hi > 0xffff;
    const int need = (count + kWave - 1) / kWave;
    const int stride = need > apart ? need : apart;
    int base = 0;
    for (int r0 = 0; r0 < stride; r0 += 2) {
        // nodes b and b + 1 of the lane; past the instance's last node the
        // values are dropped (the row's end is followed by a spare value)
        const int b = __mul24(lane, stride) + r0;
        const bool on0 = b < count, on1 = r0 + 1 < stride && b + 1 < count;
        NodeValues<T> zv = *reinterpret_cast<const NodeValues<T>*>(z + (on0 ? b : 0));
        double x[2], dt[2];
        x[0] = fma((double)b, Cd, j0);
        x[1] = x[0] + Cd;
        node_dtau<2>(d.ndeg, d.c, coef, x, dt);
        int g[2];
        T u[2], ta[2][W];
        cpx<T> c[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const double S = fma(dfn, dt[e], -hnn), fl = floor(S);
            g[e] = (int)fl;
            u[e] = (T)fma(-2.0, S - fl, 1.0);
            c[e] = node_heterodyne(d.fc * dt[e], cpx<T>{zv.v[e].x, zv.v[e].y});
        }
        if (r0 == 0) base = uniform(g[0]);
        if (on0) {
            V* cells = strip + (g[0] - base);
            node_taps<T, W, NE, 2>(poly, u, ta);
            if (pair) {
                if (!on1) c[1] = cpx<T>{T(0), T(0)};
                const bool same = !on1 || g[1] == g[0];
#pragma unroll
                for (int t = 0; t <= W; ++t) {
                    const T q = same ? (t < W ? ta[1][t < W ? t : 0] : T(0)) : (t > 0 ? ta[1][t > 0 ? t - 1 : 0] : T(0));
                    V v = cells[t];
                    if (t < W) {
                        v.x = fma(ta[0][t < W ? t : 0], c[0].x, v.x);
                        v.y = fma(ta[0][t < W ? t : 0], c[0].y, v.y);
                    }
                    v.x = fma(q, c[1].x, v.x);
                    v.y = fma(q, c[1].y, v.y);
                    cells[t] = v;
                    lane_order();
                }
            } else {
#pragma unroll
                for (int t = 0; t < W; ++t) {
                    V v = cells[t];
                    v.x = fma(ta[0][t], c[0].x, v.x);
                    v.y = fma(ta[0][t], c[0].y, v.y);
                    cells[t] = v;
                    lane_order();
                }
            }
        }
        lane_order();
        if (!pair && on1) {
            V* cells = strip + (g[1] - base);
            node_taps<T, W, NE, 1>(poly, u + 1, ta + 1);
#pragma unroll
            for (int t = 0; t < W; ++t) {
                V v = cells[t];
                v.x = fma(ta[1][t], c[1].x, v.x);
                v.y = fma(ta[1][t], c[1].y, v.y);
                cells[t] = v;
                lane_order();
            }
        }
        lane_order();
    }
    return base + 1;      // tap 0 of S lands on cell floor(S) + 1
}

// The outputs of bin k of an instance, as the fused epilogue writes them (of the
// class's own type: FP32 node classes have FP32 outputs): power rows (mode 1) or
// spectra and power at the bin offsets (mode 2).
template <typename T>
__device__ __forceinline__ void node_store(const NodeArgs& a, const EpilogueOut& o, const InstDev& d, int k, cpx<T> X)
{
    const T pw = X.x * X.x + X.y * X.y;
    if (o.mode == 1) {
        reinterpret_cast<T*>(o.rows)[a.row_base + (int64_t)d.entry * a.kmax + k] = pw;
    } else {
        if (o.spectra) reinterpret_cast<cpx<T>*>(o.spectra)[d.bin_off + k] = X;
        if (o.power) reinterpret_cast<T*>(o.power)[d.bin_off + k] = pw;
    }
}

__device__ __forceinline__ int floor_mod(int x, int n)
{
    const int r = x % n;
    return r < 0 ? r + n : r;
}

// Sum of the strip's cells that fold onto cell x of the periodic grid (base:
// the strip's first cell modulo n).
template <typename T, typename V>
__device__ __forceinline__ cpx<T> node_fold(const V* strip, int base, int len, int x, int n)
{
    int p = x - base;
    if (p < 0) p += n;
    cpx<T> s{T(0), T(0)};
    for (; p < len; p += n) {
        const V v = strip[p];
        s.x += v.x;
        s.y += v.y;
    }
    return s;
}

// Small grids (n <= kNodeDftMax): a workgroup takes 16 instances, four per
// wave, spreads each onto a strip of unwrapped cells in LDS, folds the strip
// onto the periodic grid in place (real parts, then imaginary parts), and
// transforms the 16 grids at once: X = F G with F [2 K][2 n] the DFT of the
// wanted modes with the deconvolution in its rows, a 16-column matrix product
// (FP32: in four chains; 128 cells in two of them erred by 2.6e-7 instead of
// 2.25e-7).
template <typename T, int W, int NE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 8 : 1))) void
node_spread_dft_kernel(NodeArgs a0, EpilogueOut o0)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T* lds = reinterpret_cast<T*>(smem_raw);
    const int wave = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t item0 = (int64_t)blockIdx.x * kNodeBatch;
    {
        const int n = a0.n, gs = a0.gstride, imo = a0.im_off;
        uint4* words = reinterpret_cast<uint4*>(smem_raw);
        for (int q = threadIdx.x; q < kNodeBatch * gs * (int)sizeof(T) / 16; q += kBlock) words[q] = uint4{0, 0, 0, 0};
        NodePoly<T, W, NE> poly;
        poly.load(a0.poly);
        __syncthreads();
#pragma unroll 1
        for (int q = 0; q < kNodeBatch / 4; ++q) {
            const int64_t item = item0 + wave * (kNodeBatch / 4) + q;
            if (item >= a0.count) break;
            const InstDev d = load_const<InstDev>(as_const(a0.inst + item));
            T* grid = lds + (wave * (kNodeBatch / 4) + q) * gs;
            auto* strip = reinterpret_cast<typename Cell<T>::v*>(grid);
            const int base = floor_mod(node_strip<T, W, NE>(d, a0, poly, 0, d.nodes, lane, strip), n);
            cpx<T> v[kNodeDftMax / kWave];
#pragma unroll
            for (int e = 0; e < kNodeDftMax / kWave; ++e)
                if (lane + e * kWave < n) v[e] = node_fold<T>(strip, base, a0.strip, lane + e * kWave, n);
            lane_order();
#pragma unroll
            for (int e = 0; e < kNodeDftMax / kWave; ++e)
                if (lane + e * kWave < n) {
                    grid[lane + e * kWave] = v[e].x;
                    grid[imo + lane + e * kWave] = v[e].y;
                }
        }
    }
    __syncthreads();
    // FP32: the arguments once more, from where the kernel got them (kept in
    // scalar registers across the spreading they would spill)
    NodeArgs a = a0;
    EpilogueOut o = o0;
    if constexpr (sizeof(T) == 4) {
        const NR_CONST char* args = (const NR_CONST char*)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(args));
        a = load_const<NodeArgs>(args);
        o = load_const<EpilogueOut>(args + sizeof(NodeArgs));
    }
    const int gs = a.gstride, imo = a.im_off;
    const int nn = lane & 15, kq = lane >> 4;
    const T* __restrict__ col = lds + nn * gs + kq;
    const int half = a.ksteps / 2;
    const int64_t item = item0 + nn;
    for (int tile = wave; tile < a.mtiles; tile += 4) {
        const T* __restrict__ A = reinterpret_cast<const T*>(a.dft) + (int64_t)tile * a.ksteps * 64 + lane;
        constexpr int CH = sizeof(T) == 8 ? 1 : 2;
        typename Mfma<T>::acc c0[CH] = {}, c1[CH] = {};
        for (int ks = 0; ks < half; ks += 4) {
            T ar[4], ai[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ar[e] = A[(ks + e) * 64];
                ai[e] = A[(half + ks + e) * 64];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                c0[e % CH] = Mfma<T>::step(ar[e], col[4 * (ks + e)], c0[e % CH]);
                c1[e % CH] = Mfma<T>::step(ai[e], col[imo + 4 * (ks + e)], c1[e % CH]);
            }
        }
        if (item >= a.count) continue;
        const InstDev* __restrict__ d = a.inst + item;
        const int K = d->K, q0 = 8 * tile + 2 * kq - a.m0max + d->m0;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int k = q0 + e;
            if (k < 0 || k >= K) continue;
            T xr = c0[0][2 * e] + c1[0][2 * e], xi = c0[0][2 * e + 1] + c1[0][2 * e + 1];
            if constexpr (CH == 2) {
                xr += c0[1][2 * e] + c1[1][2 * e];
                xi += c0[1][2 * e + 1] + c1[1][2 * e + 1];
            }
            node_store<T>(a, o, *d, k, cpx<T>{xr, xi});
        }
    }
}

// Large grids: a workgroup takes one instance; its four waves spread a
// quarter of the nodes each onto a strip of their own, the strips are folded
// onto the periodic grid and the workgroup runs the Stockham FFT (the grid at
// the start of LDS, its other half over the strips).
template <typename T, int W, int NE>
__global__ __launch_bounds__(kBlock) void node_spread_fft_kernel(NodeArgs a, EpilogueOut o)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ int bases[4];
    static_assert(sizeof(bases) == kNodeFftStaticLds, "counted by the plan");
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(smem_raw);
    const int wave = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n = a.n, len = a.strip;
    using V = typename Cell<T>::v;
    V* strips = reinterpret_cast<V*>(lds + n);
    const int64_t item = blockIdx.x;
    for (int q = threadIdx.x; q < 4 * len; q += kBlock) strips[q] = V{T(0), T(0)};
    __syncthreads();
    const InstDev d = load_const<InstDev>(as_const(a.inst + item));
    const int per = (d.nodes + 3) / 4, first = wave * per;
    const int count = d.nodes - first < per ? d.nodes - first : per;
    int base = 0;
    NodePoly<T, W, NE> poly;
    poly.load(a.poly);
    if (count > 0) base = node_strip<T, W, NE>(d, a, poly, first, count, lane, strips + wave * len);
    if (lane == 0) bases[wave] = floor_mod(base, n);
    __syncthreads();
    for (int c = threadIdx.x; c < n; c += kBlock) {
        cpx<T> s{T(0), T(0)};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const cpx<T> v = node_fold<T>(strips + q * len, bases[q], len, c, n);
            s.x += v.x;
            s.y += v.y;
        }
        lds[c] = s;
    }
    __syncthreads();
    const cpx<T>* res = fft_team<T>(lds, reinterpret_cast<const cpx<T>*>(a.twiddle), a.fft, threadIdx.x, kBlock);
    const T* __restrict__ dec = reinterpret_cast<const T*>(a.dec);
    for (int k = threadIdx.x; k < d.K; k += kBlock) {
        int l = k - d.m0;
        if (l < 0) l += n;
        const T f = dec[l];
        node_store<T>(a, o, d, k, cpx<T>{res[l].x * f, res[l].y * f});
    }
}

// -------------------------------------------------------------- launches --

// Workgroups of one launch at most: a launch holds fewer than 2^32 threads.
constexpr int64_t kMostBlocks = int64_t(1) << 23;

size_t filter_lds_bytes(int fp64, int D, int Q, int ksteps, int images)
{
    const int kp = 16 * ksteps, reach = images / 2 * Q + kp;
    return (size_t)((kNodeTile - 1) * D + 2 * reach + 1 + kp * ((images + 3) / 4 * 4)) * (fp64 ? 8 : 4);
}

template <typename T, int I, int MAXT>
static hipError_t launch_node_filter_k(const FilterLaunch& f, const void* strain, void* z, hipStream_t st)
{
    allow_lds(node_filter_kernel<T, I, MAXT>, f.lds);
    for (int64_t at = 0; at < f.count; at += kMostBlocks)
        node_filter_kernel<T, I, MAXT>
            <<<dim3((unsigned)std::min(f.count - at, kMostBlocks)), dim3(kBlock), f.lds, st>>>(
                f.items + at, (const T*)strain, (const T*)f.carriers, (const T*)f.window, (cpx<T>*)z);
    return hipGetLastError();
}

template <typename T, int I>
static hipError_t launch_node_filter_t(const FilterLaunch& f, const void* strain, void* z, hipStream_t st)
{
    if (f.tiles == 1) return launch_node_filter_k<T, I, 1>(f, strain, z, st);
    if (f.tiles == 2 || filter_tiles(sizeof(T) == 8) == 2) return launch_node_filter_k<T, I, 2>(f, strain, z, st);
    if constexpr (filter_tiles(sizeof(T) == 8) == 4) return launch_node_filter_k<T, I, 4>(f, strain, z, st);
    return hipErrorInvalidValue;
}

hipError_t launch_node_filter(const FilterLaunch& f, const void* strain, void* z, int strain_fp64, int fp64,
                              hipStream_t st)
{
    if (f.count <= 0) return hipSuccess;
    // (FP32 classes over double strain read samples: the strain has the nodes' type)
    if (strain_fp64 != fp64) return hipErrorInvalidValue;
    if (fp64)
        return f.images == 7 ? launch_node_filter_t<double, 7>(f, strain, z, st)
               : f.images == 9 ? launch_node_filter_t<double, 9>(f, strain, z, st)
                               : hipErrorInvalidValue;
    return f.images == 5 ? launch_node_filter_t<float, 5>(f, strain, z, st) : hipErrorInvalidValue;
}

template <typename T, int W, int NE>
static hipError_t launch_node_spread_k(const NodeArgs& a, const EpilogueOut& o, hipStream_t st)
{
    const bool small = a.mtiles > 0;
    const size_t lds = small ? (size_t)kNodeBatch * a.gstride * sizeof(T)
                             : node_fft_lds_bytes(sizeof(T) == 8, a.n, a.strip);
    const int64_t per = small ? kNodeBatch : 1;      // instances of a workgroup
    auto* kernel = small ? node_spread_dft_kernel<T, W, NE> : node_spread_fft_kernel<T, W, NE>;
    allow_lds(kernel, lds);
    for (int64_t at = 0; at < a.count; at += kMostBlocks * per) {
        NodeArgs q = a;
        q.inst = a.inst + at;
        q.count = std::min(a.count - at, kMostBlocks * per);
        kernel<<<dim3((unsigned)((q.count + per - 1) / per)), dim3(kBlock), lds, st>>>(q, o);
    }
    return hipGetLastError();
}

hipError_t launch_node_spread(const NodeArgs& a, int fp64, const EpilogueOut& o, hipStream_t st)
{
    if (a.count <= 0) return hipSuccess;
    if (!fp64 && a.w == 8) return launch_node_spread_k<float, 8, 4>(a, o, st);
    if (fp64 && a.w == 12) return launch_node_spread_k<double, 12, 7>(a, o, st);
    if (fp64 && a.w == 14) return launch_node_spread_k<double, 14, 9>(a, o, st);
    return hipErrorInvalidValue;
}

}  // namespace nr
