// Device code shared by the kernels: complex values, LDS additions and the
// mixed-radix Stockham FFT of a team of lanes.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "nr_internal.hpp"

namespace nr {

template <typename T>
struct cpx {
    T x, y;
};

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ void lds_add(float* p, float v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_add(double* p, double v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Kernels whose dynamic LDS exceeds 64 KiB must opt in to the larger limit.
template <typename K>
static void allow_lds(K* kernel, size_t bytes)
{
    if (bytes > 65536)
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// ------------------------------------------------------------------ FFT --

template <typename T>
__device__ __forceinline__ cpx<T> cmul(cpx<T> a, cpx<T> b)
{
    return cpx<T>{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename T>
__device__ __forceinline__ cpx<T> cadd(cpx<T> a, cpx<T> b)
{
    return cpx<T>{a.x + b.x, a.y + b.y};
}
template <typename T>
__device__ __forceinline__ cpx<T> csub(cpx<T> a, cpx<T> b)
{
    return cpx<T>{a.x - b.x, a.y - b.y};
}
// -i z
template <typename T>
__device__ __forceinline__ cpx<T> mul_mi(cpx<T> a)
{
    return cpx<T>{a.y, -a.x};
}

// In-register DFT of length R (forward sign): y_q = sum_r v_r exp(-2 pi i r q / R).
template <typename T>
__device__ __forceinline__ void dft_small(cpx<T>* v, int R)
{
    if (R == 2) {
        const cpx<T> a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if (R == 3) {
        const T s3 = T(0.86602540378443864676);
        const cpx<T> t = cadd(v[1], v[2]);
        const cpx<T> d = csub(v[1], v[2]);
        const cpx<T> m = cpx<T>{v[0].x - T(0.5) * t.x, v[0].y - T(0.5) * t.y};
        const cpx<T> r = cpx<T>{s3 * d.y, -s3 * d.x};  // -i s3 d
        v[0] = cadd(v[0], t);
        v[1] = cadd(m, r);
        v[2] = csub(m, r);
    } else if (R == 4) {
        const cpx<T> a = cadd(v[0], v[2]), b = csub(v[0], v[2]);
        const cpx<T> c = cadd(v[1], v[3]), d = csub(v[1], v[3]);
        v[0] = cadd(a, c);
        v[2] = csub(a, c);
        v[1] = cadd(b, mul_mi(d));
        v[3] = csub(b, mul_mi(d));
    } else {  // R == 5
        const T c1 = T(0.30901699437494742410), c2 = T(-0.80901699437494742410);
        const T s1 = T(0.95105651629515357212), s2 = T(0.58778525229247312917);
        const cpx<T> t1 = cadd(v[1], v[4]), d1 = csub(v[1], v[4]);
        const cpx<T> t2 = cadd(v[2], v[3]), d2 = csub(v[2], v[3]);
        const cpx<T> a1 = cpx<T>{v[0].x + c1 * t1.x + c2 * t2.x, v[0].y + c1 * t1.y + c2 * t2.y};
        const cpx<T> a2 = cpx<T>{v[0].x + c2 * t1.x + c1 * t2.x, v[0].y + c2 * t1.y + c1 * t2.y};
        const cpx<T> b1 = cpx<T>{s1 * d1.x + s2 * d2.x, s1 * d1.y + s2 * d2.y};
        const cpx<T> b2 = cpx<T>{s2 * d1.x - s1 * d2.x, s2 * d1.y - s1 * d2.y};
        v[0] = cadd(v[0], cadd(t1, t2));
        v[1] = cadd(a1, mul_mi(b1));
        v[4] = csub(a1, mul_mi(b1));
        v[2] = cadd(a2, mul_mi(b2));
        v[3] = csub(a2, mul_mi(b2));
    }
}

// Lanes cooperating on one transform: 16 for grids up to 128 points (sixteen
// transforms per workgroup), one wave up to 512, the whole workgroup above
// (which keeps the LDS of the largest grids within one workgroup).
__host__ __device__ __forceinline__ int team_size_for(int n) { return n <= 128 ? 16 : (n <= 512 ? kWave : kBlock); }

// Synchronise the lanes of a team: teams inside one wave only need their LDS
// writes completed (the wave runs in lockstep); larger teams use the
// workgroup barrier.  Uniform across the workgroup.
__device__ __forceinline__ void team_sync(int ts)
{
    if (ts > kWave) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
}

// Stockham autosort FFT of the team's n points (ping-pong between buf[0..n)
// and buf[n..2n)).  Pass with radix R and span Ns (product of the earlier
// radices): butterfly j (0 <= j < n/R) takes inputs j + r n/R, applies the
// twiddles exp(-2 pi i r k / (Ns R)) with k = j mod Ns, and writes output q
// to (j / Ns) Ns R + k + q Ns.  tw is the LDS copy of exp(-2 pi i t / n).
// Every lane of the workgroup runs every pass.  Returns the buffer holding
// the result.
// One pass of radix R (a compile-time constant, so the R values of a
// butterfly stay in registers).
template <typename T, int R>
__device__ __forceinline__ void fft_pass(const cpx<T>* src, cpx<T>* dst, const cpx<T>* tw, int n, int Ns, int tid,
                                         int ts)
{
    const int nb = n / R;
    const int twstep = n / (Ns * R);
    for (int j = tid; j < nb; j += ts) {
        const int k = j % Ns;
        cpx<T> v[R];
        v[0] = src[j];
#pragma unroll
        for (int r = 1; r < R; ++r) v[r] = cmul(src[j + r * nb], tw[r * k * twstep]);
        dft_small(v, R);
        const int base = (j / Ns) * Ns * R + k;
#pragma unroll
        for (int q = 0; q < R; ++q) dst[base + q * Ns] = v[q];
    }
}

template <typename T>
__device__ cpx<T>* fft_team(cpx<T>* buf, const cpx<T>* tw, const FftPlanDev& fp, int tid, int ts)
{
    const int n = fp.n;
    cpx<T>* src = buf;
    cpx<T>* dst = buf + n;
    int Ns = 1;
    const int nr = fp.nr;
    for (int p = 0; p < nr; ++p) {
        const int R = fp.radix[p];
        switch (R) {
        case 2: fft_pass<T, 2>(src, dst, tw, n, Ns, tid, ts); break;
        case 3: fft_pass<T, 3>(src, dst, tw, n, Ns, tid, ts); break;
        case 4: fft_pass<T, 4>(src, dst, tw, n, Ns, tid, ts); break;
        default: fft_pass<T, 5>(src, dst, tw, n, Ns, tid, ts); break;
        }
        team_sync(ts);
        cpx<T>* t = src;
        src = dst;
        dst = t;
        Ns *= R;
    }
    return src;
}

}  // namespace nr
