// gfx950 kernels of the learned proposal's network (see include/nr_mlp.h):
// bfloat16 weight copies, fused three-layer forward, backward through the
// activations, deterministic weight gradients, the loss, Adam, and the
// region feature builder.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <string>

#include "../../include/nr_mlp.h"

namespace {

constexpr int IN = NR_MLP_IN, HID = NR_MLP_HIDDEN, NP = NR_MLP_PARAMS;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + HID * IN, OFF_W2 = OFF_B1 + HID,
              OFF_B2 = OFF_W2 + HID * HID, OFF_W3 = OFF_B2 + HID, OFF_B3 = OFF_W3 + HID;
static_assert(OFF_B3 + 1 == NP, "parameter layout");
constexpr int BLK = 256;   // threads of the per-parameter and gradient kernels

thread_local std::string g_mlp_error;

// ---------------------------------------------------------------- bf16 --

typedef uint16_t bf16_t;

__device__ __forceinline__ bf16_t to_bf16(float f)
{
    // round to nearest, ties to even
    const uint32_t u = __float_as_uint(f);
    return (bf16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ float from_bf16(bf16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Weight copies used by the products, rows contiguous along the contraction
// index: W1 and W2 as they are, W2t[k][j] = W2[j][k] for the backward product.
__global__ void refresh_bf16_kernel(const float* __restrict__ p, bf16_t* __restrict__ w1,
                                    bf16_t* __restrict__ w2, bf16_t* __restrict__ w2t,
                                    bf16_t* __restrict__ w3)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < HID * IN) w1[i] = to_bf16(p[OFF_W1 + i]);
    if (i < HID * HID) {
        const int j = i / HID, k = i % HID;
        const bf16_t h = to_bf16(p[OFF_W2 + i]);
        w2[i] = h;
        w2t[k * HID + j] = h;
    }
    if (i < HID) w3[i] = to_bf16(p[OFF_W3 + i]);
}

// ------------------------------------------- forward and backward by rows --

// The products are dense [16 RT rows x KW] x [KW x HID] on the matrix cores.
// The weights are bfloat16 and the activations FP32; an activation is the exact
// sum of three bfloat16 values (its 24 significant bits in eights), so each
// product is three of v_mfma_f32_16x16x32_bf16 with FP32 accumulation, in a
// chain each that are added at the end: the products are exact and keep the
// FP32 activation precision (error against 64 bits: logits 3.1e-7 ->
// 1.4e-7, gradients 1.1e-7 -> 5.6e-8), in a fifth of the matrix cycles of FP32 products
// (3 x 16 instead of 8 x 32 per 32 values), which bound the kernel before: 16
// rows on one CU are 8200 cycles a 256 x 256 layer.
//
// The 16 waves of a workgroup own 16 output columns each; the weights of a
// layer are 8 (KW = 64: 2) loads of 16 bytes per lane, all in flight at once.
// Operand layout (lane l, m = l % 16, q = l / 16): A[m][8 q + e], B[8 q + e][n =
// m], e < 8; accumulator i of lane l is C[4 q + i][m].
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int WV = HID / 16;                 // waves of a row workgroup
constexpr int XS = IN + 8, HS = HID + 8;     // LDS row strides: 16 bytes times an odd number (no bank conflicts)

// The three parts of a finite v; an infinity or NaN is its own first part.
__device__ __forceinline__ void split3(float v, bf16_t* hi, bf16_t* mid, bf16_t* lo)
{
    const uint32_t u = __float_as_uint(v);
    const bool finite = (u & 0x7f800000u) != 0x7f800000u;
    const float a = __uint_as_float(u & 0xffff0000u);
    const uint32_t r = __float_as_uint(finite ? v - a : 0.0f);
    const float b = __uint_as_float(r & 0xffff0000u);
    *hi = (bf16_t)((u >> 16) | ((u & 0x7fffffffu) > 0x7f800000u ? 0x40u : 0u));
    *mid = (bf16_t)(r >> 16);
    *lo = (bf16_t)(__float_as_uint(__uint_as_float(r) - b) >> 16);
}

// Sum over the 16 lanes of a row (DPP rotations by 8, 4, 2 and 1).
template <int N>
__device__ __forceinline__ float rotate16(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xF, 0xF, false));
}
__device__ __forceinline__ float row_sum16(float v)
{
    v += rotate16<8>(v);
    v += rotate16<4>(v);
    v += rotate16<2>(v);
    return v + rotate16<1>(v);
}

template <int KW>
struct Weights {
    uint4 w[KW / 32];      // 8 bfloat16 each
    __device__ __forceinline__ void load(const bf16_t* __restrict__ rows, int n, int q)
    {
#pragma unroll
        for (int g = 0; g < KW / 32; ++g)
            w[g] = *reinterpret_cast<const uint4*>(rows + n * KW + 32 * g + 8 * q);
    }
};

// src: three planes of RT * 16 rows.
template <int RT, int KW, int STRIDE>
__device__ __forceinline__ void rows_times_weights(const bf16_t* __restrict__ src, const Weights<KW>& w, int m, int q,
                                                   floatx4* c)
{
    floatx4 d[RT][2];
#pragma unroll
    for (int t = 0; t < RT; ++t) d[t][0] = d[t][1] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int g = 0; g < KW / 32; ++g) {
        const bf16x8 b = __builtin_bit_cast(bf16x8, w.w[g]);
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const bf16_t* row = src + (16 * t + m) * STRIDE + 32 * g + 8 * q;
            const bf16x8 hi = *reinterpret_cast<const bf16x8*>(row);
            const bf16x8 mid = *reinterpret_cast<const bf16x8*>(row + RT * 16 * STRIDE);
            const bf16x8 lo = *reinterpret_cast<const bf16x8*>(row + 2 * RT * 16 * STRIDE);
            c[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, b, c[t], 0, 0, 0);
            d[t][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mid, b, d[t][0], 0, 0, 0);
            d[t][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, b, d[t][1], 0, 0, 0);
        }
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) c[t] += d[t][0] + d[t][1];
}

// Per 16 RT rows: z = network(x); TRAIN: also keeps h1 and h2 and goes back
// through the activations, dz = (sigmoid(z) - y) / B, da2 = dz w3 [h2 > 0],
// da1 = (da2 W2) [h1 > 0], the row's h1 still in registers.  A step of 1024
// rows: 16 to 17 us (22 with FP32 products); a forward kernel of 32 workgroups
// of four waves took 31 and a backward kernel 30.  Forward alone, 5120 rows:
// 11.3 us a call (20.8 before).
template <int RT, bool TRAIN>
__global__ __launch_bounds__(64 * WV) void rows_kernel(const float* __restrict__ x, const float* __restrict__ y,
                                                       int64_t B, const float* __restrict__ p,
                                                       const bf16_t* __restrict__ w1, const bf16_t* __restrict__ w2,
                                                       const bf16_t* __restrict__ w2t, const bf16_t* __restrict__ w3,
                                                       float* __restrict__ z_out, float* __restrict__ h1_out,
                                                       float* __restrict__ h2_out, float* __restrict__ dz_out,
                                                       float* __restrict__ da2_out, float* __restrict__ da1_out)
{
    constexpr int RB = 16 * RT;
    __shared__ __align__(16) bf16_t xs[3 * RB * XS];
    __shared__ __align__(16) bf16_t hs[3 * RB * HS];
    __shared__ float dzs[RB];
    float* red = reinterpret_cast<float*>(xs);       // [WV][RB], once the inputs are used up
    static_assert(sizeof(xs) >= WV * RB * sizeof(float), "row sums fit the inputs' place");
    const int t = threadIdx.x;
    const int l = t & 63, wv = t >> 6;
    const int m = l & 15, q = l >> 4;
    const int n = 16 * wv + m;                       // the lane's output column
    const int64_t r0 = (int64_t)blockIdx.x * RB;
    const int nr = (int)((B - r0) < RB ? (B - r0) : RB);
    Weights<IN> wa;
    Weights<HID> wb;
    wa.load(w1, n, q);
    wb.load(w2, n, q);
    const float b1 = p[OFF_B1 + n], b2 = p[OFF_B2 + n];
    const float w3n = from_bf16(w3[n]);
#pragma unroll
    for (int k = 0; k < RT; ++k) {
        const int i = t + 64 * WV * k, r = i / IN, f = i % IN;
        bf16_t* at = xs + r * XS + f;
        split3(r < nr ? x[(r0 + r) * IN + f] : 0.0f, at, at + RB * XS, at + 2 * RB * XS);
    }
    __syncthreads();
    floatx4 c[RT];
#pragma unroll
    for (int k = 0; k < RT; ++k) c[k] = floatx4{b1, b1, b1, b1};
    rows_times_weights<RT, IN, XS>(xs, wa, m, q, c);
    uint32_t on1 = 0;                                // [h1 > 0] of the lane's values
#pragma unroll
    for (int k = 0; k < RT; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 16 * k + 4 * q + i;
            const float v = fmaxf(c[k][i], 0.0f);
            bf16_t* at = hs + r * HS + n;
            split3(v, at, at + RB * HS, at + 2 * RB * HS);
            if (TRAIN) {
                on1 |= (v > 0.0f ? 1u : 0u) << (4 * k + i);
                if (r < nr) h1_out[(r0 + r) * HID + n] = v;
            }
        }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < RT; ++k) c[k] = floatx4{b2, b2, b2, b2};
    rows_times_weights<RT, HID, HS>(hs, wb, m, q, c);
    if (TRAIN) wb.load(w2t, n, q);                   // the backward product's, on their way
#pragma unroll
    for (int k = 0; k < RT; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 16 * k + 4 * q + i;
            c[k][i] = fmaxf(c[k][i], 0.0f);
            if (TRAIN && r < nr) h2_out[(r0 + r) * HID + n] = c[k][i];
            // sum over the wave's 16 columns of row r, in a fixed order
            const float v = row_sum16(c[k][i] * w3n);
            if (m == 0) red[wv * RB + r] = v;
        }
    __syncthreads();
    if (t < RB) {
        float v = 0.0f;
#pragma unroll
        for (int k = 0; k < WV; k += 4)
            v += (red[k * RB + t] + red[(k + 1) * RB + t]) + (red[(k + 2) * RB + t] + red[(k + 3) * RB + t]);
        v += p[OFF_B3];
        if (t < nr) z_out[r0 + t] = v;
        if (TRAIN) {
            float d = 0.0f;
            if (t < nr) {
                d = (1.0f / (1.0f + expf(-v)) - y[r0 + t]) / (float)B;
                dz_out[r0 + t] = d;
            }
            dzs[t] = d;
        }
    }
    if (!TRAIN) return;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < RT; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 16 * k + 4 * q + i;
            const float d = c[k][i] > 0.0f ? dzs[r] * w3n : 0.0f;
            bf16_t* at = hs + r * HS + n;
            split3(d, at, at + RB * HS, at + 2 * RB * HS);
            if (r < nr) da2_out[(r0 + r) * HID + n] = d;
        }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < RT; ++k) c[k] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    rows_times_weights<RT, HID, HS>(hs, wb, m, q, c);
#pragma unroll
    for (int k = 0; k < RT; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 16 * k + 4 * q + i;
            if (r < nr) da1_out[(r0 + r) * HID + n] = (on1 >> (4 * k + i)) & 1 ? c[k][i] : 0.0f;
        }
}

// ----------------------------------------------------------- gradients --

typedef float floatx16 __attribute__((ext_vector_type(16)));

// Row of accumulator e of the lanes l / 32 = h in a 32 x 32 matrix product.
__device__ __forceinline__ int tile_row(int e, int h) { return 8 * (e >> 2) + 4 * h + (e & 3); }

// Weight gradients as dense products on the matrix cores:
//   dW1[j][k] = sum_r da1[r][j] x[r][k],   dW2[j][k] = sum_r da2[r][j] h1[r][k],
// i.e. C = A B with A[j][r] = da[r][j] and B[r][k] = x[r][k] (or h1): the
// batch row r is the contraction index.  The batch is cut into chunks of rc
// rows; workgroup (strip, chunk) accumulates a 32 x 64 strip of one matrix over
// its chunk, each of its four waves over a quarter of the rows in two
// accumulator sets, with v_mfma_f32_32x32x2f32 (FP32 operands, so the gradient
// keeps FP32 precision); the eight partial strips are added in FP64 in a fixed
// order through LDS and stored in the chunk's partial gradient.  Lane (m, h) of
// a step over rows r, r + 1 supplies A[m][h] = da[r + h][j0 + m] and B[h][n = m]
// = src[r + h][k0 + m] (each a pair of coalesced 32-float row pieces);
// accumulator e of the lane is C[8 (e / 4) + 4 h + e % 4][m].
// The bias and output-vector gradients (db1, db2, dw3, db3) are VALU sums over
// the chunk by the remaining workgroups, one entry per lane; the last workgroup
// of the launch takes the loss.  A second pass adds the chunks' partials of
// every parameter in chunk order in FP64, so the gradient is bitwise
// reproducible.  Bound by the latency of its row loads; with the quarters added
// in LDS a 1024-row step leaves 4 partial gradients of 0.33 MB where chunks of
// 32 rows left 32: 9.3 us, 13.6 before, and the second pass 3.4 us, 4.4 before.
constexpr int kW1Strips = HID / 32;                    // 32 x 64 strips of dW1 (64 columns)
constexpr int kW2Strips = (HID / 32) * (HID / 64);     // of dW2
constexpr int kVecStrips = 3 * (HID / 64) + 1;         // db1, db2, dw3 by 64 entries; db3
constexpr int kGradStrips = kW1Strips + kW2Strips + kVecStrips;
constexpr int kMaxChunks = 64;
constexpr int kMinChunkRows = 256;

__host__ __device__ inline int grad_chunk_rows(int64_t B)
{
    // at most kMaxChunks chunks; a multiple of 16: two sets of row pairs in each of four waves
    int64_t rc = (B + kMaxChunks - 1) / kMaxChunks;
    if (rc < kMinChunkRows) rc = kMinChunkRows;
    return (int)((rc + 15) & ~int64_t(15));
}

__device__ void batch_loss(const float* __restrict__ z, const float* __restrict__ y, int64_t B, double* part,
                           float* __restrict__ loss);

__global__ __launch_bounds__(BLK) void weight_grad_partial_kernel(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ z,
    const float* __restrict__ h1, const float* __restrict__ h2, const float* __restrict__ dz,
    const float* __restrict__ da1, const float* __restrict__ da2, int64_t B, int rc, int n_chunks,
    float* __restrict__ part, float* __restrict__ loss)
{
    __shared__ float sums[8][32 * 64];           // 64 KB: the partial strips of the waves' sets
    const int strip = (int)(blockIdx.x % kGradStrips), chunk = (int)(blockIdx.x / kGradStrips);
    if (chunk >= n_chunks) {
        batch_loss(z, y, B, reinterpret_cast<double*>(&sums[0][0]), loss);
        return;
    }
    const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int m = l & 31, h = l >> 5;
    const int64_t c1 = (int64_t)(chunk + 1) * rc < B ? (int64_t)(chunk + 1) * rc : B;   // end of the chunk
    const int64_t r0 = (int64_t)chunk * rc + (int64_t)wv * (rc / 4);
    const int64_t r1 = r0 + rc / 4 < c1 ? r0 + rc / 4 : c1;
    const int64_t rm = r0 + rc / 8;              // first row of the wave's second set
    float* out = part + (int64_t)chunk * NP;
    if (strip < kW1Strips + kW2Strips) {
        const float* A;
        const float* S;
        int ld, j0, k0, off, ldw;
        if (strip < kW1Strips) {
            A = da1; S = x; ld = IN; j0 = 32 * strip; k0 = 0; off = OFF_W1; ldw = IN;
        } else {
            const int g = strip - kW1Strips;
            A = da2; S = h1; ld = HID; j0 = 32 * (g / (HID / 64)); k0 = 64 * (g % (HID / 64)); off = OFF_W2;
            ldw = HID;
        }
        for (int set = 0; set < 2; ++set) {
            const int64_t ra = set ? rm : r0, rb = set ? r1 : (rm < r1 ? rm : r1);
            floatx16 ca, cb;
#pragma unroll
            for (int e = 0; e < 16; ++e) ca[e] = cb[e] = 0.0f;
            for (int64_t r = ra; r < rb; r += 16) {
                float a[8], s0[8], s1[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int64_t rr = r + 2 * u + h;
                    const bool in = rr < rb;
                    a[u] = in ? A[rr * HID + j0 + m] : 0.0f;
                    s0[u] = in ? S[rr * ld + k0 + m] : 0.0f;
                    s1[u] = in ? S[rr * ld + k0 + 32 + m] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    ca = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u], s0[u], ca, 0, 0, 0);
                    cb = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u], s1[u], cb, 0, 0, 0);
                }
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                sums[2 * wv + set][tile_row(e, h) * 64 + m] = ca[e];
                sums[2 * wv + set][tile_row(e, h) * 64 + 32 + m] = cb[e];
            }
        }
        __syncthreads();
        for (int i = threadIdx.x; i < 32 * 64; i += BLK) {
            double s = 0.0;
#pragma unroll
            for (int u = 0; u < 8; ++u) s += (double)sums[u][i];
            out[off + (j0 + i / 64) * ldw + k0 + i % 64] = (float)s;
        }
        return;
    }
    // vector gradients: one entry per lane
    const int v = strip - kW1Strips - kW2Strips;
    const int which = v / (HID / 64);          // 0 db1, 1 db2, 2 dw3, 3 db3
    const int j = (v % (HID / 64)) * 64 + l;
    for (int set = 0; set < 2; ++set) {
        const int64_t ra = set ? rm : r0, rb = set ? r1 : (rm < r1 ? rm : r1);
        float s = 0.0f;
        if (which == 0) {
#pragma unroll 8
            for (int64_t r = ra; r < rb; ++r) s += da1[r * HID + j];
        } else if (which == 1) {
#pragma unroll 8
            for (int64_t r = ra; r < rb; ++r) s += da2[r * HID + j];
        } else if (which == 2) {
#pragma unroll 8
            for (int64_t r = ra; r < rb; ++r) s = fmaf(dz[r], h2[r * HID + j], s);
        } else {
#pragma unroll 8
            for (int64_t r = ra; r < rb; ++r) s += dz[r];
        }
        sums[2 * wv + set][l] = s;
    }
    __syncthreads();
    if (wv == 0) {
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) s += (double)sums[u][l];
        if (which < 3)
            out[(which == 0 ? OFF_B1 : which == 1 ? OFF_B2 : OFF_W3) + j] = (float)s;
        else if (l == 0)
            out[OFF_B3] = (float)s;
    }
}

// Mean of softplus(z) - y z over the batch by one workgroup in a fixed order
// (part: LDS of BLK doubles).
__device__ void batch_loss(const float* __restrict__ z, const float* __restrict__ y, int64_t B, double* part,
                           float* __restrict__ loss)
{
    double s = 0.0;
    for (int64_t r = threadIdx.x; r < B; r += BLK) {
        const double zz = z[r];
        const double sp = zz > 0.0 ? zz + log1p(exp(-zz)) : log1p(exp(zz));
        s += sp - (double)y[r] * zz;
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int o = BLK / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) part[threadIdx.x] += part[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = (float)(part[0] / (double)B);
}

__global__ __launch_bounds__(BLK) void loss_kernel(const float* __restrict__ z, const float* __restrict__ y, int64_t B,
                                                   float* __restrict__ loss)
{
    __shared__ double part[BLK];
    batch_loss(z, y, B, part, loss);
}

// The bfloat16 copies of parameter i (new value q) where the products read
// them (see refresh_bf16_kernel); biases have none.
__device__ __forceinline__ void store_bf16(int i, float q, bf16_t* __restrict__ w1, bf16_t* __restrict__ w2,
                                           bf16_t* __restrict__ w2t, bf16_t* __restrict__ w3)
{
    if (i < OFF_B1) {
        w1[i] = to_bf16(q);
    } else if (i >= OFF_W2 && i < OFF_B2) {
        const int q2 = i - OFF_W2;
        const bf16_t h = to_bf16(q);
        w2[q2] = h;
        w2t[(q2 % HID) * HID + q2 / HID] = h;
    } else if (i >= OFF_W3 && i < OFF_B3) {
        w3[i - OFF_W3] = to_bf16(q);
    }
}

// One thread per parameter.  FROM_PARTS: the gradient is the sum over the
// chunks, in chunk order, of the partial gradients (FP64; else it is read
// from grad_in).  It is stored to grad_out when given.  ADAM: one Adam update
// (beta1 0.9, beta2 0.999, eps 1e-8; c1, c2 the bias corrections) of the
// masters and moments, and the bfloat16 copies of the new masters.
template <bool FROM_PARTS, bool ADAM>
__global__ void update_kernel(const float* __restrict__ part, int n_chunks, const float* __restrict__ grad_in,
                              float* __restrict__ grad_out, float* __restrict__ p, float* __restrict__ m,
                              float* __restrict__ v, float lr, float c1, float c2, bf16_t* __restrict__ w1,
                              bf16_t* __restrict__ w2, bf16_t* __restrict__ w2t, bf16_t* __restrict__ w3)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NP) return;
    float gi;
    if (FROM_PARTS) {
        double s = 0.0;
#pragma unroll 8
        for (int c = 0; c < n_chunks; ++c) s += (double)part[(int64_t)c * NP + i];
        gi = (float)s;
    } else {
        gi = grad_in[i];
    }
    if (grad_out) grad_out[i] = gi;
    if (ADAM) {
        const float mi = 0.9f * m[i] + 0.1f * gi;
        const float vi = 0.999f * v[i] + 0.001f * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float q = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
        p[i] = q;
        store_bf16(i, q, w1, w2, w2t, w3);
    }
}

// ------------------------------------------------------------- features --

// One wave per (mc, sb) region: its lanes find the loudest bin (each the first
// of its own largest, then a butterfly that keeps the lower bin of equals) and
// build the 8 x 8 patch.  As with a scan in bin order from bin 0, NaN never
// replaces a value and a NaN in bin 0 stays.
__global__ __launch_bounds__(BLK) void region_features_kernel(const float* __restrict__ stat,
                                                              const int32_t* __restrict__ n_used, int n_mc,
                                                              int n_sub, int K, double norm, float* __restrict__ out)
{
    const int64_t region = (int64_t)blockIdx.x * (BLK / 64) + (threadIdx.x >> 6);
    if (region >= (int64_t)n_mc * n_sub) return;     // whole waves
    const int mc = (int)(region / n_sub), sb = (int)(region % n_sub);
    const int t = threadIdx.x & 63;
    const float* s = stat + region * K;
    float bv = -INFINITY;
    int best = INT_MAX;                              // no value yet
    for (int k = t; k < K; k += 64)
        if (s[k] > bv || (best == INT_MAX && s[k] == bv)) {
            bv = s[k];
            best = k;
        }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(bv, o);
        const int ob = __shfl_xor(best, o);
        if (ob != INT_MAX && (best == INT_MAX || ov > bv || (ov == bv && ob < best))) {
            bv = ov;
            best = ob;
        }
    }
    const float s0 = s[0];
    const int kstar = isnan(s0) || best == INT_MAX ? 0 : best;
    const int i = t >> 3, c = t & 7;
    int m2 = mc - 3 + i;
    m2 = m2 < 0 ? 0 : (m2 >= n_mc ? n_mc - 1 : m2);
    int k = kstar - 3 + c;
    k = k < 0 ? 0 : (k >= K ? K - 1 : k);
    const int tm = m2 * n_sub + sb;
    const double N = (double)n_used[tm];
    float z = 0.0f;
    if (N > 0.0) z = (float)(((double)stat[(int64_t)tm * K + k] * norm - N) / sqrt(N));
    out[(int64_t)region * 64 + t] = z;
}

}  // namespace

// ---------------------------------------------------------------- state --

struct nr_mlp_s {
    std::string err;
    hipStream_t stream = nullptr;
    int64_t max_batch = 0;
    int64_t step = 0;
    float *p = nullptr, *m = nullptr, *v = nullptr;
    bf16_t *w1 = nullptr, *w2 = nullptr, *w2t = nullptr, *w3 = nullptr;
    float *h1 = nullptr, *h2 = nullptr, *z = nullptr, *dz = nullptr, *da1 = nullptr, *da2 = nullptr;
    float* loss = nullptr;
    float* gpart = nullptr;   // per-chunk partial gradients [gchunks][NP]
    int gchunks = 0;
    ~nr_mlp_s()
    {
        for (void* q : {(void*)p, (void*)m, (void*)v, (void*)w1, (void*)w2, (void*)w2t,
                        (void*)w3, (void*)h1, (void*)h2, (void*)z, (void*)dz, (void*)da1, (void*)da2,
                        (void*)loss, (void*)gpart})
            if (q) (void)hipFree(q);
    }
};

namespace {

bool set_err(nr_mlp m, const std::string& s)
{
    if (m)
        m->err = s;
    else
        g_mlp_error = s;
    return false;
}

nr_status hip_status(nr_mlp m, hipError_t e, const char* what)
{
    if (e == hipSuccess) return NR_OK;
    set_err(m, std::string(what) + ": " + hipGetErrorString(e));
    return e == hipErrorOutOfMemory ? NR_ERR_OUT_OF_MEMORY : NR_ERR_DEVICE;
}

template <typename T>
hipError_t dalloc(T** ptr, size_t count)
{
    return hipMalloc((void**)ptr, count * sizeof(T));
}

nr_status refresh(nr_mlp m)
{
    refresh_bf16_kernel<<<(HID * HID + 255) / 256, 256, 0, m->stream>>>(m->p, m->w1, m->w2, m->w2t, m->w3);
    return hip_status(m, hipGetLastError(), "weight copies");
}

nr_status check_batch(nr_mlp m, int64_t B)
{
    if (B < 1 || B > m->max_batch) {   // (max_batch <= 2^26: a training batch is one launch)
        set_err(m, "batch size " + std::to_string(B) + " outside [1, " + std::to_string(m->max_batch) + "]");
        return NR_ERR_INVALID_ARG;
    }
    return NR_OK;
}

// Rows per workgroup of the row kernels: 16, the shortest chain, while every
// workgroup has a CU of its own, else 32, whose rows share each load of the
// weights (forward, 8192 rows: 11.5 us with 32, 16.2 with 16; 4096 rows: 9.0
// with 16).  One launch takes at most 2^26 rows (a launch holds fewer than
// 2^32 threads).
constexpr int64_t kRowBlocks16 = 256;
template <bool TRAIN>
nr_status run_rows(nr_mlp m, const float* x, const float* y, int64_t B, float* z)
{
    constexpr int64_t kMost = int64_t(1) << 26;
    for (int64_t b0 = 0; b0 < B; b0 += kMost) {
        const int64_t n = B - b0 < kMost ? B - b0 : kMost;
        if (n > 16 * kRowBlocks16)
            rows_kernel<2, TRAIN><<<(unsigned)((n + 31) / 32), 64 * WV, 0, m->stream>>>(
                x + b0 * IN, y, n, m->p, m->w1, m->w2, m->w2t, m->w3, z + b0, m->h1, m->h2, m->dz, m->da2, m->da1);
        else
            rows_kernel<1, TRAIN><<<(unsigned)((n + 15) / 16), 64 * WV, 0, m->stream>>>(
                x + b0 * IN, y, n, m->p, m->w1, m->w2, m->w2t, m->w3, z + b0, m->h1, m->h2, m->dz, m->da2, m->da1);
        const nr_status st = hip_status(m, hipGetLastError(), TRAIN ? "forward and backward" : "forward");
        if (st != NR_OK) return st;
    }
    return NR_OK;
}

// Bias corrections of the next Adam step (advances the step count).
void adam_corrections(nr_mlp m, float* c1, float* c2)
{
    m->step += 1;
    *c1 = (float)(1.0 - std::pow(0.9, (double)m->step));
    *c2 = (float)(1.0 - std::pow(0.999, (double)m->step));
}

// Gradient of the batch into grad (or NULL); lr > 0: followed by one Adam
// update in the same pass over the parameters.  Neither: the loss alone.
nr_status run_gradient(nr_mlp m, const float* x, const float* y, int64_t B, float* grad, float* loss, float lr)
{
    nr_status st;
    if (!grad && !(lr > 0.0f)) {
        st = run_rows<false>(m, x, y, B, m->z);
        if (st != NR_OK || !loss) return st;
        loss_kernel<<<1, BLK, 0, m->stream>>>(m->z, y, B, loss);
        return hip_status(m, hipGetLastError(), "loss");
    }
    st = run_rows<true>(m, x, y, B, m->z);
    if (st != NR_OK) return st;
    const int rc = grad_chunk_rows(B);
    const int n_chunks = (int)((B + rc - 1) / rc);
    if (n_chunks > m->gchunks) {
        set_err(m, "internal: gradient chunks exceed the workspace");
        return NR_ERR_DEVICE;
    }
    weight_grad_partial_kernel<<<(unsigned)(kGradStrips * n_chunks + (loss ? 1 : 0)), BLK, 0, m->stream>>>(
        x, y, m->z, m->h1, m->h2, m->dz, m->da1, m->da2, B, rc, n_chunks, m->gpart, loss);
    if ((st = hip_status(m, hipGetLastError(), "weight gradients")) != NR_OK) return st;
    const unsigned ublocks = (NP + 255) / 256;
    if (lr > 0.0f) {
        float c1, c2;
        adam_corrections(m, &c1, &c2);
        update_kernel<true, true><<<ublocks, 256, 0, m->stream>>>(m->gpart, n_chunks, nullptr, grad, m->p, m->m,
                                                                  m->v, lr, c1, c2, m->w1, m->w2, m->w2t, m->w3);
    } else {
        update_kernel<true, false><<<ublocks, 256, 0, m->stream>>>(m->gpart, n_chunks, nullptr, grad, nullptr,
                                                                   nullptr, nullptr, 0.0f, 1.0f, 1.0f, nullptr,
                                                                   nullptr, nullptr, nullptr);
    }
    return hip_status(m, hipGetLastError(), "gradient sum / Adam");
}

nr_status run_adam(nr_mlp m, const float* grad, float lr)
{
    float c1, c2;
    adam_corrections(m, &c1, &c2);
    update_kernel<false, true><<<(NP + 255) / 256, 256, 0, m->stream>>>(nullptr, 0, grad, nullptr, m->p, m->m, m->v,
                                                                        lr, c1, c2, m->w1, m->w2, m->w2t, m->w3);
    return hip_status(m, hipGetLastError(), "adam");
}

}  // namespace

extern "C" {

nr_status nr_mlp_create(nr_mlp* out, int64_t max_batch, void* stream)
{
    if (!out) {
        g_mlp_error = "out is NULL";
        return NR_ERR_INVALID_ARG;
    }
    *out = nullptr;
    if (max_batch < 1 || max_batch > (int64_t(1) << 26)) {
        g_mlp_error = "max_batch must be in [1, 2^26]";
        return NR_ERR_INVALID_ARG;
    }
    nr_mlp m = new (std::nothrow) nr_mlp_s();
    if (!m) {
        g_mlp_error = "host allocation failed";
        return NR_ERR_OUT_OF_MEMORY;
    }
    m->stream = (hipStream_t)stream;
    m->max_batch = max_batch;
    hipError_t e = hipSuccess;
    const size_t act = (size_t)max_batch * HID;
    if (e == hipSuccess) e = dalloc(&m->p, NP);
    if (e == hipSuccess) e = dalloc(&m->m, NP);
    if (e == hipSuccess) e = dalloc(&m->v, NP);
    if (e == hipSuccess) e = dalloc(&m->w1, (size_t)HID * IN);
    if (e == hipSuccess) e = dalloc(&m->w2, (size_t)HID * HID);
    if (e == hipSuccess) e = dalloc(&m->w2t, (size_t)HID * HID);
    if (e == hipSuccess) e = dalloc(&m->w3, (size_t)HID);
    if (e == hipSuccess) e = dalloc(&m->h1, act);
    if (e == hipSuccess) e = dalloc(&m->h2, act);
    if (e == hipSuccess) e = dalloc(&m->da1, act);
    if (e == hipSuccess) e = dalloc(&m->da2, act);
    if (e == hipSuccess) e = dalloc(&m->z, (size_t)max_batch);
    if (e == hipSuccess) e = dalloc(&m->dz, (size_t)max_batch);
    if (e == hipSuccess) e = dalloc(&m->loss, 1);
    // chunks of any batch B <= max_batch: at most min(kMaxChunks, ceil(B / kMinChunkRows))
    m->gchunks = (int)std::min<int64_t>(kMaxChunks, (max_batch + kMinChunkRows - 1) / kMinChunkRows);
    if (e == hipSuccess) e = dalloc(&m->gpart, (size_t)m->gchunks * NP);
    if (e == hipSuccess) e = hipMemsetAsync(m->p, 0, NP * sizeof(float), m->stream);
    if (e == hipSuccess) e = hipMemsetAsync(m->m, 0, NP * sizeof(float), m->stream);
    if (e == hipSuccess) e = hipMemsetAsync(m->v, 0, NP * sizeof(float), m->stream);
    if (e != hipSuccess) {
        g_mlp_error = std::string("device allocation failed: ") + hipGetErrorString(e);
        delete m;
        return NR_ERR_OUT_OF_MEMORY;
    }
    if (refresh(m) != NR_OK) {
        g_mlp_error = m->err;
        delete m;
        return NR_ERR_DEVICE;
    }
    *out = m;
    return NR_OK;
}

nr_status nr_mlp_set_params(nr_mlp m, const float* host_params)
{
    if (!m || !host_params) return NR_ERR_INVALID_ARG;
    nr_status st = hip_status(m, hipMemcpyAsync(m->p, host_params, NP * sizeof(float), hipMemcpyHostToDevice, m->stream),
                              "parameter upload");
    if (st == NR_OK) st = hip_status(m, hipMemsetAsync(m->m, 0, NP * sizeof(float), m->stream), "moments");
    if (st == NR_OK) st = hip_status(m, hipMemsetAsync(m->v, 0, NP * sizeof(float), m->stream), "moments");
    if (st == NR_OK) st = refresh(m);
    if (st == NR_OK) st = hip_status(m, hipStreamSynchronize(m->stream), "parameter upload");
    m->step = 0;
    return st;
}

nr_status nr_mlp_get_params(nr_mlp m, float* host_params)
{
    if (!m || !host_params) return NR_ERR_INVALID_ARG;
    nr_status st = hip_status(m, hipMemcpyAsync(host_params, m->p, NP * sizeof(float), hipMemcpyDeviceToHost, m->stream),
                              "parameter download");
    if (st == NR_OK) st = hip_status(m, hipStreamSynchronize(m->stream), "parameter download");
    return st;
}

nr_status nr_mlp_get_state(nr_mlp m, float* host_state, int64_t* step)
{
    if (!m || !host_state || !step) return NR_ERR_INVALID_ARG;
    const size_t b = NP * sizeof(float);
    nr_status st = hip_status(m, hipMemcpyAsync(host_state, m->p, b, hipMemcpyDeviceToHost, m->stream), "state");
    if (st == NR_OK) st = hip_status(m, hipMemcpyAsync(host_state + NP, m->m, b, hipMemcpyDeviceToHost, m->stream), "state");
    if (st == NR_OK)
        st = hip_status(m, hipMemcpyAsync(host_state + 2 * NP, m->v, b, hipMemcpyDeviceToHost, m->stream), "state");
    if (st == NR_OK) st = hip_status(m, hipStreamSynchronize(m->stream), "state");
    if (st == NR_OK) *step = m->step;
    return st;
}

nr_status nr_mlp_set_state(nr_mlp m, const float* host_state, int64_t step)
{
    if (!m || !host_state || step < 0) return NR_ERR_INVALID_ARG;
    const size_t b = NP * sizeof(float);
    nr_status st = hip_status(m, hipMemcpyAsync(m->p, host_state, b, hipMemcpyHostToDevice, m->stream), "state");
    if (st == NR_OK) st = hip_status(m, hipMemcpyAsync(m->m, host_state + NP, b, hipMemcpyHostToDevice, m->stream), "state");
    if (st == NR_OK)
        st = hip_status(m, hipMemcpyAsync(m->v, host_state + 2 * NP, b, hipMemcpyHostToDevice, m->stream), "state");
    if (st == NR_OK) st = refresh(m);
    if (st == NR_OK) st = hip_status(m, hipStreamSynchronize(m->stream), "state");
    if (st == NR_OK) m->step = step;
    return st;
}

nr_status nr_mlp_forward(nr_mlp m, const float* x, int64_t B, float* logits)
{
    if (!m || !x || !logits) return NR_ERR_INVALID_ARG;
    if (B < 1) {
        set_err(m, "batch size must be >= 1");
        return NR_ERR_INVALID_ARG;
    }
    // inference keeps no activations, so any batch size streams through
    return run_rows<false>(m, x, nullptr, B, logits);
}

nr_status nr_mlp_gradient(nr_mlp m, const float* x, const float* y, int64_t B, float* grad, float* loss)
{
    if (!m || !x || !y) return NR_ERR_INVALID_ARG;
    nr_status st = check_batch(m, B);
    if (st != NR_OK) return st;
    return run_gradient(m, x, y, B, grad, loss, 0.0f);
}

nr_status nr_mlp_adam_step(nr_mlp m, const float* grad, float lr)
{
    if (!m || !grad || !(lr > 0.0f)) return NR_ERR_INVALID_ARG;
    return run_adam(m, grad, lr);
}

nr_status nr_mlp_train_step(nr_mlp m, const float* x, const float* y, int64_t B, float lr, float* loss)
{
    if (!m || !x || !y || !(lr > 0.0f)) return NR_ERR_INVALID_ARG;
    nr_status st = check_batch(m, B);
    if (st != NR_OK) return st;
    return run_gradient(m, x, y, B, nullptr, loss, lr);
}

nr_status nr_mlp_region_features(const float* stat, const int32_t* n_used, int32_t n_mc, int32_t n_sub,
                                 int32_t K, double norm, float* features, void* stream)
{
    if (!stat || !n_used || !features || n_mc < 1 || n_sub < 1 || K < 1 || K > 4096 || !(norm > 0.0)) {
        g_mlp_error = "invalid region feature arguments";
        return NR_ERR_INVALID_ARG;
    }
    region_features_kernel<<<(unsigned)(((int64_t)n_mc * n_sub + BLK / 64 - 1) / (BLK / 64)), BLK, 0,
                             (hipStream_t)stream>>>(
        stat, n_used, n_mc, n_sub, K, norm, features);
    return hip_status(nullptr, hipGetLastError(), "region features");
}

const char* nr_mlp_last_error(nr_mlp m) { return m ? m->err.c_str() : g_mlp_error.c_str(); }

void nr_mlp_destroy(nr_mlp m)
{
    if (!m) return;
    (void)hipStreamSynchronize(m->stream);
    delete m;
}

}  // extern "C"
