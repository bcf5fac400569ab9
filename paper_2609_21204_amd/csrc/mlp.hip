// Surrogate network kernels and their C ABI (include/dybond_mlp.h).
//
// A 4 -> 128 -> 128 -> 2 perceptron trained with mean-squared error and
// Adam.  The 128 x 128 layer is a dense contraction over the minibatch, so
// it and both GEMMs of its backward pass run on the matrix cores
// (v_mfma_f32_16x16x16_bf16: bf16 operands, FP32 accumulation), one wave per
// 16 x 16 output tile; the 4-wide input layer, the 2-wide output layer, the
// bias and weight reductions over the minibatch and Adam are plain FP32
// lanes.  Reductions run over the minibatch in a fixed order, so a training
// run is reproducible bit for bit.  An Adam step is two launches: the rows
// (k_mlp_rows: everything that stays inside 16 rows) and the parameters
// (k_mlp_grads: everything that reduces over all rows).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <numeric>
#include <random>
#include <string>
#include <vector>

#include "../../include/dybond_mlp.h"

namespace {

constexpr int kIn = 4, kHid = 128, kOut = 2;
// offsets in the flat parameter vector
constexpr uint32_t kW1 = 0, kB1 = kW1 + kHid * kIn, kW2 = kB1 + kHid, kB2 = kW2 + kHid * kHid,
                   kW3 = kB2 + kHid, kB3 = kW3 + kOut * kHid, kNP = kB3 + kOut;
static_assert(kNP == DB_MLP_PARAMS, "parameter count");

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// FP32 -> bf16, round to nearest even (NaN kept quiet).
__device__ __forceinline__ uint16_t to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ float sigmoidf_(float z) { return 1.0f / (1.0f + expf(-z)); }
__device__ __forceinline__ float siluf_(float z) { return z / (1.0f + expf(-z)); }
__device__ __forceinline__ float dsiluf_(float z) {
    const float s = sigmoidf_(z);
    return s * (1.0f + z * (1.0f - s));
}

struct Net {
    float* p;          // FP32 master parameters
    float* m;          // Adam first moments
    float* v;          // Adam second moments
    float* g;          // gradient
    uint16_t* wb;      // bf16 copy of the parameter vector (weights used; biases unused)
    uint16_t* w2t;     // bf16 W2 transposed (k, h), for the layer's backward pass
    // minibatch of bp rows (a multiple of 16): what its gradients reduce over
    float* x;          // bp x 4
    float* a2;         // bp x 128
    float* dz3;        // bp x 2
    float* dz2;        // bp x 128
    float* dz1;        // bp x 128
    uint16_t* a1t;     // 128 x ld, bf16 SiLU(z1) transposed
    uint16_t* dz2t;    // 128 x ld, bf16 dz2 transposed
    uint32_t ld;       // rows the transposed arrays have room for
};

// bf16 copies of the weight matrices (biases are read in FP32), W2 also
// transposed.
__device__ __forceinline__ void round_param(const Net& N, uint32_t k, float p) {
    const uint16_t b = to_bf16(p);
    N.wb[k] = b;
    if (k >= kW2 && k < kB2) N.w2t[((k - kW2) % kHid) * kHid + (k - kW2) / kHid] = b;
}
__global__ void k_mlp_round(Net N) {
    const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < kNP) round_param(N, k, N.p[k]);
}

// One tile of 16 rows through the whole network, and with BACK back again
// down to dz1, in one workgroup of 8 waves.  Wave w owns the hidden units
// [16 w, 16 w + 16) in both hidden layers, in the output layout of the matrix
// cores (lane l holds rows 4 (l / 16) + j, j < 4, of unit 16 w + l % 16), so
// that the pre-activations z1 and z2 stay in the registers of the lane that
// needs them again in the backward pass and only bf16 operands and the
// 2-wide output layer go through LDS.  v_mfma_f32_16x16x16_bf16: lane l
// supplies A(l % 16, 4 (l / 16) + j) and B(4 (l / 16) + j, l % 16) as 8
// contiguous bytes each.  With a kernel per layer a minibatch cost 10
// launches, 160 us, at 256 rows; the layers of a tile depend on nothing
// outside it.  A workgroup takes the tiles blockIdx, blockIdx + grid, ...,
// and keeps its W2 fragments in registers over them.
// Rows come from X (and targets from Tt) by idx, or in order when idx is
// null; rows at or past nb are zeros whose outputs are ignored.
constexpr int kRowTile = 16, kRowThreads = 512;
constexpr int kLdA = kHid + 8;        // bf16 row stride in LDS (8-byte aligned, rows on other banks)
constexpr int kLdF = kHid + 4;        // FP32 row stride in LDS
template <bool BACK>
__global__ __launch_bounds__(kRowThreads) void k_mlp_rows(Net N, const float* __restrict__ X,
                                                          const float* __restrict__ Tt,
                                                          const uint32_t* __restrict__ idx, uint32_t nb,
                                                          uint32_t tiles, float* __restrict__ y_out) {
    __shared__ float4 xs[kRowTile];
    __shared__ float2 ts[kRowTile], dz3s[kRowTile];
    __shared__ __attribute__((aligned(16))) uint16_t ab[kRowTile * kLdA];
    __shared__ __attribute__((aligned(16))) uint16_t db[kRowTile * kLdA];
    __shared__ __attribute__((aligned(16))) float a2s[kRowTile * kLdF];
    __shared__ __attribute__((aligned(16))) float w3s[kOut * kHid];
    const int tid = (int)threadIdx.x, l = tid & 63, r = l & 15, q4 = (l >> 4) * 4;
    const uint32_t h = (uint32_t)(tid >> 6) * 16u + (uint32_t)r;       // this lane's hidden unit
    // what depends on the weights alone
    bf16x4 w2f[kHid / 16];
#pragma unroll
    for (int k = 0; k < kHid / 16; ++k)
        w2f[k] = *reinterpret_cast<const bf16x4*>(N.wb + kW2 + h * kHid + k * 16 + q4);
    const bf16x4 w1 = *reinterpret_cast<const bf16x4*>(N.wb + kW1 + h * kIn);
    const float b1 = N.p[kB1 + h], b2 = N.p[kB2 + h];
    if (tid < kOut * kHid) w3s[tid] = from_bf16(N.wb[kW3 + tid]);
    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const uint32_t row0 = tile * kRowTile;
        __syncthreads();                 // the last tile's LDS is free
        if (tid < kRowTile) {
            const uint32_t b = row0 + (uint32_t)tid;
            const uint32_t src = b < nb ? (idx ? idx[b] : b) : 0u;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (b < nb) v = reinterpret_cast<const float4*>(X)[src];
            xs[tid] = v;
            if (BACK) {
                reinterpret_cast<float4*>(N.x)[b] = v;
                float2 t = make_float2(0.f, 0.f);
                if (b < nb) t = reinterpret_cast<const float2*>(Tt)[src];
                ts[tid] = t;
            }
        }
        __syncthreads();
        // layer 1: z1 = W1 x + b1, a1 = SiLU(z1) rounded to bf16
        float z1[4];
        bf16x4 a1;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float4 x = xs[q4 + j];
            float z = b1;
            z = fmaf(from_bf16((uint16_t)w1[0]), x.x, z);
            z = fmaf(from_bf16((uint16_t)w1[1]), x.y, z);
            z = fmaf(from_bf16((uint16_t)w1[2]), x.z, z);
            z = fmaf(from_bf16((uint16_t)w1[3]), x.w, z);
            z1[j] = z;
            a1[j] = (short)to_bf16(siluf_(z));
            ab[(q4 + j) * kLdA + h] = (uint16_t)a1[j];
        }
        if (BACK) *reinterpret_cast<bf16x4*>(N.a1t + (size_t)h * N.ld + row0 + q4) = a1;
        __syncthreads();
        // layer 2 on the matrix cores: z2(b, h) = sum_k a1(b, k) W2(h, k) + b2(h)
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < kHid / 16; ++k)
            acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                *reinterpret_cast<const bf16x4*>(ab + r * kLdA + k * 16 + q4), w2f[k], acc, 0, 0, 0);
        float z2[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            z2[j] = acc[j] + b2;
            const float a = siluf_(z2[j]);
            a2s[(q4 + j) * kLdF + h] = a;
            if (BACK) N.a2[(size_t)(row0 + q4 + j) * kHid + h] = a;
        }
        __syncthreads();
        // layer 3: y = sigmoid(W3 a2 + b3); dz3 = dL/dz3 for the mean-squared
        // error over the nb valid rows
        if (tid < kRowTile * kOut) {
            const uint32_t b = row0 + (uint32_t)(tid / kOut);
            const int o = tid % kOut;
            const f32x4* a = reinterpret_cast<const f32x4*>(a2s + (tid / kOut) * kLdF);
            const f32x4* w = reinterpret_cast<const f32x4*>(w3s + o * kHid);
            float z = N.p[kB3 + o];
            // (a serial chain: its LDS reads are issued 32 units ahead)
#pragma unroll
            for (int k0 = 0; k0 < kHid / 4; k0 += 8) {
                f32x4 av[8], wv[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    av[k] = a[k0 + k];
                    wv[k] = w[k0 + k];
                }
#pragma unroll
                for (int k = 0; k < 32; ++k) z = fmaf(wv[k / 4][k % 4], av[k / 4][k % 4], z);
            }
            const float y = sigmoidf_(z);
            if (y_out && b < nb) y_out[(size_t)b * kOut + o] = y;
            if (BACK) {
                const float t = o ? ts[tid / kOut].y : ts[tid / kOut].x;
                const float dy = b < nb ? 2.0f * (y - t) / (float)(nb * kOut) : 0.0f;
                const float d = dy * y * (1.0f - y);
                reinterpret_cast<float*>(dz3s)[tid] = d;
                N.dz3[(size_t)b * kOut + o] = d;
            }
        }
        if (!BACK) continue;
        __syncthreads();
        // back through layer 3: dz2 = (dz3 W3) * SiLU'(z2), kept in FP32 and bf16
        bf16x4 d2;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float2 d3 = dz3s[q4 + j];
            float da = fmaf(d3.x, w3s[h], 0.0f);
            da = fmaf(d3.y, w3s[kHid + h], da);
            const float dz = da * dsiluf_(z2[j]);
            d2[j] = (short)to_bf16(dz);
            db[(q4 + j) * kLdA + h] = (uint16_t)d2[j];
            N.dz2[(size_t)(row0 + q4 + j) * kHid + h] = dz;
        }
        *reinterpret_cast<bf16x4*>(N.dz2t + (size_t)h * N.ld + row0 + q4) = d2;
        __syncthreads();
        // da1(b, k) = sum_h dz2(b, h) W2(h, k) on the matrix cores, then
        // dz1 = da1 * SiLU'(z1)
        f32x4 da1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < kHid / 16; ++k)
            da1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                *reinterpret_cast<const bf16x4*>(db + r * kLdA + k * 16 + q4),
                *reinterpret_cast<const bf16x4*>(N.w2t + h * kHid + k * 16 + q4), da1, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) N.dz1[(size_t)(row0 + q4 + j) * kHid + h] = da1[j] * dsiluf_(z1[j]);
    }
}

// mean-squared error of each run of `chunk` rows of y against t (one
// workgroup per run, fixed order)
__global__ __launch_bounds__(256) void k_mlp_loss(const float* __restrict__ y, const float* __restrict__ t,
                                                  uint32_t n, uint32_t chunk, float* __restrict__ loss) {
    __shared__ float part[256];
    const uint32_t r0 = blockIdx.x * chunk, nb = min(chunk, n - r0);
    y += (size_t)r0 * kOut;
    t += (size_t)r0 * kOut;
    float s = 0.0f;
    for (uint32_t e = threadIdx.x; e < nb * kOut; e += 256) {
        const float d = y[e] - t[e];
        s = fmaf(d, d, s);
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[blockIdx.x] = part[0] / (float)(nb * kOut);
}

// What Adam holds for parameter k, read before the gradient is there.
struct AdamState { float p, m, v; };
template <bool ADAM>
__device__ __forceinline__ AdamState adam_state(const Net& N, uint32_t k) {
    return ADAM ? AdamState{N.p[k], N.m[k], N.v[k]} : AdamState{0.0f, 0.0f, 0.0f};
}
// The gradient of parameter k: stored, or taken by Adam (Kingma & Ba,
// bias-corrected) on the FP32 master parameters, then the bf16 copies;
// c1 = 1 - beta1^t, c2 = 1 - beta2^t.
template <bool ADAM>
__device__ __forceinline__ void apply_grad(const Net& N, uint32_t k, AdamState a, float g, float lr, float c1,
                                           float c2) {
    if (!ADAM) {
        N.g[k] = g;
        return;
    }
    const float m = 0.9f * a.m + 0.1f * g;
    const float v = 0.999f * a.v + 0.001f * g * g;
    N.m[k] = m;
    N.v[k] = v;
    const float p = a.p - lr * (m / c1) / (sqrtf(v / c2) + 1e-8f);
    N.p[k] = p;
    round_param(N, k, p);
}

// Every parameter gradient of a minibatch and the Adam update, one launch of
// 40 workgroups.  Workgroups 0 to 15: dW2(h, k) = sum_b dz2(b, h) a1(b, k) on
// the matrix cores, one wave per 16 x 16 tile, the operands read along b from
// the transposed copies.  The others: the reductions over 16 columns each of
// a2 (dW3), dz2 (db2, db3) and dz1 (dW1, db1) in FP32 in row order, one chain
// per parameter.  A chain is a serial sum over the rows; from global memory it
// waited for a load per few rows (72 us at 256 rows), so the workgroup first
// brings kGradRows rows of its columns into LDS with all loads in flight, and
// a thread sums up to three chains of one column from one LDS read.  Sixteen
// columns and one tile row to a workgroup, because one CU has only so many
// misses in flight: with all 128 columns in one workgroup the launch took 18
// us at 256 rows.
constexpr int kGradThreads = 256, kGradRows = 256, kGradCols = 16;
constexpr uint32_t kGradTiles = (kHid / 16) * (kHid / 16) / (kGradThreads / 64);       // workgroups of dW2
constexpr uint32_t kGradGrid = kGradTiles + 3 * (kHid / kGradCols);
template <bool ADAM>
__global__ __launch_bounds__(kGradThreads) void k_mlp_grads(Net N, uint32_t bp, float lr, float c1, float c2) {
    const int tid = (int)threadIdx.x;
    if (blockIdx.x < kGradTiles) {
        const int l = tid & 63, r = l & 15, q4 = (l >> 4) * 4;
        const uint32_t wave = blockIdx.x * (kGradThreads / 64) + (uint32_t)(tid >> 6);
        const uint32_t hm = (wave / 8) * 16, kn = (wave % 8) * 16;
        const uint16_t* a = N.dz2t + (size_t)(hm + r) * N.ld + q4;
        const uint16_t* b = N.a1t + (size_t)(kn + r) * N.ld + q4;
        const uint32_t k0 = kW2 + (hm + q4) * kHid + kn + r;
        AdamState st[4];
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (uint32_t b0 = 0; b0 < bp; b0 += 256) {
            bf16x4 av[16], bv[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const uint32_t at = min(b0 + 16u * k, bp - 16u);
                av[k] = *reinterpret_cast<const bf16x4*>(a + at);
                bv[k] = *reinterpret_cast<const bf16x4*>(b + at);
            }
            if (b0 == 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j) st[j] = adam_state<ADAM>(N, k0 + j * kHid);
            }
#pragma unroll
            for (int k = 0; k < 16; ++k)
                if (b0 + 16u * k < bp) acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av[k], bv[k], acc, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) apply_grad<ADAM>(N, k0 + j * kHid, st[j], acc[j], lr, c1, c2);
        return;
    }
    constexpr int kQuads = kGradRows * kGradCols / 4 / kGradThreads;                   // 16-byte loads per thread
    __shared__ f32x4 rows4[kGradRows * kGradCols / 4];
    __shared__ __attribute__((aligned(16))) float side[kGradRows * kIn];               // x (4 per row) or dz3 (2 per row)
    float* const rows = reinterpret_cast<float*>(rows4);
    const uint32_t part = (blockIdx.x - kGradTiles) / (kHid / kGradCols);              // 0: a2, 1: dz2, 2: dz1
    const uint32_t c0 = ((blockIdx.x - kGradTiles) % (kHid / kGradCols)) * kGradCols;
    const float* src = (part == 0 ? N.a2 : (part == 1 ? N.dz2 : N.dz1)) + c0;
    const float* ssrc = part == 2 ? N.x : N.dz3;
    const uint32_t sw = part == 2 ? kIn : kOut;
    // thread (col, half): chains of column col, times side columns 2 half and
    // 2 half + 1, and alone; db3 sums side columns with two more threads
    const uint32_t lc = (uint32_t)tid % kGradCols, half = (uint32_t)tid / kGradCols, col = c0 + lc;
    const bool weights = tid < (part == 0 ? kGradCols : (part == 1 ? 0 : 2 * kGradCols));
    const bool b3 = part == 1 && c0 == 0 && tid >= kGradCols && tid < kGradCols + kOut;
    const bool bias = (part != 0 && tid < kGradCols) || b3;
    const uint32_t p0 = part == 0 ? kW3 + col : kW1 + col * kIn + 2u * half, p1 = part == 0 ? p0 + kHid : p0 + 1u;
    const uint32_t pb = b3 ? kB3 + lc : (part == 1 ? kB2 : kB1) + col;
    const float* const uc = b3 ? side + lc : rows + lc;
    const uint32_t us = b3 ? sw : kGradCols;
    const float* const wc = side + (weights ? 2u * half : 0u);
    AdamState a0{}, a1{}, ab{};
    if (weights) {
        a0 = adam_state<ADAM>(N, p0);
        a1 = adam_state<ADAM>(N, p1);
    }
    if (bias) ab = adam_state<ADAM>(N, pb);
    float s0 = 0.0f, s1 = 0.0f, sb = 0.0f;
    for (uint32_t b0 = 0; b0 < bp; b0 += kGradRows) {
        const uint32_t nr = min((uint32_t)kGradRows, bp - b0);      // a multiple of 16
        f32x4 v[kQuads];
        float sv[kIn];
#pragma unroll
        for (int k = 0; k < kQuads; ++k) {
            const uint32_t e = (uint32_t)(tid + k * kGradThreads), b = min(e / (kGradCols / 4), nr - 1u);
            v[k] = *reinterpret_cast<const f32x4*>(src + (size_t)(b0 + b) * kHid + (e % (kGradCols / 4)) * 4);
        }
#pragma unroll
        for (int k = 0; k < kIn; ++k) sv[k] = ssrc[(size_t)b0 * sw + min((uint32_t)(tid + k * kGradThreads), nr * sw - 1u)];
        __syncthreads();                 // the rows before these have been summed
#pragma unroll
        for (int k = 0; k < kQuads; ++k) rows4[tid + k * kGradThreads] = v[k];
#pragma unroll
        for (int k = 0; k < kIn; ++k) side[tid + k * kGradThreads] = sv[k];
        __syncthreads();
        if (!weights && !bias) continue;
        // 16 rows are read while the 16 before them are summed
        float u[16];
        float2 w[16];
        auto read = [&](uint32_t b) {
#pragma unroll
            for (uint32_t k = 0; k < 16; ++k) {
                u[k] = uc[(b + k) * us];
                w[k] = *reinterpret_cast<const float2*>(wc + (b + k) * sw);
            }
        };
        read(0);
        for (uint32_t b = 0; b < nr; b += 16) {
            float cu[16];
            float2 cw[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                cu[k] = u[k];
                cw[k] = w[k];
            }
            read(b + 16 < nr ? b + 16 : b);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                s0 = fmaf(cw[k].x, cu[k], s0);
                s1 = fmaf(cw[k].y, cu[k], s1);
                sb += cu[k];
            }
        }
    }
    if (weights) {
        apply_grad<ADAM>(N, p0, a0, s0, lr, c1, c2);
        apply_grad<ADAM>(N, p1, a1, s1, lr, c1, c2);
    }
    if (bias) apply_grad<ADAM>(N, pb, ab, sb, lr, c1, c2);
}

}  // namespace

struct db_mlp {
    int device = 0;
    hipStream_t stream = nullptr;
    uint32_t bmax = 0;           // rows per minibatch, multiple of 16
    uint64_t adam_t = 0;
    Net N{};
    std::vector<void*> allocs;
    std::string err;
    float* dX = nullptr;         // training set on the device, and its outputs
    float* dT = nullptr;
    float* dY = nullptr;
    uint64_t cap_rows = 0;
    uint32_t* dIdx = nullptr;    // row orders: two slots
    uint32_t* hIdx = nullptr;    // the same in pinned memory
    uint64_t cap_idx = 0;        // entries of one slot
    hipEvent_t idx_done[2] = {nullptr, nullptr};   // the copy out of a pinned slot
    float* hRows = nullptr;      // pinned rows of a prediction: kPredictRows x 4 in, x 2 out
    uint64_t cap_pred = 0;
};

namespace {

db_status mfail(db_mlp* s, db_status st, const char* fmt, ...) {
    if (s) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        s->err = buf;
    }
    return st;
}

#define MCHK(s, call)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (call);                                                              \
        if (e_ != hipSuccess) return mfail((s), DB_EDEVICE, "%s: %s", #call, hipGetErrorString(e_)); \
    } while (0)

template <class T>
db_status malloc_n(db_mlp* s, T*& p, size_t n) {
    void* q = nullptr;
    if (hipMalloc(&q, std::max<size_t>(n, 1) * sizeof(T)) != hipSuccess)
        return mfail(s, DB_ENOMEM, "device allocation of %zu bytes failed", n * sizeof(T));
    s->allocs.push_back(q);
    p = static_cast<T*>(q);
    return DB_OK;
}

#define MALLOC(s, p, n)                               \
    do {                                              \
        db_status st_ = malloc_n((s), (p), (n));      \
        if (st_ != DB_OK) return st_;                 \
    } while (0)

inline unsigned blocks(uint64_t n, unsigned bs) { return (unsigned)((n + bs - 1) / bs); }

// Minibatch orders on their way to the device, and rows of a prediction, go
// through pinned buffers (allocated on first use: 2 x 1 MiB, or 2 x 4 B a row
// up to 2 x 16 MiB, and at most 1.5 MiB).  Predictions of more than
// kPredictRows rows take turns through the buffer at the same rate: 65 536 rows
// 109 us, 300 000 509 us (1.66 and 1.70 us per 1000).
constexpr uint64_t kIdxSlot = 262144, kIdxPinnedMax = 16 * kIdxSlot, kPredictRows = 65536;
// Workgroups of the forward pass over many rows: two per CU; each keeps its
// weights over its tiles.
constexpr uint32_t kRowGrid = 512;

void launch_rows(db_mlp* s, const float* x, uint64_t n, float* y) {
    const uint32_t tiles = (uint32_t)((n + kRowTile - 1) / kRowTile);
    hipLaunchKernelGGL(k_mlp_rows<false>, dim3(std::min(tiles, kRowGrid)), dim3(kRowThreads), 0, s->stream, s->N, x,
                       (const float*)nullptr, (const uint32_t*)nullptr, (uint32_t)n, tiles, y);
}

// Forward and backward over the nb rows idx names (the first nb when null),
// then the gradients: into N.g (lr <= 0) or into the parameters.
void launch_minibatch(db_mlp* s, const uint32_t* idx, uint32_t nb, float* y, float lr, float c1, float c2) {
    const uint32_t tiles = (nb + kRowTile - 1) / kRowTile, bp = tiles * kRowTile;
    hipLaunchKernelGGL(k_mlp_rows<true>, dim3(tiles), dim3(kRowThreads), 0, s->stream, s->N, (const float*)s->dX,
                       (const float*)s->dT, idx, nb, tiles, y);
    if (lr > 0.0f)
        hipLaunchKernelGGL(k_mlp_grads<true>, dim3(kGradGrid), dim3(kGradThreads), 0, s->stream, s->N, bp, lr, c1, c2);
    else
        hipLaunchKernelGGL(k_mlp_grads<false>, dim3(kGradGrid), dim3(kGradThreads), 0, s->stream, s->N, bp, 0.0f, 1.0f,
                           1.0f);
}

db_status upload_rows(db_mlp* s, const float* x, const float* t, uint64_t n) {
    if (n > s->cap_rows) {
        for (void* q : {(void*)s->dX, (void*)s->dT, (void*)s->dY}) {
            auto it = std::find(s->allocs.begin(), s->allocs.end(), q);
            if (it != s->allocs.end()) {
                (void)hipFree(q);
                s->allocs.erase(it);
            }
        }
        s->dX = nullptr;
        s->dT = nullptr;
        s->dY = nullptr;
        s->cap_rows = 0;
        MALLOC(s, s->dX, n * kIn);
        MALLOC(s, s->dT, n * kOut);
        MALLOC(s, s->dY, n * kOut);
        s->cap_rows = n;
    }
    MCHK(s, hipMemcpyAsync(s->dX, x, n * kIn * sizeof(float), hipMemcpyHostToDevice, s->stream));
    MCHK(s, hipMemcpyAsync(s->dT, t, n * kOut * sizeof(float), hipMemcpyHostToDevice, s->stream));
    return DB_OK;
}

// (bitwise on the exponent, without an early exit, so that the loop is vectorised)
bool finite_rows(const float* a, uint64_t count) {
    uint32_t bad = 0;
    for (uint64_t k = 0; k < count; ++k) {
        uint32_t u;
        std::memcpy(&u, a + k, 4);
        bad |= (u & 0x7F800000u) == 0x7F800000u ? 1u : 0u;
    }
    return bad == 0u;
}

// The device and pinned buffers of the minibatch orders.  Above kIdxPinnedMax
// rows (or where pinned memory is short) an order goes straight from the
// host's own array, one epoch at a time (hIdx stays null).
db_status index_buffers(db_mlp* s, uint64_t n) {
    const bool pin = n <= kIdxPinnedMax;
    const uint64_t slot = pin ? std::max<uint64_t>(kIdxSlot, n) : n;
    if (s->dIdx && slot <= s->cap_idx && (s->hIdx || !pin)) return DB_OK;
    MCHK(s, hipStreamSynchronize(s->stream));
    if (s->hIdx) (void)hipHostFree(s->hIdx);
    s->hIdx = nullptr;
    s->cap_idx = 0;
    auto it = std::find(s->allocs.begin(), s->allocs.end(), (void*)s->dIdx);
    if (s->dIdx && it != s->allocs.end()) {
        (void)hipFree(s->dIdx);
        s->allocs.erase(it);
    }
    s->dIdx = nullptr;
    for (auto& e : s->idx_done)
        if (!e) MCHK(s, hipEventCreateWithFlags(&e, hipEventDisableTiming));
    MALLOC(s, s->dIdx, (pin ? 2 : 1) * slot);
    s->cap_idx = slot;
    void* h = nullptr;
    if (pin && hipHostMalloc(&h, 2 * slot * sizeof(uint32_t), hipHostMallocDefault) == hipSuccess) s->hIdx = (uint32_t*)h;
    else if (pin) (void)hipGetLastError();
    return DB_OK;
}

}  // namespace

extern "C" {

db_status db_mlp_create(uint32_t batch_max, int device, db_mlp** out) {
    if (!out) return DB_EINVAL;
    *out = nullptr;
    if (batch_max < 1 || batch_max > 4096) return DB_EINVAL;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) {
        (void)hipGetLastError();
        return DB_EDEVICE;
    }
    db_mlp* s = new db_mlp();
    s->device = device;
    s->bmax = (batch_max + 15u) & ~15u;
    auto bad = [&](db_status st) {
        db_mlp_destroy(s);
        return st;
    };
    if (hipSetDevice(device) != hipSuccess || hipStreamCreateWithFlags(&s->stream, hipStreamNonBlocking) != hipSuccess)
        return bad(DB_EDEVICE);
    Net& N = s->N;
    const size_t b = s->bmax;
    db_status st = DB_OK;
    auto A = [&](auto*& p, size_t n) { if (st == DB_OK) st = malloc_n(s, p, n); };
    A(N.p, kNP); A(N.m, kNP); A(N.v, kNP); A(N.g, kNP); A(N.wb, kNP); A(N.w2t, kHid * kHid);
    A(N.x, b * kIn); A(N.a2, b * kHid); A(N.dz3, b * kOut); A(N.dz2, b * kHid); A(N.dz1, b * kHid);
    A(N.a1t, b * kHid); A(N.dz2t, b * kHid);
    N.ld = (uint32_t)b;
    if (st != DB_OK) return bad(st);
    for (void* q : {(void*)N.p, (void*)N.m, (void*)N.v, (void*)N.g})
        if (hipMemsetAsync(q, 0, kNP * sizeof(float), s->stream) != hipSuccess) return bad(DB_EDEVICE);
    if (hipMemsetAsync(N.wb, 0, kNP * sizeof(uint16_t), s->stream) != hipSuccess ||
        hipMemsetAsync(N.w2t, 0, kHid * kHid * sizeof(uint16_t), s->stream) != hipSuccess ||
        hipStreamSynchronize(s->stream) != hipSuccess)
        return bad(DB_EDEVICE);
    *out = s;
    return DB_OK;
}

void db_mlp_destroy(db_mlp* s) {
    if (!s) return;
    (void)hipSetDevice(s->device);
    if (s->stream) (void)hipStreamSynchronize(s->stream);
    for (void* q : s->allocs) (void)hipFree(q);
    if (s->hIdx) (void)hipHostFree(s->hIdx);
    if (s->hRows) (void)hipHostFree(s->hRows);
    for (hipEvent_t e : s->idx_done)
        if (e) (void)hipEventDestroy(e);
    if (s->stream) (void)hipStreamDestroy(s->stream);
    delete s;
}

db_status db_mlp_set_params(db_mlp* s, const float* params, uint64_t count) {
    if (!s || !params) return DB_EINVAL;
    if (count != kNP) return mfail(s, DB_EINVAL, "expected %u parameters, got %llu", kNP, (unsigned long long)count);
    MCHK(s, hipSetDevice(s->device));
    MCHK(s, hipMemcpyAsync(s->N.p, params, kNP * sizeof(float), hipMemcpyHostToDevice, s->stream));
    MCHK(s, hipMemsetAsync(s->N.m, 0, kNP * sizeof(float), s->stream));
    MCHK(s, hipMemsetAsync(s->N.v, 0, kNP * sizeof(float), s->stream));
    hipLaunchKernelGGL(k_mlp_round, dim3(blocks(kNP, 256)), dim3(256), 0, s->stream, s->N);
    MCHK(s, hipGetLastError());
    MCHK(s, hipStreamSynchronize(s->stream));
    s->adam_t = 0;
    return DB_OK;
}

db_status db_mlp_get_params(db_mlp* s, float* params, uint64_t count) {
    if (!s || !params) return DB_EINVAL;
    if (count != kNP) return mfail(s, DB_EINVAL, "expected %u parameters, got %llu", kNP, (unsigned long long)count);
    MCHK(s, hipSetDevice(s->device));
    MCHK(s, hipMemcpyAsync(params, s->N.p, kNP * sizeof(float), hipMemcpyDeviceToHost, s->stream));
    MCHK(s, hipStreamSynchronize(s->stream));
    return DB_OK;
}

db_status db_mlp_predict(db_mlp* s, const float* x, uint64_t n, float* y) {
    if (!s || (!x && n) || (!y && n)) return DB_EINVAL;
    if (n == 0) return DB_OK;
    if (!finite_rows(x, n * kIn)) return mfail(s, DB_EINVAL, "non-finite input");
    MCHK(s, hipSetDevice(s->device));
    // rows go through pinned memory, which the kernel reads and writes itself
    // (a copy, a launch per layer and a wait for every batch_max rows took
    // 2.5 ms for 65 536 rows)
    const uint64_t cap = std::min<uint64_t>(n, kPredictRows);
    if (cap > s->cap_pred) {
        if (s->hRows) (void)hipHostFree(s->hRows);
        s->hRows = nullptr;
        s->cap_pred = 0;
        const uint64_t want = std::min<uint64_t>(kPredictRows, std::max<uint64_t>(cap, 1024));
        void* h = nullptr;
        if (hipHostMalloc(&h, want * (kIn + kOut) * sizeof(float), hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return mfail(s, DB_ENOMEM, "pinned host allocation failed");
        }
        s->hRows = (float*)h;
        s->cap_pred = want;
    }
    float* const hx = s->hRows;
    float* const hy = s->hRows + s->cap_pred * kIn;
    for (uint64_t r0 = 0; r0 < n; r0 += s->cap_pred) {
        const uint64_t nb = std::min<uint64_t>(s->cap_pred, n - r0);
        std::memcpy(hx, x + r0 * kIn, nb * kIn * sizeof(float));
        launch_rows(s, hx, nb, hy);
        MCHK(s, hipGetLastError());
        MCHK(s, hipStreamSynchronize(s->stream));
        std::memcpy(y + r0 * kOut, hy, nb * kOut * sizeof(float));
    }
    return DB_OK;
}

db_status db_mlp_loss_grad(db_mlp* s, const float* x, const float* t, uint32_t n, float* loss, float* grad) {
    if (!s || !x || !t || !loss || !grad) return DB_EINVAL;
    if (n < 1 || n > s->bmax) return mfail(s, DB_EINVAL, "n must be in [1, %u]", s->bmax);
    if (!finite_rows(x, (uint64_t)n * kIn) || !finite_rows(t, (uint64_t)n * kOut))
        return mfail(s, DB_EINVAL, "non-finite input or target");
    MCHK(s, hipSetDevice(s->device));
    db_status st = upload_rows(s, x, t, n);
    if (st != DB_OK) return st;
    launch_minibatch(s, nullptr, n, s->dY, 0.0f, 1.0f, 1.0f);
    float* const dl = s->N.dz3;                  // the backward pass is done with dz3
    hipLaunchKernelGGL(k_mlp_loss, dim3(1), dim3(256), 0, s->stream, (const float*)s->dY, (const float*)s->dT, n, n, dl);
    MCHK(s, hipGetLastError());
    MCHK(s, hipMemcpyAsync(grad, s->N.g, kNP * sizeof(float), hipMemcpyDeviceToHost, s->stream));
    MCHK(s, hipMemcpyAsync(loss, dl, sizeof(float), hipMemcpyDeviceToHost, s->stream));
    MCHK(s, hipStreamSynchronize(s->stream));
    return DB_OK;
}

db_status db_mlp_train(db_mlp* s, const float* x, const float* t, uint64_t n, uint32_t batch, uint32_t epochs,
                       float lr, uint64_t seed, float* final_loss) {
    if (!s || !x || !t) return DB_EINVAL;
    if (n < 1 || n > 0xFFFFFFFFull) return mfail(s, DB_EINVAL, "n out of range");
    if (batch < 1 || batch > s->bmax) return mfail(s, DB_EINVAL, "batch must be in [1, %u]", s->bmax);
    if (!(lr > 0.0f) || !std::isfinite(lr)) return mfail(s, DB_EINVAL, "learning rate must be positive");
    if (!finite_rows(x, n * kIn) || !finite_rows(t, n * kOut)) return mfail(s, DB_EINVAL, "non-finite input or target");
    MCHK(s, hipSetDevice(s->device));
    db_status st = upload_rows(s, x, t, n);
    if (st != DB_OK) return st;
    st = index_buffers(s, n);
    if (st != DB_OK) return st;
    std::mt19937_64 gen(seed);
    std::vector<uint32_t> perm(n);
    std::iota(perm.begin(), perm.end(), 0u);
    // epochs are drawn in groups that fill a slot, while the device works on
    // the group before
    const bool pinned = s->hIdx != nullptr;
    const uint32_t group = pinned ? (uint32_t)std::max<uint64_t>(1, s->cap_idx / n) : 1u;
    for (uint32_t e0 = 0, turn = 0; e0 < epochs; e0 += group, ++turn) {
        const uint32_t ne = std::min(group, epochs - e0);
        const uint64_t at = pinned ? (turn & 1u) * s->cap_idx : 0;
        uint32_t* const d = s->dIdx + at;
        // the last copy out of this slot (or out of `perm`) must be done
        if (pinned && turn >= 2) MCHK(s, hipEventSynchronize(s->idx_done[turn & 1u]));
        else if (!pinned && turn) MCHK(s, hipStreamSynchronize(s->stream));
        for (uint32_t e = 0; e < ne; ++e) {
            for (uint64_t k = n - 1; k > 0; --k) std::swap(perm[k], perm[gen() % (k + 1)]);
            if (pinned) std::memcpy(s->hIdx + at + (size_t)e * n, perm.data(), n * sizeof(uint32_t));
        }
        const uint32_t* const h = pinned ? s->hIdx + at : perm.data();
        MCHK(s, hipMemcpyAsync(d, h, (size_t)ne * n * sizeof(uint32_t), hipMemcpyHostToDevice, s->stream));
        MCHK(s, hipEventRecord(s->idx_done[turn & 1u], s->stream));
        for (uint32_t e = 0; e < ne; ++e)
            for (uint64_t r0 = 0; r0 < n; r0 += batch) {
                ++s->adam_t;
                const float c1 = (float)(1.0 - std::pow(0.9, (double)s->adam_t));
                const float c2 = (float)(1.0 - std::pow(0.999, (double)s->adam_t));
                launch_minibatch(s, d + (size_t)e * n + r0, (uint32_t)std::min<uint64_t>(batch, n - r0), nullptr, lr, c1,
                                 c2);
            }
        MCHK(s, hipGetLastError());
    }
    if (!final_loss) {
        MCHK(s, hipStreamSynchronize(s->stream));
        return DB_OK;
    }
    // mean-squared error over all rows, from the errors of batch_max rows at a time
    const uint32_t chunks = (uint32_t)((n + s->bmax - 1) / s->bmax);
    launch_rows(s, s->dX, n, s->dY);
    // (one error per run of bmax rows, and x has 4 words per row)
    hipLaunchKernelGGL(k_mlp_loss, dim3(chunks), dim3(256), 0, s->stream, (const float*)s->dY, (const float*)s->dT,
                       (uint32_t)n, s->bmax, s->dX);
    std::vector<float> l(chunks);
    MCHK(s, hipGetLastError());
    MCHK(s, hipMemcpyAsync(l.data(), s->dX, chunks * sizeof(float), hipMemcpyDeviceToHost, s->stream));
    MCHK(s, hipStreamSynchronize(s->stream));
    double acc = 0.0;
    for (uint32_t k = 0; k < chunks; ++k)
        acc += (double)l[k] * (double)std::min<uint64_t>(s->bmax, n - (uint64_t)k * s->bmax);
    *final_loss = (float)(acc / (double)n);
    return DB_OK;
}

const char* db_mlp_last_error(const db_mlp* s) { return s ? s->err.c_str() : "null handle"; }

}  // extern "C"
