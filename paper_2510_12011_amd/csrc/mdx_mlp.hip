// Per-node MLP of the learned warm start: 4 -> 64 -> 64 -> 64 -> 1, ReLU,
// BF16 weights and activations, FP32 accumulation, on the BF16 MFMA of
// gfx950.  Forward (inference), gradient of the mean-squared error
// (training) and Adam.
//
// Parameter vector (FP32 master copy, 8,705 values):
//   W1[64][4] b1[64] W2[64][64] b2[64] W3[64][64] b3[64] W4[64] b4
//
// Arithmetic: layer 1 in FP32 VALU with BF16-rounded W1 on FP32 features;
// h1 = bf16(relu(z1)); layers 2 and 3 on MFMA (BF16 operands, FP32
// accumulators) plus FP32 bias; h2 = bf16(relu(z2)); h3 = relu(z3) in FP32;
// y = sum bf16(W4) h3 + b4 in FP32.
//
// Inference gives a wavefront tiles of 32 nodes.  Hidden layers are computed
// as transposed products Z^T = W H^T (M = output unit, N = node, K = input
// unit).  With the 32x32 MFMAs the accumulator element held in register v of
// lane l is Z^T[8(v/4) + 4(l/32) + v%4][l%32], which the next layer's B operand
// takes from registers with no data exchange (the weights' columns are read in
// that order).
#include "mdx_device.h"
#include "mdx_internal.h"

#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

namespace mdx {

namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int NH = 64;
constexpr int OFF_W1 = 0, OFF_B1 = 256, OFF_W2 = 320, OFF_B2 = 4416, OFF_W3 = 4480,
              OFF_B3 = 8576, OFF_W4 = 8640, OFF_B4 = 8704;
constexpr int NPARAM = 8705;
constexpr int WSTRIDE = 68;   // LDS row stride (bf16) of W2/W3: 8-byte aligned, fewer conflicts

__device__ __forceinline__ unsigned short f2bf(float f)
{
    unsigned u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);   // round to nearest even (finite inputs)
    return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float((unsigned)h << 16); }
__device__ __forceinline__ float round_bf(float f) { return bf2f(f2bf(f)); }

// ---------------------------------------------------------------------------
// Inference (the warm start of every time step), every layer on
// v_mfma_f32_32x32x16_bf16:
//   layer 1: the FP32 features enter as a BF16 pair hi + lo (x = hi + lo to
//            about 2^-17 relative): B rows 0..3 hi, 4..7 lo, 8..15 zero and
//            A columns W1, W1, 0, so one MFMA gives BF16(W1) x in FP32;
//   layers 2, 3: K-step s of a 64-unit layer reads, in lane half h, the
//            accumulator registers 8 (s % 2) .. + 7 of the previous layer's
//            output tile s / 2 -- units 16 s + 8 (j / 4) + 4 h + j % 4 for
//            j = 0..7 -- so the weight fragment takes those columns (two
//            8-byte LDS reads) and no data moves between lanes;
//   biases:  FP32, loaded as the accumulators' initial values;
//   BF16 rounding of the activations by the hardware conversion
//   (round to nearest even, as f2bf).
// No pre-activations are kept, so several wavefronts share a SIMD.
// ---------------------------------------------------------------------------
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8n __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x16 mfma16(s16x8 a, s16x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8n, a),
                                                    __builtin_bit_cast(bf16x8n, b), c, 0, 0, 0);
}

__device__ __forceinline__ s16x8 cat8(bf16x4 lo, bf16x4 hi)
{
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// A fragment of a hidden layer's W (64 x 64, LDS row stride WSTRIDE) for
// output tile ot and K-step s: row 32 ot + l % 32, the columns listed above
__device__ __forceinline__ s16x8 frag_w16(const unsigned short *w, int ot, int s, int lane)
{
    const unsigned short *row = w + (32 * ot + (lane & 31)) * WSTRIDE + 16 * s + 4 * (lane >> 5);
    return cat8(*reinterpret_cast<const bf16x4 *>(row), *reinterpret_cast<const bf16x4 *>(row + 8));
}
typedef __bf16 bf16x2n __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned pack_bf16(float a, float b)
{
    f32x2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2n));
}
__device__ __forceinline__ bf16x4 pack_bf16x4(float a, float b, float c, float d)
{
    u32x2 u = {pack_bf16(a, b), pack_bf16(c, d)};
    return __builtin_bit_cast(bf16x4, u);
}
// bf16(relu(a)), ... for four values: ReLU after the rounding, on the packed
// pairs as signed 16-bit integers (a BF16 value is negative exactly when its
// bit pattern is, and rounding to nearest keeps the sign, so max(bits, 0)
// maps negatives, -0 included, to +0 and keeps the rest)
typedef short s16x2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned relu_bf16x2(float a, float b)
{
    const s16x2v zero = {0, 0};
    const s16x2v v = __builtin_bit_cast(s16x2v, pack_bf16(a, b));
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(v, zero));
}
__device__ __forceinline__ bf16x4 relu_pack_bf16x4(float a, float b, float c, float d)
{
    u32x2 u = {relu_bf16x2(a, b), relu_bf16x2(c, d)};
    return __builtin_bit_cast(bf16x4, u);
}

// ReLU in FP32 as a signed-integer max on the bit pattern: values with the
// sign bit set (negatives, -0) become +0, the rest are kept.  fmaxf would
// add a canonicalising max per value.
__device__ __forceinline__ float relu_bits(float x) { return __int_as_float(max(__float_as_int(x), 0)); }

struct alignas(16) InferLds {
    float b1[NH], b2[NH], b3[NH], w4[NH];   // FP32 biases, BF16-rounded w4
    unsigned short w1[NH * 16];             // BF16 [W1 W1 0]: columns 0..3, 4..7, 8..15
    unsigned short w2[NH * WSTRIDE];
    unsigned short w3[NH * WSTRIDE];
    float b4;
};

// bias (or w4) values of the units held by this lane in output tile ot, in
// accumulator order: v = 4 g + j -> unit 32 ot + 8 g + 4 half + j
__device__ __forceinline__ f32x16 unit_frag(const float *v, int ot, int half)
{
    f32x16 r;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const float4 q = *reinterpret_cast<const float4 *>(v + 32 * ot + 8 * g + 4 * half);
        r[4 * g + 0] = q.x;
        r[4 * g + 1] = q.y;
        r[4 * g + 2] = q.z;
        r[4 * g + 3] = q.w;
    }
    return r;
}

// The network's input per node: stored standardised features (X), or the
// features formed from the state as the feature pass forms them (same
// expressions, so the same bits): V, V - V_prev, s / Cm, the neighbour
// aggregate, standardised.
// fetch() issues a node's loads (zeros past n, or for lanes that hold no
// node), form() turns them into the network's input, so that the loads of
// the next nodes can be in flight while the current ones are computed.
template <bool STATE>
struct FeatRaw;
template <>
struct FeatRaw<false> {
    float4 x;
};
template <>
struct FeatRaw<true> {
    double v, vp, s;
    float k;
};

struct FeatIn {
    const float4 *X;
    const double *V, *Vprev, *src;
    const float *kvp;
    double inv_cm;   // 1 / Cm
    MlpNorm nm;
    template <bool STATE>
    __device__ __forceinline__ FeatRaw<STATE> fetch(int64_t i, bool ok) const
    {
        if constexpr (STATE) {
            FeatRaw<true> r{0.0, 0.0, 0.0, 0.0f};
            if (ok) r = {V[i], Vprev[i], src[i], kvp[i]};
            return r;
        } else {
            FeatRaw<false> r{make_float4(0.f, 0.f, 0.f, 0.f)};
            if (ok) r.x = X[i];
            return r;
        }
    }
    template <bool STATE>
    __device__ __forceinline__ float4 form(const FeatRaw<STATE> &r, bool ok) const
    {
        if (!ok) return make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (STATE) {
            const float fx = (float)r.v, fy = (float)(r.v - r.vp), fz = (float)(r.s * inv_cm);
            return make_float4((fx - nm.mean[0]) * nm.inv_std[0],
                               (fy - nm.mean[1]) * nm.inv_std[1],
                               (fz - nm.mean[2]) * nm.inv_std[2],
                               (r.k - nm.mean[3]) * nm.inv_std[3]);
        } else {
            return r.x;
        }
    }
};

template <bool STATE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_mlp_forward(const float *__restrict__ P, int64_t n,
                                                     FeatIn in, float *__restrict__ y)
{
    __shared__ InferLds w;
    {
        // the weights into LDS, every load issued before the first
        // conversion: a fixed stride of 256 threads (the launch's size),
        // fully unrolled (a loop over blockDim.x waited on each load in turn)
        constexpr int NT = 256, R = NH * NH / NT;
        const int t = threadIdx.x;
        float a2[R], a3[R], a1[4];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            a2[j] = P[OFF_W2 + t + NT * j];
            a3[j] = P[OFF_W3 + t + NT * j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = t + NT * j, o = i / 16, k = i % 16;
            a1[j] = k < 8 ? P[OFF_W1 + 4 * o + (k & 3)] : 0.0f;
        }
        float bb[4] = {0.0f, 0.0f, 0.0f, 0.0f}, b4 = 0.0f;
        if (t < NH) {
            bb[0] = P[OFF_B1 + t];
            bb[1] = P[OFF_B2 + t];
            bb[2] = P[OFF_B3 + t];
            bb[3] = P[OFF_W4 + t];
        }
        if (t == 0) b4 = P[OFF_B4];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int i = t + NT * j, o = i / NH, k = i % NH;
            w.w2[o * WSTRIDE + k] = f2bf(a2[j]);
            w.w3[o * WSTRIDE + k] = f2bf(a3[j]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) w.w1[t + NT * j] = f2bf(a1[j]);
        if (t < NH) {
            w.b1[t] = bb[0];
            w.b2[t] = bb[1];
            w.b3[t] = bb[2];
            w.w4[t] = round_bf(bb[3]);
        }
        if (t == 0) w.b4 = b4;
    }
    __syncthreads();

    const int lane = threadIdx.x & 63, half = lane >> 5;
    // two 32-node tiles per pass share every weight and bias fragment read
    // from LDS and give each wavefront two independent MFMA chains to
    // interleave (one tile per pass took 44-49 us on 1.26M nodes, two 26-28)
    const int64_t n_pairs = ((n + 31) / 32 + 1) / 2;
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / 64);
    const int64_t pr0 = (int64_t)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
    FeatRaw<STATE> raw[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int64_t nd = (2 * pr0 + b) * 32 + (lane & 31);
        raw[b] = in.fetch<STATE>(nd, pr0 < n_pairs && half == 0 && nd < n);
    }
    for (int64_t pr = pr0; pr < n_pairs; pr += waves) {
        // weights are re-read from LDS for every pair: held in registers
        // across pairs they would take ~200 VGPRs and leave one wavefront
        // per SIMD to hide the latency of the layer chain
        asm volatile("" ::: "memory");
        int64_t node[2];
        s16x8 xb[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            node[b] = (2 * pr + b) * 32 + (lane & 31);
            const float4 x = in.form<STATE>(raw[b], half == 0 && node[b] < n);
            const bf16x4 xh = pack_bf16x4(x.x, x.y, x.z, x.w);
            const float4 xr = make_float4(x.x - bf2f((unsigned short)xh[0]),
                                          x.y - bf2f((unsigned short)xh[1]),
                                          x.z - bf2f((unsigned short)xh[2]),
                                          x.w - bf2f((unsigned short)xh[3]));
            xb[b] = cat8(xh, pack_bf16x4(xr.x, xr.y, xr.z, xr.w));
        }
        // the next pair's loads, issued once this pair's inputs are formed
        // (loads retire in order) and in flight during its layers
        const int64_t pn = pr + waves;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int64_t nd = (2 * pn + b) * 32 + (lane & 31);
            raw[b] = in.fetch<STATE>(nd, pn < n_pairs && half == 0 && nd < n);
        }
        // layer 1
        bf16x4 h1[2][8];
#pragma unroll
        for (int ot = 0; ot < 2; ++ot) {
            const s16x8 a =
                *reinterpret_cast<const s16x8 *>(w.w1 + (32 * ot + (lane & 31)) * 16 + 8 * half);
            const f32x16 bias = unit_frag(w.b1, ot, half);
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const f32x16 acc = mfma16(a, xb[b], bias);
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    h1[b][4 * ot + g] = relu_pack_bf16x4(acc[4 * g], acc[4 * g + 1],
                                                         acc[4 * g + 2], acc[4 * g + 3]);
            }
        }
        // layer 2
        bf16x4 h2[2][8];
#pragma unroll
        for (int ot = 0; ot < 2; ++ot) {
            f32x16 acc[2];
            acc[0] = acc[1] = unit_frag(w.b2, ot, half);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const s16x8 wf = frag_w16(w.w2, ot, ks, lane);
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[b] = mfma16(wf, cat8(h1[b][2 * ks], h1[b][2 * ks + 1]), acc[b]);
            }
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    h2[b][4 * ot + g] = relu_pack_bf16x4(acc[b][4 * g], acc[b][4 * g + 1],
                                                         acc[b][4 * g + 2], acc[b][4 * g + 3]);
        }
        // layer 3 and the output unit
        float sum[2] = {0.0f, 0.0f};
#pragma unroll
        for (int ot = 0; ot < 2; ++ot) {
            f32x16 acc[2];
            acc[0] = acc[1] = unit_frag(w.b3, ot, half);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const s16x8 wf = frag_w16(w.w3, ot, ks, lane);
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[b] = mfma16(wf, cat8(h2[b][2 * ks], h2[b][2 * ks + 1]), acc[b]);
            }
            const f32x16 w4 = unit_frag(w.w4, ot, half);
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) sum[b] += w4[v] * relu_bits(acc[b][v]);
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const float t = sum[b] + __shfl_xor(sum[b], 32, 64);
            if (half == 0 && node[b] < n) y[node[b]] = t + w.b4;
        }
    }
}

// ---------------------------------------------------------------------------
// Training: gradient of L = (1/n) sum_i (y_i - t_i)^2.  Each workgroup
// accumulates its samples' gradient in registers and writes it to its own
// slice of `partials` (NPARAM values + its loss sum), reduced afterwards in a
// fixed order by k_mlp_reduce -- no atomics, deterministic.
//
// At the training batch of 8,192 samples a workgroup has one tile of 32 nodes,
// so what counts is the length of the chain: weights in, three layers forward,
// two back, four gradient products.  Four wavefronts share the tile, each
// computing 16 of the 64 units of every layer (16x16x32 MFMA: lane l holds
// row or column l % 16 and k = 8 (l / 16) .. + 7 of the operands, and rows
// 4 (l / 16) .. + 3 of column l % 16 of the result).  A layer's output goes to
// LDS twice: node by node for the next layer's B operand, and unit by unit for
// the weight gradients dW = dZ H^T, products over the tile's nodes, which run
// under the latency of the next layer back.  Bias gradients are the same
// products with a column of ones.  On 8,192 samples with one wavefront a tile,
// 32x32x8 MFMAs and partials read, added to and written per product it was
// 98 us; 12 us now.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int TW = 72;   // LDS row strides (bf16), 16-byte rows: a weight's or a node's 64 units,
constexpr int TN = 40;   // a unit's 32 nodes

struct alignas(16) TrainLds {
    unsigned short w2[NH * TW], w3[NH * TW];     // [output][input]
    unsigned short w2t[NH * TW], w3t[NH * TW];   // [input][output]
    unsigned short by_node[2][32 * TW];          // the layer in hand [node][unit]
    unsigned short h1[NH * TN], h2[NH * TN], h3[NH * TN];   // activations [unit][node]
    unsigned short d1[NH * TN], d2[NH * TN], d3[NH * TN];   // dL/dz [unit][node]
    unsigned short x[4 * TN], dy[TN];
    float w1[NH][4];                             // BF16-rounded
    float b1[NH], b2[NH], b3[NH], w4[NH];        // w4 BF16-rounded
    float ysum[4][32];                           // a wavefront's part of y
    float b4;
};
static_assert(2 * sizeof(TrainLds) <= 160 * 1024, "two workgroups a compute unit");

__device__ __forceinline__ f32x4 mfma32(s16x8 a, s16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8n, a),
                                                   __builtin_bit_cast(bf16x8n, b), c, 0, 0, 0);
}
__device__ __forceinline__ s16x8 frag(const unsigned short *s, int stride, int row, int k)
{
    return *reinterpret_cast<const s16x8 *>(s + row * stride + k);
}

__global__ __launch_bounds__(256, 2) void k_mlp_grad(const float *__restrict__ P, int64_t n,
                                                     const float *__restrict__ X,
                                                     const float *__restrict__ Tgt,
                                                     int tiles_per_group,
                                                     float *__restrict__ partials)
{
    __shared__ TrainLds L;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r = lane & 15, q = lane >> 4;
    const int64_t t0 = (int64_t)blockIdx.x * tiles_per_group;
    const int64_t t1 = min(t0 + tiles_per_group, (n + 31) / 32);

    // the lane's two nodes of a tile
    float4 x[2];
    float tg[2];
    bool valid[2];
    auto fetch = [&](int64_t tile) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int64_t node = tile * 32 + 16 * b + r;
            valid[b] = node < n;
            x[b] = make_float4(0.f, 0.f, 0.f, 0.f);
            tg[b] = 0.0f;
            if (valid[b]) {
                x[b] = reinterpret_cast<const float4 *>(X)[node];
                tg[b] = Tgt[node];
            }
        }
    };
    fetch(t0);
    {   // weights into LDS, every load issued before the first conversion
        constexpr int R = NH * NH / 256;
        float a2[R], a3[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            a2[j] = P[OFF_W2 + tid + 256 * j];
            a3[j] = P[OFF_W3 + tid + 256 * j];
        }
        const float a1 = P[OFF_W1 + tid];
        float bb[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (tid < NH) {
            bb[0] = P[OFF_B1 + tid];
            bb[1] = P[OFF_B2 + tid];
            bb[2] = P[OFF_B3 + tid];
            bb[3] = P[OFF_W4 + tid];
        }
        if (tid == 0) L.b4 = P[OFF_B4];
        const int k = tid & 63;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int o = wave + 4 * j;
            const unsigned short c2 = f2bf(a2[j]), c3 = f2bf(a3[j]);
            L.w2[o * TW + k] = c2;
            L.w3[o * TW + k] = c3;
            L.w2t[k * TW + o] = c2;
            L.w3t[k * TW + o] = c3;
        }
        L.w1[tid / 4][tid % 4] = round_bf(a1);
        if (tid < NH) {
            L.b1[tid] = bb[0];
            L.b2[tid] = bb[1];
            L.b3[tid] = bb[2];
            L.w4[tid] = round_bf(bb[3]);
        }
    }
    __syncthreads();

    const int u0 = 16 * wave + 4 * q;   // the lane's units u0 .. u0 + 3 of every layer
    const s16x8 none = {0, 0, 0, 0, 0, 0, 0, 0};
    const short bf_one = 0x3f80;
    const s16x8 ones = {bf_one, bf_one, bf_one, bf_one, bf_one, bf_one, bf_one, bf_one};
    const s16x8 bias_col = r == 0 ? ones : none;
    f32x4 gw3[4] = {}, gw2[4] = {}, gb3 = {}, gb2 = {}, gw1 = {}, gw4 = {}, gb4 = {};
    float loss = 0.0f;
    const float scale = (float)(2.0 * (1.0 / (double)n));

    // a layer's values at the lane's units of node 16 b + r
    auto put = [&](unsigned short *by_node, unsigned short *by_unit, int b, const float (&v)[4]) {
        const int j = 16 * b + r;
        const bf16x4 h = pack_bf16x4(v[0], v[1], v[2], v[3]);
        if (by_node) *reinterpret_cast<bf16x4 *>(by_node + j * TW + u0) = h;
#pragma unroll
        for (int i = 0; i < 4; ++i) by_unit[(u0 + i) * TN + j] = (unsigned short)h[i];
    };
    // 16 rows of w (this wavefront's) times the layer in hand, at 16 b .. + 15
    auto layer = [&](const unsigned short *w, const unsigned short *by_node, f32x4 (&acc)[2]) {
        acc[0] = acc[1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const s16x8 a = frag(w, TW, 16 * wave + r, 32 * s + 8 * q);
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[b] = mfma32(a, frag(by_node, TW, 16 * b + r, 32 * s + 8 * q), acc[b]);
        }
    };
    // rows 16 wave .. + 15 of D S^T and of D's row sums
    auto product = [&](const unsigned short *D, const unsigned short *S, f32x4 (&gw)[4], f32x4 &gb) {
        const s16x8 a = frag(D, TN, 16 * wave + r, 8 * q);
#pragma unroll
        for (int c = 0; c < 4; ++c) gw[c] = mfma32(a, frag(S, TN, 16 * c + r, 8 * q), gw[c]);
        gb = mfma32(a, bias_col, gb);
    };

    for (int64_t tile = t0; tile < t1; ++tile) {
        float z1[2][4], z2[2][4], z3[2][4], v[4];
        f32x4 acc[2];
        // layer 1 (FP32)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 w = *reinterpret_cast<const float4 *>(L.w1[u0 + i]);
                z1[b][i] = L.b1[u0 + i] + w.x * x[b].x + w.y * x[b].y + w.z * x[b].z + w.w * x[b].w;
                v[i] = fmaxf(z1[b][i], 0.0f);
            }
            put(L.by_node[0], L.h1, b, v);
            if (wave == b && q == 0) {
                const bf16x4 f = pack_bf16x4(x[b].x, x[b].y, x[b].z, x[b].w);
#pragma unroll
                for (int i = 0; i < 4; ++i) L.x[i * TN + 16 * b + r] = (unsigned short)f[i];
            }
        }
        __syncthreads();
        layer(L.w2, L.by_node[0], acc);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                z2[b][i] = acc[b][i] + L.b2[u0 + i];
                v[i] = fmaxf(z2[b][i], 0.0f);
            }
            put(L.by_node[1], L.h2, b, v);
        }
        __syncthreads();
        // layer 3 and the output unit
        layer(L.w3, L.by_node[1], acc);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            float s = 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                z3[b][i] = acc[b][i] + L.b3[u0 + i];
                v[i] = fmaxf(z3[b][i], 0.0f);
                s += L.w4[u0 + i] * v[i];
            }
            put(nullptr, L.h3, b, v);
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            if (q == 0) L.ysum[wave][16 * b + r] = s;
        }
        __syncthreads();
        // dz3 = dy W4 (z3 > 0)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int j = 16 * b + r;
            const float y = ((L.ysum[0][j] + L.ysum[1][j]) + (L.ysum[2][j] + L.ysum[3][j])) + L.b4;
            const float res = valid[b] ? y - tg[b] : 0.0f;
            const float dy = scale * res;
            if (wave == 0 && q == 0) {
                loss += res * res;
                L.dy[j] = f2bf(dy);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = z3[b][i] > 0.0f ? dy * L.w4[u0 + i] : 0.0f;
            put(L.by_node[0], L.d3, b, v);
        }
        if (tile + 1 < t1) fetch(tile + 1);
        __syncthreads();
        // dz2 = W3^T dz3 (z2 > 0); the gradients of layer 3 and the output unit
        layer(L.w3t, L.by_node[0], acc);
        product(L.d3, L.h2, gw3, gb3);
        {
            const s16x8 a = r == 0 ? *reinterpret_cast<const s16x8 *>(L.dy + 8 * q) : none;
            gw4 = mfma32(a, frag(L.h3, TN, 16 * wave + r, 8 * q), gw4);
            gb4 = mfma32(a, bias_col, gb4);
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = z2[b][i] > 0.0f ? acc[b][i] : 0.0f;
            put(L.by_node[1], L.d2, b, v);
        }
        __syncthreads();
        // dz1 = W2^T dz2 (z1 > 0)
        layer(L.w2t, L.by_node[1], acc);
        product(L.d2, L.h1, gw2, gb2);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = z1[b][i] > 0.0f ? acc[b][i] : 0.0f;
            put(nullptr, L.d1, b, v);
        }
        __syncthreads();
        {
            const s16x8 f = r < 4 ? *reinterpret_cast<const s16x8 *>(L.x + r * TN + 8 * q)
                                  : r == 4 ? ones : none;
            gw1 = mfma32(frag(L.d1, TN, 16 * wave + r, 8 * q), f, gw1);
        }
        if (tile + 1 < t1) __syncthreads();   // before this tile's h1 and x are overwritten
    }

    float *part = partials + (int64_t)blockIdx.x * (NPARAM + 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = u0 + i;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            part[OFF_W2 + m * NH + 16 * c + r] = gw2[c][i];
            part[OFF_W3 + m * NH + 16 * c + r] = gw3[c][i];
        }
        if (r < 4) part[OFF_W1 + m * 4 + r] = gw1[i];
        if (r == 4) part[OFF_B1 + m] = gw1[i];
        if (r == 0) {
            part[OFF_B2 + m] = gb2[i];
            part[OFF_B3 + m] = gb3[i];
        }
    }
    if (q == 0) part[OFF_W4 + 16 * wave + r] = gw4[0];
    if (wave == 0) {
        loss = wave_sum((double)loss);
        if (lane == 0) {
            part[OFF_B4] = gb4[0];
            part[NPARAM] = loss;
        }
    }
}

// 32 parameters a workgroup, the groups' rows in eight slices: one thread a
// parameter walked 256 rows one after the other (60 us; 4.5 us now).
__global__ __launch_bounds__(256) void k_mlp_reduce(int groups, const float *__restrict__ partials,
                                                    int64_t n, float *__restrict__ grad,
                                                    float *__restrict__ loss)
{
    __shared__ float part[8][32];
    const int c = threadIdx.x & 31, slice = threadIdx.x >> 5;
    const int p = blockIdx.x * 32 + c;
    float s = 0.0f;
    if (p <= NPARAM) {
        const float *row = partials + p;
#pragma unroll 16
        for (int g = slice; g < groups; g += 8) s += row[(int64_t)g * (NPARAM + 1)];
    }
    part[slice][c] = s;
    __syncthreads();
    if (slice || p > NPARAM) return;
    s = ((part[0][c] + part[1][c]) + (part[2][c] + part[3][c]))
      + ((part[4][c] + part[5][c]) + (part[6][c] + part[7][c]));
    if (p < NPARAM)
        grad[p] = s;
    else if (loss)
        loss[0] = (float)((double)s / (double)n);
}

__global__ __launch_bounds__(256) void k_adam(float *__restrict__ P, float *__restrict__ m,
                                              float *__restrict__ v, const float *__restrict__ g,
                                              float lr, float b1, float b2, float eps, float c1,
                                              float c2)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= NPARAM) return;
    const float gi = g[p];
    const float mi = b1 * m[p] + (1.0f - b1) * gi;
    const float vi = b2 * v[p] + (1.0f - b2) * gi * gi;
    m[p] = mi;
    v[p] = vi;
    P[p] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

}  // namespace

int mlp_nparams() { return NPARAM; }

int mlp_grad_groups(int64_t n, int max_groups)
{
    const int64_t tiles = (n + 31) / 32;
    const int64_t tpg = std::max<int64_t>(1, (tiles + max_groups - 1) / max_groups);
    return (int)((tiles + tpg - 1) / tpg);
}

size_t mlp_grad_scratch_bytes(int64_t n)
{
    return sizeof(float) * (size_t)(NPARAM + 1) * (size_t)mlp_grad_groups(n, kGradGroups);
}

// Partials of the allocation-free gradient entry point: at most
// kNoAllocGroups workgroups of NPARAM + 1 floats (8.9 MB).  Every device the
// library runs on holds its own copy until the process ends; host code never
// names this array directly (its host-side symbol is not a device address)
// but only the address that mlp_noalloc_scratch resolves per device.
static __device__ __align__(256) float scratch[(size_t)kNoAllocGroups * (NPARAM + 1)];

float *mlp_noalloc_scratch(int device)
{
    static std::mutex mu;
    static std::vector<float *> table;
    std::lock_guard<std::mutex> lock(mu);
    if (device < 0) return nullptr;
    if ((size_t)device >= table.size()) table.resize((size_t)device + 1, nullptr);
    if (!table[device]) {
        int cur = -1;
        if (hipGetDevice(&cur) != hipSuccess || cur != device) return nullptr;
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
        table[device] = static_cast<float *>(ptr);
    }
    return table[device];
}

// inference grid: 160 registers per lane leave three wavefronts per SIMD,
// i.e. three 256-thread workgroups per CU on 256 CUs, all resident at once
constexpr int64_t kInferGroups = 768;

void launch_mlp_forward(hipStream_t s, const float *P, int64_t n, const float *X, float *y)
{
    if (n <= 0) return;
    const int64_t pairs = ((n + 31) / 32 + 1) / 2;
    const int blocks = (int)std::min<int64_t>((pairs + 3) / 4, kInferGroups);
    const FeatIn in{reinterpret_cast<const float4 *>(X), nullptr, nullptr, nullptr, nullptr, 1.0,
                    MlpNorm{}};
    hipLaunchKernelGGL(k_mlp_forward<false>, dim3(blocks), dim3(256), 0, s, P, n, in, y);
}

void launch_mlp_forward_state(hipStream_t s, const float *P, int64_t n, const double *V,
                              const double *Vprev, const double *src, const float *kvp, double cm,
                              const MlpNorm &nm, float *y)
{
    if (n <= 0) return;
    const int64_t pairs = ((n + 31) / 32 + 1) / 2;
    const int blocks = (int)std::min<int64_t>((pairs + 3) / 4, kInferGroups);
    const FeatIn in{nullptr, V, Vprev, src, kvp, 1.0 / cm, nm};
    hipLaunchKernelGGL(k_mlp_forward<true>, dim3(blocks), dim3(256), 0, s, P, n, in, y);
}

// Workgroups of a gradient: one a compute unit, two from eight tiles of 32
// samples each on.  More rows of partials, 35 KB each, cost more to write and
// sum than the second workgroup gains (gradient and reduction, 256 and 512
// workgroups: 16,384 samples 18 and 24 us, 65,536 33 and 33, 262,144 92 and
// 69; with 1,024 it is 78).
constexpr int kGradLaunch = 256;
constexpr int64_t kGradLaunchTwice = 2048;   // tiles

void launch_mlp_grad(hipStream_t s, const float *P, int64_t n, const float *X, const float *T,
                     float *grad, float *loss, float *partials, int max_groups)
{
    const int64_t tiles = (n + 31) / 32;
    const int groups = mlp_grad_groups(
        n, std::min(max_groups, tiles < kGradLaunchTwice ? kGradLaunch : 2 * kGradLaunch));
    const int tpg = (int)((tiles + groups - 1) / groups);
    hipLaunchKernelGGL(k_mlp_grad, dim3(groups), dim3(256), 0, s, P, n, X, T, tpg, partials);
    hipLaunchKernelGGL(k_mlp_reduce, dim3((NPARAM + 1 + 31) / 32), dim3(256), 0, s, groups,
                       partials, n, grad, loss);
}

void launch_adam(hipStream_t s, float *P, float *m, float *v, const float *g, int t, double lr,
                 double b1, double b2, double eps)
{
    const double c1 = 1.0 - std::pow(b1, (double)t), c2 = 1.0 - std::pow(b2, (double)t);
    hipLaunchKernelGGL(k_adam, dim3((NPARAM + 255) / 256), dim3(256), 0, s, P, m, v, g, (float)lr,
                       (float)b1, (float)b2, (float)eps, (float)c1, (float)c2);
}

}  // namespace mdx
