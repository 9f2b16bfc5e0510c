// libfpo learned proposal (not part of the paper): training labels from the
// plain walk, the MLP's FP32 training kernels, FP16 fragment packing and the
// matrix-core inference the render's skip pre-pass uses.
//
// Training step for a batch of n rays (fpo_mlp_loss_grad):
//   1. mlp_grad_kernel, 64 rays a block at a time: encoding, forward pass, loss,
//      dL/d(outputs), hidden-layer deltas and the weight gradient on FP32 matrix
//      cores, activations and deltas in LDS; one partial gradient per block.
//   2. mlp_reduce_kernel: the partials summed in a fixed order (deterministic)
//      into the gradient and the batch loss.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <string>

#include "fpo.h"
#include "fpo_device.h"
#include "fpo_internal.h"
#include "fpo_proposal.h"

namespace fpo {
namespace dev {

// ---------------------------------------------------------------------------
// Labels
// ---------------------------------------------------------------------------
template <int MODE>
struct LabelVisitor {
    const TreeDev& T;
    const float* b;
    const void* snap;
    float Tr;
    float stop_T;
    float t_first, t_last;
    bool hit;

    __device__ inline bool segment(int leaf, float t0, float t1)
    {
        const float delta = t1 - t0;
        float sraw;
        if constexpr (MODE >= 16) {
            float v[32];
            sraw = SnapEval<MODE - 16>::sigma(snap, leaf, v);
        } else {
            float k[LeafEval<MODE>::kSigmaWords * LeafEval<MODE>::W];
            float scale;
            sraw = LeafEval<MODE>::sigma(T, leaf, b, k, scale);
        }
        const float sig = T.sigma_scale * fmaxf(sraw, 0.0f);
        if (!(sig * delta > 0.0f)) return false;
        if (!hit) t_first = t0;
        hit = true;
        t_last = t1;
        Tr *= __expf(-sig * delta);
        return Tr < stop_T;
    }
};

struct LabelLaunch {
    TreeDev tree;
    const float* o;
    const float* d;
    const int32_t* t_idx;
    const float* basis;
    const float* tau;
    const void* snap;
    int64_t snap_stride;
    int64_t n;
    int32_t n_t;
    float stop_T;
    float* labels;
    float* inputs;
};

template <int MODE>
__global__ __launch_bounds__(kBlock) void labels_kernel(LabelLaunch a)
{
    __shared__ int s_stack[kStackLevels * kBlock];
    const int64_t r_id = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r_id >= a.n) return;
    int ti = a.t_idx[r_id];
    ti = min(max(ti, 0), a.n_t - 1);
    float b[FPO_BASIS_STRIDE];
    const float4* brow = reinterpret_cast<const float4*>(a.basis + (int64_t)ti * FPO_BASIS_STRIDE);
#pragma unroll
    for (int i = 0; i < FPO_BASIS_STRIDE / 4; ++i) {
        const float4 v = brow[i];
        b[4 * i] = v.x; b[4 * i + 1] = v.y; b[4 * i + 2] = v.z; b[4 * i + 3] = v.w;
    }
    const void* snap = a.snap;
    if constexpr (MODE >= 16) {
        const size_t rec = (MODE - 16) == FPO_F32 ? 128 : 64;
        snap = static_cast<const char*>(a.snap) + (size_t)ti * (size_t)a.snap_stride * rec;
    }
    LabelVisitor<MODE> lv{a.tree, b, snap, 1.0f, a.stop_T, 0.0f, 0.0f, false};
    const float ox = a.o[3 * r_id], oy = a.o[3 * r_id + 1], oz = a.o[3 * r_id + 2];
    Ray r;
    float x[kMlpIn];
    float len = 1.0f;
    if (setup_ray(ox, oy, oz, a.d[3 * r_id], a.d[3 * r_id + 1], a.d[3 * r_id + 2], r)) {
        len = r.t_len;
        walk(a.tree, r, s_stack + threadIdx.x, lv);
        proposal_inputs(r, a.tau[ti], x);
    } else {
        // no chord: origin and normalised direction
        const float dx = a.d[3 * r_id], dy = a.d[3 * r_id + 1], dz = a.d[3 * r_id + 2];
        const float inv = 1.0f / sqrtf(dx * dx + dy * dy + dz * dz);
        x[0] = ox; x[1] = oy; x[2] = oz;
        x[3] = dx * inv; x[4] = dy * inv; x[5] = dz * inv;
        x[6] = a.tau[ti];
    }
    a.labels[3 * r_id] = lv.hit ? 1.0f : 0.0f;
    a.labels[3 * r_id + 1] = lv.hit ? lv.t_first / len : 0.0f;
    a.labels[3 * r_id + 2] = lv.hit ? lv.t_last / len : 0.0f;
#pragma unroll
    for (int c = 0; c < kMlpIn; ++c) a.inputs[kMlpIn * r_id + c] = x[c];
}

// ---------------------------------------------------------------------------
// FP32 training kernels
// ---------------------------------------------------------------------------
constexpr int kChunk = 64;               // rays a block takes at a time
constexpr int kGradBlocks = 256;         // one block (136 KB of LDS) per CU
constexpr int kParamsPad = FPO_MLP_N_PARAMS_PADDED;
constexpr float kQIn = 0.1f;
constexpr float kQOut = 0.9f;

__device__ inline void encode_f32(const float* x, float* g)
{
#pragma unroll
    for (int c = 0; c < kMlpIn; ++c)
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const float a = x[c] * (float)(1 << f);
            g[12 * c + 2 * f] = sinpif(a);
            g[12 * c + 2 * f + 1] = cospif(a);
        }
}

// Forward pass of one ray in FP32: the three outputs.
__device__ inline void forward_f32(const float* __restrict__ P, const float* g, float* o)
{
    float z[kMlpH], a[kMlpH];
#pragma unroll
    for (int j = 0; j < kMlpH; ++j) z[j] = P[kP1 + kMlpPE * kMlpH + j];
#pragma unroll
    for (int k = 0; k < kMlpPE; ++k) {
        const float gk = g[k];
#pragma unroll
        for (int j = 0; j < kMlpH; ++j) z[j] = fmaf(gk, P[kP1 + k * kMlpH + j], z[j]);
    }
#pragma unroll
    for (int j = 0; j < kMlpH; ++j) {
        a[j] = fmaxf(z[j], 0.0f);
        z[j] = P[kP2 + kMlpH * kMlpH + j];
    }
#pragma unroll
    for (int k = 0; k < kMlpH; ++k) {
#pragma unroll
        for (int j = 0; j < kMlpH; ++j) z[j] = fmaf(a[k], P[kP2 + k * kMlpH + j], z[j]);
    }
#pragma unroll
    for (int e = 0; e < 3; ++e) o[e] = P[kP3 + kMlpH * 3 + e];
#pragma unroll
    for (int k = 0; k < kMlpH; ++k)
#pragma unroll
        for (int e = 0; e < 3; ++e) o[e] = fmaf(fmaxf(z[k], 0.0f), P[kP3 + k * 3 + e], o[e]);
}

__global__ __launch_bounds__(kBlock) void mlp_forward_kernel(const float* __restrict__ P, const float* __restrict__ X,
                                                             int64_t n, float* __restrict__ out)
{
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r >= n) return;
    float x[kMlpIn], g[kMlpPE], o[3];
#pragma unroll
    for (int c = 0; c < kMlpIn; ++c) x[c] = X[r * kMlpIn + c];
    encode_f32(x, g);
    forward_f32(P, g, o);
#pragma unroll
    for (int e = 0; e < 3; ++e) out[r * 3 + e] = o[e];
}

__device__ inline float sigmoid_exact(float v) { return 1.0f / (1.0f + expf(-v)); }

// log(1 + u) for u in [0, 1] in FP32 only: with w = 1 + u rounded, the ratio
// u / (w - 1) corrects the rounding of w (Goldberg, "What every computer
// scientist should know about floating-point arithmetic", 1991, Thm. 4), so
// logf(w) suffices; the library's log1pf would bring an FP64 instruction in.
__device__ inline float log1p_unit(float u)
{
    const float w = 1.0f + u;
    return w == 1.0f ? u : logf(w) * (u / (w - 1.0f));
}

// LDS of mlp_grad_kernel.  Activation rows of 68 floats spread the float4 reads
// of 16 rows over all banks, weight rows of 80 the reads of 16 columns of 4 rows.
constexpr int kLd = 68;
constexpr int kLdW1 = 80;
struct GradLds {
    float w1[kMlpPE][kLdW1];
    float w2[kMlpH][kLd];
    float w3[kMlpH * 3];
    float b1[kMlpH], b2[kMlpH], b3[4];
    float g[kMlpPE][kLd];                // encoded inputs of the block's 64 rays
    float a1[kMlpH][kLd], a2[kMlpH][kLd];
    float d1[kMlpH][kLd], d2[kMlpH][kLd];
    float go[3][kLd];
    float loss[kBlock / kWave];
};
static_assert(sizeof(GradLds) <= 160 * 1024, "LDS of a CU");

// What one lane writes to LDS before this is there for the wave's others after it.
__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Gradient of the batch loss, 64 rays per block and turn, 16 per wave.  All
// products run on v_mfma_f32_16x16x4f32 (FP32 operands and sums), which adds
// its four products in order, so the forward pass and the deltas, whose K runs
// over units in order (step s takes 4 s + kq from lane group kq), are the same
// bits as fused multiply-adds one by one: which units are on does not depend on
// how the work is cut.  Lane (kq, n) works on ray n of its wave; an accumulator
// tile holds units 16 m + 4 kq + q of that ray.  Activations and deltas pass
// through LDS, [unit][ray], from where the next product reads its operand;
// after a barrier wave w forms columns 16 w .. 16 w + 15 of the weight
// gradients, its K being the block's 64 rays.  Bound by the latency around the
// matrix cores' 420 steps of 32 cycles per wave and turn (one wave per SIMD):
// a 16,384-ray batch is one turn of 256 blocks.  Before, one thread per ray
// (64 blocks) wrote 344 floats a ray, which a second kernel read back to form
// the weight gradient in 16 x 16 tiles: 118 + 48 us for that batch; this takes
// 25 us, of which about 12 are the rays' work, 5 the partial gradient's stores and the
// rest the launch and the weights (7 us more while each came as a single float).
__global__ __launch_bounds__(kBlock) void mlp_grad_kernel(const float* __restrict__ P, const float* __restrict__ X,
                                                          const float* __restrict__ Y, const int32_t* __restrict__ idx,
                                                          int64_t n_rays, int64_t n_chunks, float inv_n,
                                                          float* __restrict__ part)
{
    __shared__ __align__(16) GradLds S;
    const int tid = threadIdx.x;
    const int wv = tid / kWave;
    const int ln = tid % kWave;
    const int n = ln & 15;
    const int kq = ln >> 4;
    // the weights, every load in flight at once; parameters that are not 16-byte
    // aligned come as single floats
    constexpr int kW = kMlpH / 4;            // float4 per row
    constexpr int kLoads1 = (kMlpPE * kW + kBlock - 1) / kBlock, kLoads2 = kMlpH * kW / kBlock;
    const bool wide = (reinterpret_cast<uintptr_t>(P) & 15) == 0;
    auto load4 = [&](int at) {
        if (wide) return *reinterpret_cast<const f32x4*>(P + at);
        return f32x4{P[at], P[at + 1], P[at + 2], P[at + 3]};
    };
    f32x4 l1[kLoads1], l2[kLoads2];
#pragma unroll
    for (int i = 0; i < kLoads1; ++i) {
        const int e = i * kBlock + tid;
        l1[i] = e < kMlpPE * kW ? load4(kP1 + e * 4) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int i = 0; i < kLoads2; ++i) l2[i] = load4(kP2 + (i * kBlock + tid) * 4);
#pragma unroll
    for (int i = 0; i < kLoads1; ++i) {
        const int e = i * kBlock + tid;
        if (e < kMlpPE * kW) *reinterpret_cast<f32x4*>(&S.w1[e / kW][e % kW * 4]) = l1[i];
    }
#pragma unroll
    for (int i = 0; i < kLoads2; ++i) {
        const int e = i * kBlock + tid;
        *reinterpret_cast<f32x4*>(&S.w2[e / kW][e % kW * 4]) = l2[i];
    }
    if (tid < kMlpH * 3) S.w3[tid] = P[kP3 + tid];
    if (tid < kMlpH) {
        S.b1[tid] = P[kP1 + kMlpPE * kMlpH + tid];
        S.b2[tid] = P[kP2 + kMlpH * kMlpH + tid];
    }
    if (tid < 3) S.b3[tid] = P[kP3 + kMlpH * 3 + tid];
    __syncthreads();

    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 acc1[6], acc2[5], acc3[2];         // this wave's columns of dW1, dW2, dW3
#pragma unroll
    for (int t = 0; t < 6; ++t) acc1[t] = zero;
#pragma unroll
    for (int t = 0; t < 5; ++t) acc2[t] = zero;
    acc3[0] = acc3[1] = zero;
    float loss_sum = 0.0f;
    const int ray = 16 * wv + n;             // column of the LDS rows

    for (int64_t ch = blockIdx.x; ch < n_chunks; ch += gridDim.x) {
        const int64_t r = ch * kChunk + ray;
        const bool live = r < n_rays;
        const int64_t row = live ? (idx ? (int64_t)idx[r] : r) : 0;
        float x[kMlpIn], y[3];
#pragma unroll
        for (int c = 0; c < kMlpIn; ++c) x[c] = live ? X[row * kMlpIn + c] : 0.0f;
#pragma unroll
        for (int e = 0; e < 3; ++e) y[e] = live ? Y[row * 3 + e] : 0.0f;

        // encoding: lane group kq takes arguments 4 t + kq, argument i being input
        // i / 6 times 2^(i % 6), features 2 i (sine) and 2 i + 1 (cosine)
#pragma unroll
        for (int t = 0; t < (6 * kMlpIn + 3) / 4; ++t) {
            float arg = 0.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = 4 * t + q;
                if (i < 6 * kMlpIn) arg = kq == q ? x[i / 6] * (float)(1 << (i % 6)) : arg;
            }
            if (4 * t + kq < 6 * kMlpIn) {
                S.g[8 * t + 2 * kq][ray] = live ? sinpif(arg) : 0.0f;
                S.g[8 * t + 2 * kq + 1][ray] = live ? cospif(arg) : 0.0f;
            }
        }
        wave_lds_sync();
        // layer 1
        f32x4 z[4];
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) z[m][q] = S.b1[16 * m + 4 * kq + q];
#pragma unroll
        for (int s = 0; s < kMlpPE / 4; ++s) {
            const float v = S.g[4 * s + kq][ray];
#pragma unroll
            for (int m = 0; m < 4; ++m)
                z[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(S.w1[4 * s + kq][16 * m + n], v, z[m], 0, 0, 0);
        }
        uint32_t on1 = 0, on2 = 0;           // z > 0 of this lane's 16 units
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                on1 |= (uint32_t)(z[m][q] > 0.0f) << (4 * m + q);
                S.a1[16 * m + 4 * kq + q][ray] = live ? fmaxf(z[m][q], 0.0f) : 0.0f;
                z[m][q] = S.b2[16 * m + 4 * kq + q];
            }
        wave_lds_sync();
        // layer 2
#pragma unroll
        for (int s = 0; s < kMlpH / 4; ++s) {
            const float v = S.a1[4 * s + kq][ray];
#pragma unroll
            for (int m = 0; m < 4; ++m)
                z[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(S.w2[4 * s + kq][16 * m + n], v, z[m], 0, 0, 0);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                on2 |= (uint32_t)(z[m][q] > 0.0f) << (4 * m + q);
                S.a2[16 * m + 4 * kq + q][ray] = live ? fmaxf(z[m][q], 0.0f) : 0.0f;
            }
        wave_lds_sync();
        // outputs: rows 0 .. 2 of a tile, in lane group 0; to all four of the ray's lanes
        f32x4 oz = {S.b3[0], S.b3[1], S.b3[2], 0.0f};
#pragma unroll
        for (int s = 0; s < kMlpH / 4; ++s) {
            const float w = n < 3 ? S.w3[(4 * s + kq) * 3 + n] : 0.0f;
            oz = __builtin_amdgcn_mfma_f32_16x16x4f32(w, S.a2[4 * s + kq][ray], oz, 0, 0, 0);
        }
        float o[3];
#pragma unroll
        for (int e = 0; e < 3; ++e) o[e] = __shfl(oz[e], n, kWave);
        // loss and dL/do: logistic loss on the hit logit, pinball on the sigmoid
        // of the interval outputs for rays that hit
        float loss = fmaxf(o[0], 0.0f) - y[0] * o[0] + log1p_unit(expf(-fabsf(o[0])));
        float go[3];
        go[0] = sigmoid_exact(o[0]) - y[0];
        const bool hit = y[0] > 0.5f;
        const float qq[2] = {kQIn, kQOut};
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float sg = sigmoid_exact(o[1 + e]);
            const float u = y[1 + e] - sg;
            const float w = qq[e] - (u < 0.0f ? 1.0f : 0.0f);
            loss += hit ? u * w : 0.0f;
            go[1 + e] = hit ? -w * sg * (1.0f - sg) : 0.0f;
        }
#pragma unroll
        for (int e = 0; e < 3; ++e) go[e] = live ? go[e] * inv_n : 0.0f;
        if (kq == 0) {
#pragma unroll
            for (int e = 0; e < 3; ++e) S.go[e][ray] = go[e];
            loss_sum += live ? loss * inv_n : 0.0f;
        }
        // deltas: d2 = (W3 go) . [z2 > 0]; d1 = (W2 d2) . [z1 > 0]
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int u = 16 * m + 4 * kq + q;
                float v = 0.0f;
#pragma unroll
                for (int e = 0; e < 3; ++e) v = fmaf(go[e], S.w3[u * 3 + e], v);
                S.d2[u][ray] = ((on2 >> (4 * m + q)) & 1) ? v : 0.0f;
                z[m][q] = 0.0f;
            }
        wave_lds_sync();
#pragma unroll
        for (int s = 0; s < kMlpH / 4; ++s) {
            const float v = S.d2[4 * s + kq][ray];
#pragma unroll
            for (int m = 0; m < 4; ++m)
                z[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(S.w2[16 * m + n][4 * s + kq], v, z[m], 0, 0, 0);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                S.d1[16 * m + 4 * kq + q][ray] = ((on1 >> (4 * m + q)) & 1) && live ? z[m][q] : 0.0f;
        __syncthreads();

        // weight gradients: K step (k, q) takes rays 16 k + 4 kq + q
        const float one = n == 0 ? 1.0f : 0.0f;          // bias tile: row 0
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int at = 16 * k + 4 * kq;
            const f32x4 e1 = *reinterpret_cast<const f32x4*>(&S.d1[16 * wv + n][at]);
            const f32x4 e2 = *reinterpret_cast<const f32x4*>(&S.d2[16 * wv + n][at]);
            const f32x4 e3 = n < 3 ? *reinterpret_cast<const f32x4*>(&S.go[n][at]) : zero;
#pragma unroll
            for (int t = 0; t < 6; ++t) {
                f32x4 v;
                if (t < 5) {
                    v = *reinterpret_cast<const f32x4*>(&S.g[16 * t + n][at]);
                } else {                                 // rows 80 .. 83, then the bias row
                    v = n == 4 ? f32x4{1.0f, 1.0f, 1.0f, 1.0f} : zero;
                    if (n < 4) v = *reinterpret_cast<const f32x4*>(&S.g[80 + n][at]);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) acc1[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[q], e1[q], acc1[t], 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(&S.a1[16 * t + n][at]);
#pragma unroll
                for (int q = 0; q < 4; ++q) acc2[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[q], e2[q], acc2[t], 0, 0, 0);
            }
            const f32x4 v = *reinterpret_cast<const f32x4*>(&S.a2[16 * wv + n][at]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc2[4] = __builtin_amdgcn_mfma_f32_16x16x4f32(one, e2[q], acc2[4], 0, 0, 0);
                acc3[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[q], e3[q], acc3[0], 0, 0, 0);
                acc3[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(one, e3[q], acc3[1], 0, 0, 0);
            }
        }
        __syncthreads();
    }

    float* out = part + (int64_t)blockIdx.x * kParamsPad;
    const int j = 16 * wv + n;
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = 16 * t + 4 * kq + q;
            if (k <= kMlpPE) out[kP1 + k * kMlpH + j] = acc1[t][q];
        }
#pragma unroll
    for (int t = 0; t < 5; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = 16 * t + 4 * kq + q;
            if (k <= kMlpH) out[kP2 + k * kMlpH + j] = acc2[t][q];
        }
    if (n < 3) {
#pragma unroll
        for (int q = 0; q < 4; ++q) out[kP3 + (16 * wv + 4 * kq + q) * 3 + n] = acc3[0][q];
        if (wv == 0 && kq == 0) out[kP3 + kMlpH * 3 + n] = acc3[1][0];
    }
    loss_sum = wave_sum(loss_sum);
    if (ln == 0) S.loss[wv] = loss_sum;
    __syncthreads();
    if (tid == 0) out[FPO_MLP_N_PARAMS] = (S.loss[0] + S.loss[1]) + (S.loss[2] + S.loss[3]);
}

// grad += the partials' sum, loss += their last float's.  32 parameters a
// block, 8 threads each over every eighth partial (as many loads in flight),
// combined in a fixed order.
__global__ __launch_bounds__(256) void mlp_reduce_kernel(const float* __restrict__ part, int n_part,
                                                         float* __restrict__ grad, float* __restrict__ loss)
{
    __shared__ float red[8][32];
    const int c = threadIdx.x & 31, q = threadIdx.x >> 5;
    const int i = blockIdx.x * 32 + c;
    float s = 0.0f;
    if (i < kParamsPad) {
#pragma unroll 8
        for (int b = q; b < n_part; b += 8) s += part[(int64_t)b * kParamsPad + i];
    }
    red[q][c] = s;
    __syncthreads();
    if (q != 0 || i >= kParamsPad) return;
    s = ((red[0][c] + red[1][c]) + (red[2][c] + red[3][c])) + ((red[4][c] + red[5][c]) + (red[6][c] + red[7][c]));
    if (i < FPO_MLP_N_PARAMS) grad[i] += s;
    else loss[0] += s;
}

// ---------------------------------------------------------------------------
// FP16 fragments and matrix-core inference
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void mlp_pack_kernel(const float* __restrict__ P, unsigned char* __restrict__ out)
{
    const int id = blockIdx.x * 256 + threadIdx.x;
    if (id < kFrags * 64) {
        const int fi = id / 64, ln = id % 64;
        const int m = ln & 15, q = ln >> 4;
        _Float16 h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float v = 0.0f;
            if (fi < kFrag2) {                       // A = W1^T: [64 out][96 features]
                const int mt = fi / 6, kb = fi % 6;
                const int row = 16 * mt + m, k = 16 * kb + 4 * q + e;
                if (k < kMlpPE) v = P[kP1 + k * kMlpH + row];
            } else if (fi < kFrag3) {                // A = W2^T
                const int g = fi - kFrag2, mt = g / 4, kb = g % 4;
                const int row = 16 * mt + m, k = 16 * kb + 4 * q + e;
                v = P[kP2 + k * kMlpH + row];
            } else {                                 // A = W3^T, rows 0..2 of 16
                const int kb = fi - kFrag3;
                const int k = 16 * kb + 4 * q + e;
                if (m < 3) v = P[kP3 + k * 3 + m];
            }
            h[e] = (_Float16)v;
        }
        reinterpret_cast<f16x4*>(out)[id] = f16x4{h[0], h[1], h[2], h[3]};
        return;
    }
    const int b = id - kFrags * 64;
    float* bias = reinterpret_cast<float*>(out + kPackedBias);
    if (b < 64) bias[b] = P[kP1 + kMlpPE * kMlpH + b];
    else if (b < 128) bias[b] = P[kP2 + kMlpH * kMlpH + (b - 64)];
    else if (b < 131) bias[b] = P[kP3 + kMlpH * 3 + (b - 128)];
    else if (b == 131) bias[b] = 0.0f;
}

__global__ __launch_bounds__(kBlock) void mlp_infer_kernel(const unsigned char* __restrict__ packed,
                                                           const float* __restrict__ X, int64_t n,
                                                           float* __restrict__ out)
{
    const int64_t base = ((int64_t)blockIdx.x * kBlock + threadIdx.x) & ~(int64_t)63;
    if (base >= n) return;                      // whole waves only
    const int64_t r = base + (threadIdx.x & 63);
    const bool live = r < n;
    float x[kMlpIn];
#pragma unroll
    for (int c = 0; c < kMlpIn; ++c) x[c] = live ? X[r * kMlpIn + c] : 0.0f;
    float o[3];
    mlp_infer_wave(reinterpret_cast<const uint2*>(packed), reinterpret_cast<const float*>(packed + kPackedBias), x, o);
    if (live)
#pragma unroll
        for (int e = 0; e < 3; ++e) out[r * 3 + e] = o[e];
}

}  // namespace dev
}  // namespace fpo

using namespace fpo;

static int64_t mlp_ld(int64_t n) { return (n + dev::kChunk - 1) / dev::kChunk * dev::kChunk; }

extern "C" int64_t fpo_mlp_workspace_floats(int64_t n)
{
    ApiRange api_range_("fpo_mlp_workspace_floats");
    if (n < 1) return 0;
    // fixed by the interface; the partial gradients take at most kGradBlocks *
    // kParamsPad floats of it
    return 344 * mlp_ld(n) + (mlp_ld(n) + 1023) / 1024 * dev::kParamsPad;
}

template <int MODE>
static void launch_labels(const dev::LabelLaunch& a, int64_t grid, hipStream_t s)
{
    hipLaunchKernelGGL(dev::labels_kernel<MODE>, dim3((unsigned)grid), dim3(dev::kBlock), 0, s, a);
}

extern "C" fpo_status fpo_ray_labels(const fpo_tree_view* tree, const float* o, const float* d, const int32_t* t_idx,
                                     const float* basis, const float* tau, int32_t n_t, int64_t n_rays,
                                     const fpo_render_opts* opts, float* labels, float* inputs, void* stream)
{
    ApiRange api_range_("fpo_ray_labels");
    fpo_status st = check_tree(tree, opts == nullptr || opts->snapshot == nullptr);
    if (st != FPO_OK) return st;
    if ((st = check_opts(opts, tree)) != FPO_OK) return st;
    if (n_rays < 0) return fail(FPO_E_INVALID, "n_rays < 0");
    if (n_rays == 0) return FPO_OK;
    if (!o || !d || !t_idx || !basis || !tau || !labels || !inputs) return fail(FPO_E_INVALID, "NULL device pointer");
    if (n_t < 1) return fail(FPO_E_INVALID, "n_t must be >= 1");
    if (n_rays > (int64_t)INT32_MAX * dev::kBlock) return fail(FPO_E_INVALID, "too many rays");
    dev::LabelLaunch a;
    std::memset(&a, 0, sizeof(a));
    a.tree = dev::tree_dev(tree);
    a.o = o; a.d = d; a.t_idx = t_idx; a.basis = basis; a.tau = tau; a.n_t = n_t; a.n = n_rays;
    a.snap = opts->snapshot;
    a.snap_stride = opts->snapshot_cam_stride;
    a.stop_T = opts->stop_T;
    a.labels = labels;
    a.inputs = inputs;
    const int64_t grid = (n_rays + dev::kBlock - 1) / dev::kBlock;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int mode = opts->snapshot ? 16 + (int)opts->snapshot_dtype : (int)tree->dtype;
    switch (mode) {
        case FPO_F32: launch_labels<FPO_F32>(a, grid, s); break;
        case FPO_BF16: launch_labels<FPO_BF16>(a, grid, s); break;
        case FPO_FP8_E4M3: launch_labels<FPO_FP8_E4M3>(a, grid, s); break;
        case dev::kSnapF32: launch_labels<dev::kSnapF32>(a, grid, s); break;
        case dev::kSnapBF16: launch_labels<dev::kSnapBF16>(a, grid, s); break;
        default: return fail(FPO_E_INVALID, "unknown render mode");
    }
    return launch_status("fpo_ray_labels");
}

extern "C" fpo_status fpo_mlp_forward(const float* params, const float* inputs, int64_t n, float* out, void* stream)
{
    ApiRange api_range_("fpo_mlp_forward");
    if (n < 0) return fail(FPO_E_INVALID, "n < 0");
    if (n == 0) return FPO_OK;
    if (!params || !inputs || !out) return fail(FPO_E_INVALID, "NULL device pointer");
    if (n > (int64_t)INT32_MAX * dev::kBlock) return fail(FPO_E_INVALID, "n too large");
    const int64_t grid = (n + dev::kBlock - 1) / dev::kBlock;
    hipLaunchKernelGGL(dev::mlp_forward_kernel, dim3((unsigned)grid), dim3(dev::kBlock), 0,
                       static_cast<hipStream_t>(stream), params, inputs, n, out);
    return launch_status("fpo_mlp_forward");
}

extern "C" fpo_status fpo_mlp_loss_grad(const float* params, const float* inputs, const float* labels,
                                        const int32_t* idx, int64_t n, float* workspace, float* grad, float* loss,
                                        void* stream)
{
    ApiRange api_range_("fpo_mlp_loss_grad");
    if (n < 1) return fail(FPO_E_INVALID, "n must be >= 1");
    if (!params || !inputs || !labels || !workspace || !grad || !loss) return fail(FPO_E_INVALID, "NULL device pointer");
    if ((reinterpret_cast<uintptr_t>(workspace) & 15) != 0) return fail(FPO_E_INVALID, "workspace must be 16-byte aligned");
    if (mlp_ld(n) > (int64_t)1 << 30) return fail(FPO_E_INVALID, "batch too large");
    hipStream_t s = static_cast<hipStream_t>(stream);
    // a block takes every kGradBlocks-th chunk of 64 rays; the partials (39 KB
    // per block, at most one block per chunk) fit the workspace's 86 KB a chunk
    const int64_t chunks = mlp_ld(n) / dev::kChunk;
    const int blocks = (int)std::min<int64_t>(chunks, dev::kGradBlocks);
    hipLaunchKernelGGL(dev::mlp_grad_kernel, dim3(blocks), dim3(dev::kBlock), 0, s, params, inputs, labels, idx, n,
                       chunks, 1.0f / (float)n, workspace);
    fpo_status st = launch_status("fpo_mlp_loss_grad");
    if (st != FPO_OK) return st;
    hipLaunchKernelGGL(dev::mlp_reduce_kernel, dim3((dev::kParamsPad + 31) / 32), dim3(256), 0, s, workspace, blocks,
                       grad, loss);
    return launch_status("fpo_mlp_loss_grad (reduce)");
}

extern "C" fpo_status fpo_mlp_pack(const float* params, void* packed_out, void* stream)
{
    ApiRange api_range_("fpo_mlp_pack");
    if (!params || !packed_out) return fail(FPO_E_INVALID, "NULL device pointer");
    if ((reinterpret_cast<uintptr_t>(packed_out) & 15) != 0) return fail(FPO_E_INVALID, "packed_out must be 16-byte aligned");
    const int n = dev::kFrags * 64 + 132;
    hipLaunchKernelGGL(dev::mlp_pack_kernel, dim3((n + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(stream),
                       params, static_cast<unsigned char*>(packed_out));
    return launch_status("fpo_mlp_pack");
}

extern "C" fpo_status fpo_mlp_infer(const void* packed, const float* inputs, int64_t n, float* out, void* stream)
{
    ApiRange api_range_("fpo_mlp_infer");
    if (n < 0) return fail(FPO_E_INVALID, "n < 0");
    if (n == 0) return FPO_OK;
    if (!packed || !inputs || !out) return fail(FPO_E_INVALID, "NULL device pointer");
    if ((reinterpret_cast<uintptr_t>(packed) & 15) != 0) return fail(FPO_E_INVALID, "packed must be 16-byte aligned");
    if (n > (int64_t)INT32_MAX * dev::kBlock) return fail(FPO_E_INVALID, "n too large");
    const int64_t grid = (n + dev::kBlock - 1) / dev::kBlock;
    hipLaunchKernelGGL(dev::mlp_infer_kernel, dim3((unsigned)grid), dim3(dev::kBlock), 0, static_cast<hipStream_t>(stream),
                       static_cast<const unsigned char*>(packed), inputs, n, out);
    return launch_status("fpo_mlp_infer");
}
