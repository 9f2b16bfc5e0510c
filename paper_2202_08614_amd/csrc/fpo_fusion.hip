// libfpo PlenOctree fusion (Sec. 3, fine stage; Eq. 3-5).
//
// Observe pass, per view: every pixel ray walks the static PlenOctree front
// to back with the transmittance of the current leaf values; each leaf
// segment entered with T > tau is an observation of the radiance field at its
// midpoint, weighted by T times its length, accumulated per leaf with FP32
// atomics.  Apply pass: one update of Eq. 3-5 for every leaf observed in the
// view, with the view's length-weighted mean transmittance as T_i.
//
// Readings of the paper: its query points are the leaf segments (a sampler
// stepping along the ray puts a number of points proportional to the chord
// into a leaf); all observations of one leaf in one view make one update;
// z_{c,j} is updated with Y_j(d) c_c(x, d), the colour projected on the SH
// basis of the view direction.  The radiance field is an analytic stand-in
// for the generalizable network (Gaussian mixture density, logistic
// view-dependent colour).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>

#include "fpo.h"
#include "fpo_device.h"
#include "fpo_internal.h"

namespace fpo {
namespace dev {

struct FieldDev {
    float mu[FPO_FIELD_MAX_GAUSS][3];
    float inv2w2[FPO_FIELD_MAX_GAUSS];    // 1 / (2 w_g^2)
    float a[FPO_FIELD_MAX_GAUSS];
    int32_t n;
    float u[3][3];
    float v[3][3];
    float b[3];
};

struct FusionLaunch {
    TreeDev tree;
    const float* values;    // [stride][32] leaf records: sigma, z_{c,j} at 1 + 9c + j
    float* acc;             // [stride][FPO_FUSION_ACC]
    float frame[12];        // eye, forward, right * tan_x, up * tan_y
    int32_t W, H, bx;       // image size, 16 x 16 tiles per row
    float tau;
    FieldDev f;
    const int32_t* only_if; // null, or run only if it is not zero (fpo_fusion_view)
};

__device__ inline float field_sigma(const FieldDev& f, const float x[3])
{
    float s = 0.0f;
#pragma unroll
    for (int g = 0; g < FPO_FIELD_MAX_GAUSS; ++g) {
        if (g >= f.n) break;
        const float dx = x[0] - f.mu[g][0], dy = x[1] - f.mu[g][1], dz = x[2] - f.mu[g][2];
        const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
        s = fmaf(f.a[g], __expf(-r2 * f.inv2w2[g]), s);
    }
    return s;
}

__device__ inline void field_colour(const FieldDev& f, const float* x, const float* d, float* col)
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        float h = f.b[c];
#pragma unroll
        for (int a = 0; a < 3; ++a) h = fmaf(f.u[c][a], x[a], fmaf(f.v[c][a], d[a], h));
        col[c] = sigmoidf_(h);
    }
}

// Direction of a pixel's ray (not normalised).
__device__ inline void pixel_dir(const float* fr, int W, int H, int px, int py, float* d)
{
    const float sx = (float)(2 * px + 1 - W) / (float)W;
    const float sy = (float)(H - 2 * py - 1) / (float)H;
#pragma unroll
    for (int c = 0; c < 3; ++c) d[c] = fr[3 + c] + sx * fr[6 + c] + sy * fr[9 + c];
}

constexpr int kObs = 30;            // accumulator values per observation
constexpr int kObsStride = 36;      // LDS floats per staged observation (9 x 16 bytes: spreads banks)

// The lanes that shade a segment in the same step stage their observations in
// the wave's LDS buffer and then add them to the accumulators together: the
// (observation, value) pairs are dealt out over those lanes, so one atomic
// instruction covers consecutive values of one or two leaf records instead of
// the same value of up to 64 different leaves.
struct FusionVisitor {
    const float* values;
    float* acc;
    const FieldDev& f;
    float* stage;           // this wave's [64][kObsStride] LDS buffer
    int lane;
    float o[3];             // entry point: walk distances are measured from it
    float d[3];             // unit direction
    float Y[FPO_N_SH];
    float T;
    float tau;
    float sigma_scale;

    __device__ inline bool segment(int leaf, float t0, float t1)
    {
        if (!(T > tau)) return true;
        const float delta = t1 - t0;
        const bool obs = delta > 0.0f;
        const uint64_t act = __ballot(obs);
        if (obs) {
            const int k = __popcll(act);
            const int rank = __popcll(act & ((1ull << lane) - 1ull));
            const float tm = 0.5f * (t0 + t1);
            const float x[3] = {fmaf(tm, d[0], o[0]), fmaf(tm, d[1], o[1]), fmaf(tm, d[2], o[2])};
            const float sig = field_sigma(f, x);
            float col[3];
            field_colour(f, x, d, col);
            const float w = T * delta;
            float v[kObsStride];
            v[0] = w;
            v[1] = w * sig;
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int j = 0; j < FPO_N_SH; ++j) v[2 + c * FPO_N_SH + j] = w * col[c] * Y[j];
            v[29] = delta;
            v[30] = 0.0f;
            v[31] = __int_as_float(leaf);
#pragma unroll
            for (int e = 32; e < kObsStride; ++e) v[e] = 0.0f;
            float4* st = reinterpret_cast<float4*>(stage + rank * kObsStride);
#pragma unroll
            for (int q = 0; q < kObsStride / 4; ++q) st[q] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            for (int p = rank; p < k * kObs; p += k) {
                const int s = p / kObs;
                const int e = p - s * kObs;
                const float* src = stage + s * kObsStride;
                const int l = __float_as_int(src[31]);
                unsafeAtomicAdd(acc + (int64_t)l * FPO_FUSION_ACC + e, src[e]);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            T *= __expf(-sigma_scale * fmaxf(values[(int64_t)leaf * 32], 0.0f) * delta);
        }
        return !(T > tau);
    }
};

// One camera; 16 x 16 pixel tiles per block, 8 x 8 per wave (as the render).
__global__ __launch_bounds__(kBlock) void fusion_observe_kernel(FusionLaunch a)
{
    __shared__ int s_stack[kStackLevels * kBlock];
    __shared__ __align__(16) float s_obs[kBlock / kWave][kWave * kObsStride];
    if (a.only_if && *a.only_if == 0) return;
    const int wv = threadIdx.x >> 6;
    const int ln = threadIdx.x & 63;
    const int bxi = blockIdx.x % a.bx;
    const int byi = blockIdx.x / a.bx;
    const int px = bxi * 16 + (wv & 1) * 8 + (ln & 7);
    const int py = byi * 16 + (wv >> 1) * 8 + (ln >> 3);
    if (px >= a.W || py >= a.H) return;
    float dir[3];
    pixel_dir(a.frame, a.W, a.H, px, py, dir);
    Ray r;
    if (!setup_ray(a.frame[0], a.frame[1], a.frame[2], dir[0], dir[1], dir[2], r)) return;
    FusionVisitor vis{a.values, a.acc, a.f, s_obs[wv], ln};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        vis.o[c] = r.o[c];
        vis.d[c] = r.d[c];
    }
    sh9(r.d[0], r.d[1], r.d[2], vis.Y);
    vis.T = 1.0f;
    vis.tau = a.tau;
    vis.sigma_scale = a.tree.sigma_scale;
    walk(a.tree, r, s_stack + threadIdx.x, vis);
}

// Eq. 3-5 of one observed leaf: values V, weight and count from the view's sums A
// and observed length len.
__device__ inline void update_leaf(const float* A, float len, float* V, float& weight, int32_t& count)
{
    const float inv = 1.0f / len;
    const float Ti = A[0] * inv;                     // length-weighted mean transmittance
    const float Wp = weight;
    const float den = 1.0f / (Wp + Ti);
    V[0] = fmaf(Wp, V[0], A[1] * inv) * den;                                  // Eq. 3
#pragma unroll
    for (int q = 0; q < 27; ++q) V[1 + q] = fmaf(Wp, V[1 + q], A[2 + q] * inv) * den;   // Eq. 4
    const int32_t C = count + 1;                                                // Eq. 5
    count = C;
    weight = (float)(C - 1) / (float)C * Wp + Ti / (float)C;
}

// Eq. 3-5 for every observed leaf, then clear its accumulator.
__global__ __launch_bounds__(kBlock) void fusion_apply_kernel(float4* values, float* weight, int32_t* count,
                                                              float4* acc, int64_t n, const int32_t* only_if)
{
    const int64_t l = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (l >= n || (only_if && *only_if == 0)) return;
    float4* A4 = acc + l * (FPO_FUSION_ACC / 4);
    const float len = A4[7].y;                       // acc[29]
    if (!(len > 0.0f)) return;
    float A[FPO_FUSION_ACC];
    float V[32];
    float4* V4 = values + l * 8;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        const float4 x = A4[w];
        A[4 * w] = x.x; A[4 * w + 1] = x.y; A[4 * w + 2] = x.z; A[4 * w + 3] = x.w;
        const float4 y = V4[w];
        V[4 * w] = y.x; V[4 * w + 1] = y.y; V[4 * w + 2] = y.z; V[4 * w + 3] = y.w;
    }
    update_leaf(A, len, V, weight[l], count[l]);
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        V4[w] = make_float4(V[4 * w], V[4 * w + 1], V[4 * w + 2], V[4 * w + 3]);
        A4[w] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
}

// --------------------------------------------------------------------------
// One view at once (fpo_fusion_view).  The observations of a leaf are few (a
// leaf covers a handful of pixels) and arrive from all over the grid, so
// instead of 30 atomic adds each they are kept: the walk appends each observed
// segment {t0, t1, T, ray part} to its leaf's linked list (one atomic exchange
// of the list's head), and a second kernel, one thread per leaf, goes through
// the list, evaluates the field and applies Eq. 3-5 to sums that never leave
// its registers.  The rays are walked in parts (see walk_parts), with T from 1
// in each part; the second kernel multiplies by the transmittance in front of
// the part and drops what is entered with T <= tau.
// One 800x800 view of 2 M leaves: 1.94 ms with atomic sums (walk and sums 1.65,
// apply 0.29), 0.58 ms so (walk 0.35, bound by its chains of reads as the
// renders are; the leaves' pass 0.22).
// --------------------------------------------------------------------------
// The nodes are dealt out in chunks from kPools counters, each with its share
// of them, on a cache line of its own: with a single counter and chunks of 128
// the walk of an 800x800 view took 774 us, mostly waiting for it.
constexpr int kNodeChunk = 64;       // nodes a wave takes at a time (at least its lanes)
constexpr int kPools = 64;
constexpr int kPoolStride = 32;      // int32 from one counter to the next
constexpr int kPoolInts = kPools * kPoolStride + 1;   // the last one: overflow

struct ListLaunch {
    TreeDev tree;
    const float* values;
    float frame[12];
    int32_t W, H, bx;       // image size, blocks per row of tiles
    float tau;
    int32_t* pool;          // [kPoolInts] nodes taken from each share; overflow
    int32_t* head;          // [n_leaves] last node of the leaf's list, -1 none
    float4* node;           // [kPools * share] t0, t1, T, pixel * parts + part
    int32_t* next;          // [kPools * share]
    float* Tin;             // [H * W * parts] transmittance in front of the part
    int32_t share;          // nodes per counter
    int64_t n_leaves;
};

// The list form of ListLaunch's second kernel.
struct GatherLaunch {
    ListLaunch l;
    FieldDev f;
    float* weight;
    int32_t* count;
    float* acc;
    int32_t parts;
};

__global__ __launch_bounds__(kBlock) void fusion_clear_kernel(int32_t* pool, int4* head, int64_t n4)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n4) head[i] = make_int4(-1, -1, -1, -1);
    if (i < kPoolInts) pool[i] = 0;
}

struct ListVisitor {
    const ListLaunch& a;
    volatile int* chunk;    // this wave's {next node, end} in LDS
    int which;              // counter the wave takes chunks from
    int lane;
    int id;                 // pixel * parts + part
    float T;
    float sigma;            // of the leaf being visited (prefetch_leaf)
    int pend_node, pend_prev;   // an exchange whose result is not stored yet

    __device__ inline void flush()
    {
        if (pend_node >= 0) a.next[pend_node] = pend_prev;
        pend_node = -1;
    }

    __device__ inline bool segment(int leaf, float t0, float t1)
    {
        if (!(T > a.tau)) return true;
        const float delta = t1 - t0;
        if (delta > 0.0f) {
            const uint64_t act = __ballot(1);
            const int rank = __popcll(act & ((1ull << lane) - 1ull));
            const int k = __popcll(act);
            const int lead = __ffsll((unsigned long long)act) - 1;
            int at = 0;
            if (lane == lead) {
                at = chunk[0];
                if (at + k > chunk[1]) {
                    at = atomicAdd(a.pool + which * kPoolStride, kNodeChunk);
                    if (at < 0 || at > a.share - kNodeChunk) {
                        a.pool[kPoolInts - 1] = 1;   // no room: the view is done with atomic sums instead
                        at = -1;
                    } else {
                        at += which * a.share;
                        chunk[1] = at + kNodeChunk;
                    }
                }
                if (at >= 0) chunk[0] = at + k;
            }
            at = __shfl(at, lead, kWave);
            if (at < 0) return true;
            const int n = at + rank;
            a.node[n] = make_float4(t0, t1, T, __int_as_float(id));
            flush();
            pend_prev = atomicExch(a.head + leaf, n);
            pend_node = n;
            T *= __expf(-a.tree.sigma_scale * fmaxf(sigma, 0.0f) * delta);
        }
        return !(T > a.tau);
    }
};

__device__ inline void prefetch_leaf(ListVisitor& v, int leaf) { v.sigma = v.a.values[(int64_t)leaf * 32]; }

// 64 / PARTS pixels per wave, four waves per block.
template <int PARTS>
__global__ __launch_bounds__(kBlock) void fusion_list_kernel(ListLaunch a)
{
    constexpr int kSlots = kWave / PARTS;
    constexpr int kW = PARTS == 8 ? 4 : 2;
    constexpr int kH = kSlots / kW;
    __shared__ int s_stack[kStackLevels * kBlock];
    __shared__ int s_chunk[kBlock / kWave][2];
    const int wv = threadIdx.x / kWave;
    const int ln = threadIdx.x % kWave;
    const int part = ln / kSlots, slot = ln % kSlots;
    if (ln < 2) s_chunk[wv][ln] = 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int px = (blockIdx.x % a.bx) * 2 * kW + (wv & 1) * kW + slot % kW;
    const int py = (blockIdx.x / a.bx) * 2 * kH + (wv >> 1) * kH + slot / kW;
    if (px >= a.W || py >= a.H) return;               // all lanes of a pixel together
    float dir[3];
    pixel_dir(a.frame, a.W, a.H, px, py, dir);
    // distances run from the cube's face, as in fusion_observe_kernel: a leaf
    // seen only through a sliver is updated like any other, so the segments
    // have to be the same ones.  The parts divide the stretch inside the
    // leaves' bounds (widened, so that a ray that misses them meets no leaf).
    Ray r, rb;
    float lo[3], hi[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        lo[c] = a.tree.box_lo[c] - 1e-4f;
        hi[c] = a.tree.box_hi[c] + 1e-4f;
    }
    if (!setup_ray(a.frame[0], a.frame[1], a.frame[2], dir[0], dir[1], dir[2], r) ||
        !setup_ray_in(lo, hi, a.frame[0], a.frame[1], a.frame[2], dir[0], dir[1], dir[2], rb))
        return;
    ListVisitor vis{a, s_chunk[wv], (int)(blockIdx.x * (kBlock / kWave) + wv) % kPools, ln, (py * a.W + px) * PARTS + part, 1.0f, 0.0f, -1, -1};
    NoStop ns;
    const float b0 = rb.t_in - r.t_in;
    const float t0 = part == 0 ? 0.0f : fmaxf(fmaf(rb.t_len, (float)part * (1.0f / PARTS), b0), 0.0f);
    const float t1 = part == PARTS - 1 ? __builtin_inff()
                                       : fmaxf(fmaf(rb.t_len, (float)(part + 1) * (1.0f / PARTS), b0), 0.0f);
    walk<true, kBlock, true>(a.tree, r, s_stack + threadIdx.x, vis, t1, ns, t0);
    vis.flush();
    float Tin = 1.0f;
#pragma unroll
    for (int q = 0; q < PARTS - 1; ++q) {
        const float Tq = __shfl(vis.T, q * kSlots + slot, kWave);
        if (q < part) Tin *= Tq;
    }
    a.Tin[vis.id] = Tin;
}

__global__ __launch_bounds__(kBlock) void fusion_gather_kernel(GatherLaunch a)
{
    const int64_t l = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (l >= a.l.n_leaves || a.l.pool[kPoolInts - 1] != 0) return;
    int n = a.l.head[l];
    float4* A4 = reinterpret_cast<float4*>(a.acc) + l * (FPO_FUSION_ACC / 4);
    const float before = A4[7].y;                     // length from earlier observe calls
    if (n < 0 && !(before > 0.0f)) return;
    float A[FPO_FUSION_ACC];
#pragma unroll
    for (int e = 0; e < FPO_FUSION_ACC; ++e) A[e] = 0.0f;
    const bool had = before != 0.0f;
    if (had) {
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const float4 x = A4[w];
            A[4 * w] = x.x; A[4 * w + 1] = x.y; A[4 * w + 2] = x.z; A[4 * w + 3] = x.w;
        }
    }
    while (n >= 0) {
        const float4 s = a.l.node[n];
        n = a.l.next[n];
        const int id = __float_as_int(s.w);
        const float T = a.l.Tin[id] * s.z;
        if (!(T > a.l.tau)) continue;
        const int pix = id / a.parts;
        float dir[3];
        pixel_dir(a.l.frame, a.l.W, a.l.H, pix % a.l.W, pix / a.l.W, dir);
        Ray r;
        if (!setup_ray(a.l.frame[0], a.l.frame[1], a.l.frame[2], dir[0], dir[1], dir[2], r)) continue;
        const float delta = s.y - s.x;
        const float tm = 0.5f * (s.x + s.y);
        const float x[3] = {fmaf(tm, r.d[0], r.o[0]), fmaf(tm, r.d[1], r.o[1]), fmaf(tm, r.d[2], r.o[2])};
        float col[3], Y[FPO_N_SH];
        field_colour(a.f, x, r.d, col);
        sh9(r.d[0], r.d[1], r.d[2], Y);
        const float w = T * delta;
        A[0] += w;
        A[1] = fmaf(w, field_sigma(a.f, x), A[1]);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int j = 0; j < FPO_N_SH; ++j) A[2 + c * FPO_N_SH + j] = fmaf(w * col[c], Y[j], A[2 + c * FPO_N_SH + j]);
        A[29] += delta;
    }
    if (!(A[29] > 0.0f)) {
        // nothing observed that counts; a length that is not a number stays, as sums would
        if (had)
#pragma unroll
            for (int w = 0; w < 8; ++w) A4[w] = make_float4(A[4 * w], A[4 * w + 1], A[4 * w + 2], A[4 * w + 3]);
        return;
    }
    float V[32];
    float4* V4 = reinterpret_cast<float4*>(const_cast<float*>(a.l.values)) + l * 8;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        const float4 y = V4[w];
        V[4 * w] = y.x; V[4 * w + 1] = y.y; V[4 * w + 2] = y.z; V[4 * w + 3] = y.w;
    }
    update_leaf(A, A[29], V, a.weight[l], a.count[l]);
#pragma unroll
    for (int w = 0; w < 8; ++w) V4[w] = make_float4(V[4 * w], V[4 * w + 1], V[4 * w + 2], V[4 * w + 3]);
    if (had)
#pragma unroll
        for (int w = 0; w < 8; ++w) A4[w] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

}  // namespace dev

// What fpo_fusion_observe checks, and its launch.
static fpo_status fusion_launch(const fpo_tree_view* tree, const float* values, const fpo_camera* cam,
                                const fpo_field* field, float tau, float* acc, dev::FusionLaunch& a)
{
    fpo_status st = check_tree(tree, false, true);
    if (st != FPO_OK) return st;
    if (!values || !acc) return fail(FPO_E_INVALID, "NULL device pointer");
    if (!cam || !field) return fail(FPO_E_INVALID, "NULL camera or field");
    if (!(tau > 0.0f && tau < 1.0f)) return fail(FPO_E_INVALID, "tau must be in (0, 1)");
    if (field->n_gauss < 0 || field->n_gauss > FPO_FIELD_MAX_GAUSS)
        return fail(FPO_E_INVALID, "field n_gauss must be in 0..FPO_FIELD_MAX_GAUSS");
    std::memset(&a, 0, sizeof(a));
    if ((st = camera_frame(*cam, a.frame)) != FPO_OK) return st;
    if ((int64_t)cam->width * cam->height > (1ll << 30)) return fail(FPO_E_INVALID, "image too large");
    for (int g = 0; g < field->n_gauss; ++g) {
        const float w = field->w[g];
        if (!(w > 0.0f) || !std::isfinite(w)) return fail(FPO_E_INVALID, "field widths must be positive");
        for (int c = 0; c < 3; ++c) a.f.mu[g][c] = field->mu[g][c];
        a.f.inv2w2[g] = (float)(1.0 / (2.0 * (double)w * (double)w));
        a.f.a[g] = field->a[g];
    }
    a.f.n = field->n_gauss;
    std::memcpy(a.f.u, field->u, sizeof(a.f.u));
    std::memcpy(a.f.v, field->v, sizeof(a.f.v));
    std::memcpy(a.f.b, field->b, sizeof(a.f.b));
    a.tree = dev::tree_dev(tree);
    a.values = values;
    a.acc = acc;
    a.W = cam->width;
    a.H = cam->height;
    a.bx = (cam->width + 15) / 16;
    a.tau = tau;
    return FPO_OK;
}
}  // namespace fpo

using namespace fpo;

extern "C" fpo_status fpo_fusion_observe(const fpo_tree_view* tree, const float* values, const fpo_camera* cam,
                                         const fpo_field* field, float tau, float* acc, void* stream)
{
    ApiRange api_range_("fpo_fusion_observe");
    dev::FusionLaunch a;
    const fpo_status st = fusion_launch(tree, values, cam, field, tau, acc, a);
    if (st != FPO_OK) return st;
    const int64_t grid = (int64_t)a.bx * ((cam->height + 15) / 16);
    hipLaunchKernelGGL(dev::fusion_observe_kernel, dim3((unsigned)grid), dim3(dev::kBlock), 0,
                       static_cast<hipStream_t>(stream), a);
    return launch_status("fpo_fusion_observe");
}

extern "C" fpo_status fpo_fusion_apply(float* values, float* weight, int32_t* count, float* acc, int64_t n_leaves,
                                       void* stream)
{
    ApiRange api_range_("fpo_fusion_apply");
    if (n_leaves < 0) return fail(FPO_E_INVALID, "n_leaves < 0");
    if (n_leaves == 0) return FPO_OK;
    if (!values || !weight || !count || !acc) return fail(FPO_E_INVALID, "NULL device pointer");
    if (((reinterpret_cast<uintptr_t>(values)) | (reinterpret_cast<uintptr_t>(acc))) & 15)
        return fail(FPO_E_INVALID, "values and acc must be 16-byte aligned");
    if (n_leaves > (int64_t)INT32_MAX * dev::kBlock) return fail(FPO_E_INVALID, "too many leaves");
    const int64_t grid = (n_leaves + dev::kBlock - 1) / dev::kBlock;
    hipLaunchKernelGGL(dev::fusion_apply_kernel, dim3((unsigned)grid), dim3(dev::kBlock), 0,
                       static_cast<hipStream_t>(stream), reinterpret_cast<float4*>(values), weight, count,
                       reinterpret_cast<float4*>(acc), n_leaves, static_cast<const int32_t*>(nullptr));
    return launch_status("fpo_fusion_apply");
}

// Lanes per ray of a view's walk.  With 16, 8 and 1, in us: 300x300 at depth 9
// (800 k leaves) 116 118 528, at depth 7 (60 k) 77 80 250; 800x800 and
// 1000x1000 at depth 9 (2 M) 600 580 1055 and 812 741 1180; 900x900 at depth 7
// (100 k) 655 542 763.
static int fusion_parts(int max_depth, int64_t pixels) { return pixels <= (512ll << max_depth) ? 16 : 8; }

namespace {
// Workspace of fpo_fusion_view: pool counters, list heads, transmittances,
// nodes and their links, each from a 256-byte boundary.
struct ViewLayout {
    int64_t head, Tin, node, next, bytes;
    int32_t cap;
};
int64_t up256(int64_t v) { return (v + 255) / 256 * 256; }
// with room for cap nodes
ViewLayout view_layout(int64_t n_leaves, int64_t lanes, int64_t cap)
{
    ViewLayout v;
    v.cap = (int32_t)cap;
    v.head = up256(dev::kPoolInts * 4);
    v.Tin = up256(v.head + (n_leaves + 3) / 4 * 16);
    v.node = up256(v.Tin + lanes * 4);
    v.next = up256(v.node + cap * 16);
    v.bytes = up256(v.next + cap * 4);
    return v;
}
}  // namespace

extern "C" int64_t fpo_fusion_view_bytes(const fpo_tree_view* tree, const fpo_camera* cam)
{
    if (check_tree(tree, false, true) != FPO_OK || !cam || cam->width < 1 || cam->height < 1) return 0;
    const int64_t px = (int64_t)cam->width * cam->height;
    if (px > (1ll << 26)) return 0;
    const int64_t lanes = px * fusion_parts(tree->max_depth, px);
    // Views of the benchmark's blobs need 9 nodes a pixel at depth 9, 6 at depth
    // 8, 8 and 5 at depth 7, with a third of the pixels meeting the scene and
    // 5 to 8 nodes of every wave's last chunk left over for each of its pixels.
    const int64_t cap = px * ((1ll << tree->max_depth) / 16 + 8) + 2 * dev::kPools * dev::kNodeChunk;
    if (cap > (100ll << 20)) return 0;
    return view_layout(tree->n_leaves, lanes, cap).bytes;
}

extern "C" fpo_status fpo_fusion_view(const fpo_tree_view* tree, float* values, float* weight, int32_t* count,
                                      const fpo_camera* cam, const fpo_field* field, float tau, float* acc,
                                      void* workspace, int64_t workspace_bytes, void* stream)
{
    ApiRange api_range_("fpo_fusion_view");
    dev::FusionLaunch o;
    fpo_status st = fusion_launch(tree, values, cam, field, tau, acc, o);
    if (st != FPO_OK) return st;
    if (!weight || !count) return fail(FPO_E_INVALID, "NULL device pointer");
    if (((reinterpret_cast<uintptr_t>(values)) | (reinterpret_cast<uintptr_t>(acc))) & 15)
        return fail(FPO_E_INVALID, "values and acc must be 16-byte aligned");
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return fail(FPO_E_INVALID, "fpo_fusion_view needs a 256-byte aligned workspace");
    const int64_t px = (int64_t)cam->width * cam->height;
    if (px > (1ll << 26)) return fail(FPO_E_INVALID, "image too large");
    const int parts = fusion_parts(tree->max_depth, px);
    const int64_t lanes = px * parts;
    // as many nodes as fit
    const int64_t fixed = view_layout(tree->n_leaves, lanes, 0).bytes + 1024;
    if (workspace_bytes < fixed) return fail(FPO_E_INVALID, "workspace_bytes below the lists' heads");
    const ViewLayout v = view_layout(tree->n_leaves, lanes, std::min<int64_t>((workspace_bytes - fixed) / 20, INT32_MAX / 2));
    char* base = static_cast<char*>(workspace);
    dev::GatherLaunch g;
    std::memset(&g, 0, sizeof(g));
    dev::ListLaunch& a = g.l;
    a.tree = o.tree;
    a.values = values;
    std::memcpy(a.frame, o.frame, sizeof(a.frame));
    a.W = o.W;
    a.H = o.H;
    a.tau = tau;
    a.pool = reinterpret_cast<int32_t*>(base);
    a.head = reinterpret_cast<int32_t*>(base + v.head);
    a.Tin = reinterpret_cast<float*>(base + v.Tin);
    a.node = reinterpret_cast<float4*>(base + v.node);
    a.next = reinterpret_cast<int32_t*>(base + v.next);
    a.share = v.cap / dev::kPools;
    a.n_leaves = tree->n_leaves;
    g.f = o.f;
    g.weight = weight;
    g.count = count;
    g.acc = acc;
    g.parts = parts;
    const int tw = parts == 8 ? 8 : 4, th = 256 / parts / tw;      // four waves of 64 / parts pixels
    a.bx = (a.W + tw - 1) / tw;
    const int64_t tiles = (int64_t)a.bx * ((a.H + th - 1) / th);
    const int64_t n4 = (tree->n_leaves + 3) / 4;
    const dim3 block(dev::kBlock), leaves((unsigned)((tree->n_leaves + dev::kBlock - 1) / dev::kBlock));
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(dev::fusion_clear_kernel, dim3((unsigned)((std::max<int64_t>(n4, dev::kPoolInts) + dev::kBlock - 1) / dev::kBlock)),
                       block, 0, s, a.pool, reinterpret_cast<int4*>(a.head), n4);
    if (parts == 16) hipLaunchKernelGGL(dev::fusion_list_kernel<16>, dim3((unsigned)tiles), block, 0, s, a);
    else hipLaunchKernelGGL(dev::fusion_list_kernel<8>, dim3((unsigned)tiles), block, 0, s, a);
    if ((st = launch_status("fpo_fusion_view")) != FPO_OK) return st;
    hipLaunchKernelGGL(dev::fusion_gather_kernel, leaves, block, 0, s, g);
    // more segments than nodes: the gather left everything as it was
    o.only_if = a.pool + dev::kPoolInts - 1;
    hipLaunchKernelGGL(dev::fusion_observe_kernel, dim3((unsigned)((int64_t)o.bx * ((o.H + 15) / 16))), block, 0, s, o);
    hipLaunchKernelGGL(dev::fusion_apply_kernel, leaves, block, 0, s, reinterpret_cast<float4*>(values), weight, count,
                       reinterpret_cast<float4*>(acc), tree->n_leaves, static_cast<const int32_t*>(o.only_if));
    return launch_status("fpo_fusion_view");
}
