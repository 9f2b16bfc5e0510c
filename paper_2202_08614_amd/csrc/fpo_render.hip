// libfpo render entry points: camera renders, ray renders, traces, camera
// ray generation and coefficient packing (gfx950).
//
// Work mapping for camera renders: one wave64 renders an 8x8 pixel tile, a
// 256-thread block a 16x16 tile.  Blocks are dispatched round-robin over the
// 8 XCDs of the MI355X (each with its own L2); the block-to-tile map hands the
// XCDs whole rows of tiles in turn (xcd_row), the skip pre-pass a contiguous
// band each.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>

#include "fpo.h"
#include "fpo_device.h"
#include "fpo_internal.h"
#include "fpo_proposal.h"

namespace fpo {
namespace dev {

constexpr int kCamsPerLaunch = 16;
// Camera kernel blocks: cam_waves(mode) waves of 8x8 pixels, over a 16x16
// tile (4 waves, snapshot modes) or one 8x8 tile (1 wave, Fourier modes).
// The Fourier kernels hold 94 or more VGPRs (at most 5 waves per SIMD), and
// one-wave blocks let a finished wave's slot take the next block at once:
// 2.4% (1.9% with two launches in flight) per launch; the snapshot kernel
// (64 VGPRs) was 1.9% slower so.
constexpr int cam_waves(int mode) { return mode >= 16 ? 4 : 1; }
// A wave of `parts` lanes per ray (render_cam_kernel) takes 64 / parts pixels:
// 8x8, 8x4, 4x4, 4x2 or 2x2.
constexpr int wave_tile_w(int parts) { return parts <= 2 ? 8 : parts <= 8 ? 4 : 2; }
constexpr int wave_tile_h(int parts) { return 64 / parts / wave_tile_w(parts); }
constexpr int cam_tile_w(int waves, int parts) { return (waves >= 2 ? 2 : 1) * wave_tile_w(parts); }
constexpr int cam_tile_h(int waves, int parts) { return (waves >= 4 ? 2 : 1) * wave_tile_h(parts); }

struct CamDev {
    float frame[12];                 // eye, forward, right * tan_x, up * tan_y
    float basis[FPO_BASIS_STRIDE];   // Eq. 8 at the camera's time
    const void* snap;                // snapshot planes for this camera (snapshot mode)
};

struct CamLaunch {
    TreeDev tree;
    CamDev cam[kCamsPerLaunch];
    float* rgb;                      // [n_cams][H][W][3] of this launch
    float* Tout;                     // [n_cams][H][W] or null
    const float2* skip;              // skip modes: [n_cams][H][W] (t_start, t_end) from the cube entry
    const uint32_t* bits;            // coarse occupancy (suffix checks)
    int32_t W, H, bx_per_cam, blocks_per_cam, n_cams;
    int32_t cbx_per_cam, crows_per_cam;     // camera kernel tiles (cam_tile_w x cam_tile_h of the mode)
    uint32_t snap_bytes;             // BUF kernels: bytes of one camera's snapshot records
    float bg[3];
    float stop_T;
    // Last: with these two in front of snap_bytes the compiler took 120 instead
    // of 94 registers for the F32 coefficient kernels and up to 140 for the other
    // layouts (4 and 3 waves per SIMD instead of 5).
    int32_t group_rows;              // tile rows per XCD group (xcd_row)
    int32_t mix_cams;                // rows of all cameras in turn (cam_row)
};
static_assert(sizeof(CamLaunch) <= 4096, "kernel argument block too large");

// Skip pre-pass: per pixel, the part of the chord the render has to walk.
struct SkipLaunch {
    float frame[kCamsPerLaunch][12];
    float tau[kCamsPerLaunch];       // t / T mod 1 of each camera
    const uint32_t* bits;
    const unsigned char* packed;     // proposal weights (MLP variant)
    float2* skip;                    // [n_cams][H][W]
    int32_t W, H, bx_per_cam, blocks_per_cam, n_cams;
};

// Block index -> logical tile, giving XCD x (blocks x, x+8, ...) the
// contiguous range [x * per, (x + 1) * per).  gridDim.x is a multiple of 8.
__device__ inline int xcd_band(int bid, int nblocks)
{
    const int per = nblocks >> 3;
    return (bid & 7) * per + (bid >> 3);
}

// Camera kernels: block index -> tile row of the launch, counted in the order
// of cam_row, and column bx.  The rows go out in groups
// of group_rows, eight groups at a time, one per XCD; the XCDs' order turns by
// one from one eight to the next.  render_impl chooses the group.
__device__ inline int xcd_row(int bid, int bx_per_row, int group_rows, int& bx)
{
    const int j = bid >> 3;
    const int r = j / bx_per_row;            // row among this XCD's rows
    bx = j - r * bx_per_row;
    const int k = r / group_rows;
    return (8 * k + (((bid & 7) + k) & 7)) * group_rows + (r - k * group_rows);
}

// Row `row` of the launch, in the order it goes out: camera ci and tile row by;
// false past the last.  Each camera's rows go from its middle outwards (middle,
// one above, one below, ...), or with mix_cams all cameras' middle rows first:
// a wave through the scene takes a fifth of a launch, so these start early and
// the empty rows at the edge fill the time they need at the end.
__device__ inline bool cam_row(int row, const CamLaunch& a, int& ci, int& by)
{
    int i;
    if (a.mix_cams) {
        i = row / a.n_cams;
        ci = row - i * a.n_cams;
        if (i >= a.crows_per_cam) return false;
    } else {
        ci = row / a.crows_per_cam;
        i = row - ci * a.crows_per_cam;
        if (ci >= a.n_cams) return false;
    }
    by = (a.crows_per_cam - 1) / 2 + ((i & 1) ? (i + 1) / 2 : -(i / 2));
    return true;
}

// Skip pre-pass: per pixel, a part of the chord [t_start, t_end] outside
// which the ray provably meets no leaf.  Coarse variant: the first and last
// set coarse cells on the chord (a forward and a backward scan).  Proposal
// variant: the network's entry guess is accepted if the scan up to it is
// clear, else the walk starts at the first set cell that scan met; its exit
// guess is accepted if the backward scan from the cube exit down to it is
// clear, else the walk ends at the exit of the last set cell; a predicted
// miss is checked like the coarse variant (forward scan only).  (inf, inf)
// marks a ray with nothing to walk.
//
// The proposal variant runs in two kernels: proposal_infer_kernel evaluates
// the network (FP16 matrix cores, its fragments in LDS, grid-stride over
// tiles so each block reads the weights once) and leaves each pixel's
// prediction (s_in, s_out as fractions of the chord, s_in < 0 for a predicted
// miss) in the skip buffer; skip_scan_kernel<true> then turns it into the
// proven interval.  The scans are latency-bound and run at the occupancy of a
// small kernel instead of the network's.
struct PixelRay {
    int ci, px, py;
    bool inside;
};

__device__ inline PixelRay pixel_of(const SkipLaunch& a, int lin)
{
    PixelRay p;
    p.ci = lin / a.blocks_per_cam;
    const int tb = lin - p.ci * a.blocks_per_cam;
    const int bx = tb % a.bx_per_cam;
    const int by = tb / a.bx_per_cam;
    const int wv = threadIdx.x >> 6;
    const int ln = threadIdx.x & 63;
    p.px = bx * 16 + (wv & 1) * 8 + (ln & 7);
    p.py = by * 16 + (wv >> 1) * 8 + (ln >> 3);
    p.inside = p.px < a.W && p.py < a.H;
    return p;
}

__device__ inline bool pixel_ray(const SkipLaunch& a, const PixelRay& p, Ray& r)
{
    const float* fr = a.frame[p.ci];
    const float sx = (float)(2 * p.px + 1 - a.W) / (float)a.W;
    const float sy = (float)(a.H - 2 * p.py - 1) / (float)a.H;
    const float dx = fr[3] + sx * fr[6] + sy * fr[9];
    const float dy = fr[4] + sx * fr[7] + sy * fr[10];
    const float dz = fr[5] + sx * fr[8] + sy * fr[11];
    return setup_ray(fr[0], fr[1], fr[2], dx, dy, dz, r) && p.inside;
}

__global__ __launch_bounds__(kBlock) void proposal_infer_kernel(SkipLaunch a)
{
    __shared__ uint2 s_frag[kFrags * 64];
    __shared__ float s_bias[132];
    const uint2* F = reinterpret_cast<const uint2*>(a.packed);
    for (int i = threadIdx.x; i < kFrags * 64; i += kBlock) s_frag[i] = F[i];
    if (threadIdx.x < 132) s_bias[threadIdx.x] = reinterpret_cast<const float*>(a.packed + kPackedBias)[threadIdx.x];
    __syncthreads();
    const int total = a.n_cams * a.blocks_per_cam;
    const int padded = (total + 7) / 8 * 8;
    for (int it = blockIdx.x; it < padded; it += gridDim.x) {
        const int lin = xcd_band(it, padded);
        if (lin >= total) continue;                     // whole blocks: every wave stays complete
        const PixelRay p = pixel_of(a, lin);
        Ray r;
        const bool ok = pixel_ray(a, p, r);
        float x[kMlpIn];
        proposal_inputs(r, a.tau[p.ci], x);
        if (!ok)
            for (int c = 0; c < kMlpIn; ++c) x[c] = 0.0f;
        float o3[3] = {0.0f, 0.0f, 0.0f};
        mlp_infer_wave(s_frag, s_bias, x, o3);          // wave-wide: every lane is active here
        if (p.inside)
            a.skip[((int64_t)p.ci * a.H + p.py) * a.W + p.px] =
                o3[0] > 0.0f ? make_float2(sigmoidf_(o3[1]), sigmoidf_(o3[2])) : make_float2(-1.0f, 0.0f);
    }
}

template <bool PROP>
__global__ __launch_bounds__(kBlock) void skip_scan_kernel(SkipLaunch a)
{
    const int total = a.n_cams * a.blocks_per_cam;
    const int lin = xcd_band(blockIdx.x, gridDim.x);
    if (lin >= total) return;
    const PixelRay p = pixel_of(a, lin);
    if (!p.inside) return;
    Ray r;
    const bool ok = pixel_ray(a, p, r);
    const int64_t pix = ((int64_t)p.ci * a.H + p.py) * a.W + p.px;
    float ts = __builtin_inff(), te = __builtin_inff();
    if (ok) {
        const float len = r.t_len;
        const float2 pred = PROP ? a.skip[pix] : make_float2(-1.0f, 0.0f);
        float pe[3], nd[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            pe[c] = fmaf(len, r.d[c], r.o[c]);
            nd[c] = -r.d[c];
        }
        if (!PROP || pred.x < 0.0f) {
            const float f = coarse_scan(a.bits, r.o, r.d, len);
            if (f < len) {
                ts = f;
                te = PROP ? len : len - coarse_scan(a.bits, pe, nd, len - f);
            }
        } else {
            // entry: accept the guess if the chord up to it is clear; exit:
            // accept the guess if the chord after it is clear, else take the
            // exit of the last set cell
            ts = coarse_scan(a.bits, r.o, r.d, pred.x * len);
            const float span = len - fmaxf(pred.y * len, ts);
            te = span > 0.0f ? len - coarse_scan(a.bits, pe, nd, span) : len;
        }
    }
    a.skip[pix] = make_float2(ts, te);
}

// SKIP: walk only the proven part [t_start, t_end] of each chord that the
// skip pre-pass left in a.skip.  BUF (snapshot modes, records within 4 GiB):
// snapshot reads through a buffer resource, and at most 64 VGPRs.
//
// PARTS > 1: that many lanes share a ray (walk_parts).
template <int MODE, bool SKIP, int N1 = FPO_N_SIGMA, int N2 = FPO_N_SH_FOURIER, bool BUF = false, int PARTS = 1,
          int WAVES = cam_waves(MODE)>
__global__ __launch_bounds__(64 * WAVES, BUF && PARTS == 1 ? 32 / WAVES : 1) void render_cam_kernel(CamLaunch a)
{
    static_assert(!BUF || MODE >= 16, "buffer reads serve snapshot records only");
    static_assert(PARTS == 1 || !SKIP, "the skip modes walk whole rays");
    constexpr int kThreads = 64 * WAVES;
    constexpr int kPix = 64 / PARTS;          // pixels of a wave
    constexpr int kWaveW = wave_tile_w(PARTS);
    constexpr int kWaveH = wave_tile_h(PARTS);
    constexpr int kTileW = cam_tile_w(WAVES, PARTS);
    constexpr int kTileH = cam_tile_h(WAVES, PARTS);
    __shared__ int s_stack[kStackLevels * kThreads];
    int bx, ci, by;
    if (!cam_row(xcd_row(blockIdx.x, a.cbx_per_cam, a.group_rows, bx), a, ci, by)) return;
    const int wv = threadIdx.x >> 6;
    const int ln = threadIdx.x & 63;
    const int part = ln / kPix;               // which part of the chord this lane walks
    const int lp = ln % kPix;
    const int px = bx * kTileW + (wv & 1) * kWaveW + lp % kWaveW;
    const int py = by * kTileH + (wv >> 1) * kWaveH + lp / kWaveW;
    if (px >= a.W || py >= a.H) return;       // all lanes of a pixel together

    const CamDev& cam = a.cam[ci];
    float b[FPO_BASIS_STRIDE];
#pragma unroll
    for (int i = 0; i < FPO_BASIS_STRIDE; ++i) b[i] = cam.basis[i];
    // exact integer numerators: no cancellation near the image centre
    const float sx = (float)(2 * px + 1 - a.W) / (float)a.W;
    const float sy = (float)(a.H - 2 * py - 1) / (float)a.H;
    const float dx = cam.frame[3] + sx * cam.frame[6] + sy * cam.frame[9];
    const float dy = cam.frame[4] + sx * cam.frame[7] + sy * cam.frame[10];
    const float dz = cam.frame[5] + sx * cam.frame[8] + sy * cam.frame[11];

    Shade<MODE, N1, N2, BUF> sh{a.tree, b, cam.snap};
    if constexpr (BUF)
        sh.srs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(cam.snap), (short)0, (int)a.snap_bytes, 0x00020000);
    sh.Tr = 1.0f;
    sh.C[0] = sh.C[1] = sh.C[2] = 0.0f;
    sh.stop_T = a.stop_T;
    Ray r;
    const int64_t pix = ((int64_t)ci * a.H + py) * a.W + px;
    // the plain walk starts on the face of the leaves' bounds (rays that miss
    // them end here); the skip pre-pass measures along the cube's chord
    bool hit;
    if constexpr (SKIP) hit = setup_ray(cam.frame[0], cam.frame[1], cam.frame[2], dx, dy, dz, r);
    else hit = setup_ray_in(a.tree.box_lo, a.tree.box_hi, cam.frame[0], cam.frame[1], cam.frame[2], dx, dy, dz, r);
    if constexpr (PARTS > 1) {
        if (hit) sh9(r.d[0], r.d[1], r.d[2], sh.Y);
        const PartFront f = walk_parts<PARTS, (MODE >= 16), kThreads>(a.tree, r, s_stack + threadIdx.x, sh, hit, part, lp);
        compose_parts<PARTS>(f, sh, part, lp);
        if (part != 0) return;
    } else if (hit) {
        sh9(r.d[0], r.d[1], r.d[2], sh.Y);
        if constexpr (!SKIP) {
            walk<(MODE >= 16), kThreads>(a.tree, r, s_stack + threadIdx.x, sh);
        } else {
            const float2 se = a.skip[pix];
            if (se.x < r.t_len) {
#pragma unroll
                for (int c = 0; c < 3; ++c) r.o[c] = fmaf(se.x, r.d[c], r.o[c]);
                r.t_len -= se.x;
                NoStop ns;
                walk<(MODE >= 16), kThreads>(a.tree, r, s_stack + threadIdx.x, sh, se.y - se.x, ns);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) a.rgb[pix * 3 + c] = fmaf(sh.Tr, a.bg[c], sh.C[c]);
    if (a.Tout) a.Tout[pix] = sh.Tr;
}

// Basis rows of a decode (fpo_render_decoded) from the kernel arguments into
// its workspace: no copy from host memory is enqueued.
constexpr int kDecodeTimes = 16;
struct BasisRows {
    float row[kDecodeTimes * FPO_BASIS_STRIDE];
};
__global__ __launch_bounds__(kBlock) void basis_rows_kernel(BasisRows b, float* out)
{
    for (int i = threadIdx.x; i < kDecodeTimes * FPO_BASIS_STRIDE; i += kBlock) out[i] = b.row[i];
}

struct RaysLaunch {
    TreeDev tree;
    const float* o;
    const float* d;
    const int32_t* t_idx;
    const float* basis;     // [n_t][32]
    const void* snap;
    int64_t snap_stride;    // leaf records between consecutive time indices' snapshots
    int64_t n;
    int32_t n_t;
    float* rgb;
    float* Tout;
    float bg[3];
    float stop_T;
    int32_t* rec_count;     // segment records (render_rays_record_kernel): per-ray count, -1 on overflow
    float4* rec;            // [n][rec_cap] records of 32 bytes
    int32_t rec_cap;
};

// A batch of rays, PARTS lanes each (walk_parts).
template <int MODE, int PARTS>
__global__ __launch_bounds__(kWave) void render_rays_kernel(RaysLaunch a)
{
    constexpr int kSlots = kWave / PARTS;
    __shared__ int s_stack[kStackLevels * kWave];
    const int part = threadIdx.x / kSlots, slot = threadIdx.x % kSlots;
    const int64_t r_id = (int64_t)blockIdx.x * kSlots + slot;
    if (r_id >= a.n) return;                  // all lanes of a ray together
    const int ti = min(max(a.t_idx[r_id], 0), a.n_t - 1);
    float b[FPO_BASIS_STRIDE];
    load_basis(a.basis, ti, b);
    const void* snap = a.snap;
    if constexpr (MODE >= 16) {
        const size_t rec = (MODE - 16) == FPO_F32 ? 128 : 64;
        snap = static_cast<const char*>(a.snap) + (size_t)ti * (size_t)a.snap_stride * rec;
    }
    Shade<MODE> sh{a.tree, b, snap};
    sh.stop_T = a.stop_T;
    sh.restart(1.0f);
    Ray r;
    const bool hit = setup_ray_in(a.tree.box_lo, a.tree.box_hi, a.o[3 * r_id], a.o[3 * r_id + 1], a.o[3 * r_id + 2],
                                  a.d[3 * r_id], a.d[3 * r_id + 1], a.d[3 * r_id + 2], r);
    if (hit) sh9(r.d[0], r.d[1], r.d[2], sh.Y);
    if constexpr (PARTS > 1) {
        const PartFront f = walk_parts<PARTS, true, kWave>(a.tree, r, s_stack + threadIdx.x, sh, hit, part, slot);
        compose_parts<PARTS>(f, sh, part, slot);
        if (part != 0) return;
    } else if (hit) {
        walk<false, kWave>(a.tree, r, s_stack + threadIdx.x, sh);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) a.rgb[r_id * 3 + c] = fmaf(sh.Tr, a.bg[c], sh.C[c]);
    if (a.Tout) a.Tout[r_id] = sh.Tr;
}

// The F32 Fourier-mode batch with each ray's segment records (FPO_RAYS_RECORD,
// collect_records).
template <int PARTS>
__global__ __launch_bounds__(kWave) void render_rays_record_kernel(RaysLaunch a)
{
    constexpr int kSlots = kWave / PARTS;
    __shared__ int s_stack[kStackLevels * kWave];
    __shared__ __align__(16) float4 s_rec[kRecStage];
    const int part = threadIdx.x / kSlots, slot = threadIdx.x % kSlots;
    const int64_t r_id = (int64_t)blockIdx.x * kSlots + slot;
    if (r_id >= a.n) return;                  // all lanes of a ray together
    const int ti = min(max(a.t_idx[r_id], 0), a.n_t - 1);
    float b[FPO_BASIS_STRIDE];
    load_basis(a.basis, ti, b);
    RecShade sh{{a.tree, b, nullptr}};
    Ray r;
    const bool hit = setup_ray_in(a.tree.box_lo, a.tree.box_hi, a.o[3 * r_id], a.o[3 * r_id + 1], a.o[3 * r_id + 2],
                                  a.d[3 * r_id], a.d[3 * r_id + 1], a.d[3 * r_id + 2], r);
    const PartRecords pr = collect_records<PARTS>(a.tree, r, s_stack + threadIdx.x, s_rec + threadIdx.x, sh, hit,
                                                  a.stop_T, part, slot);
    compose_parts<PARTS>(pr.f, sh, part, slot);
    if (part == 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c) a.rgb[r_id * 3 + c] = fmaf(sh.Tr, a.bg[c], sh.C[c]);
        if (a.Tout) a.Tout[r_id] = sh.Tr;
        a.rec_count[r_id] = pr.total <= a.rec_cap ? pr.total : -1;
    }
    if (pr.total > a.rec_cap) return;
    float4* out = a.rec + (r_id * a.rec_cap + pr.first) * 2;
    for (int k0 = 0; k0 < pr.mine; k0 += kLaneRecs) {
        if (k0 > 0) restage<PARTS>(a.tree, r, s_stack + threadIdx.x, sh, pr, part, k0);
        const int m = min(pr.mine - k0, kLaneRecs);
        for (int k = 0; k < m; ++k) {
            float4 x0 = sh.stage[128 * k], x1 = sh.stage[128 * k + 64];
            pr.finish(x0, x1);
            out[2 * (k0 + k)] = x0;
            out[2 * (k0 + k) + 1] = x1;
        }
    }
}

// Records the walk's segments, with distances from the caller's origin.
struct TraceVisitor {
    int32_t* ids;
    float* t01;
    int32_t cap;
    int32_t n;
    float t_in;
    __device__ inline bool segment(int leaf, float t0, float t1)
    {
        if (n < cap) {
            ids[n] = leaf;
            t01[2 * n] = t_in + t0;
            t01[2 * n + 1] = t_in + t1;
        }
        ++n;
        return false;
    }
};

struct TraceLaunch {
    TreeDev tree;
    const float* o;
    const float* d;
    int64_t n;
    int32_t cap;
    int32_t* ids;
    float* t01;
    int32_t* n_visits;
};

__global__ __launch_bounds__(kBlock) void trace_rays_kernel(TraceLaunch a)
{
    __shared__ int s_stack[kStackLevels * kBlock];
    const int64_t r_id = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r_id >= a.n) return;
    TraceVisitor v{a.ids + r_id * a.cap, a.t01 + r_id * a.cap * 2, a.cap, 0, 0.0f};
    Ray r;
    if (setup_ray_in(a.tree.box_lo, a.tree.box_hi, a.o[3 * r_id], a.o[3 * r_id + 1], a.o[3 * r_id + 2],
                  a.d[3 * r_id], a.d[3 * r_id + 1], a.d[3 * r_id + 2], r)) {
        v.t_in = r.t_in;
        walk(a.tree, r, s_stack + threadIdx.x, v);
    }
    a.n_visits[r_id] = v.n;
}

__global__ __launch_bounds__(kBlock) void camera_rays_kernel(const float* table, int32_t n_cams,
                                                             const int32_t* cam, const int32_t* py,
                                                             const int32_t* px, int64_t n, float* o, float* d)
{
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r >= n) return;
    const int ci = min(max(cam[r], 0), n_cams - 1);
    const float* f = table + (int64_t)ci * FPO_CAMERA_FLOATS;
    const int W = (int)f[12], H = (int)f[13];
    const float sx = (float)(2 * px[r] + 1 - W) / (float)W;
    const float sy = (float)(H - 2 * py[r] - 1) / (float)H;
    float v[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) v[a] = f[3 + a] + sx * f[6 + a] + sy * f[9 + a];
    const float inv = 1.0f / sqrtf(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        o[3 * r + a] = f[a];
        d[3 * r + a] = v[a] * inv;
    }
}

// dst word (slot, g) = coefficients 4g .. 4g+3 of leaf perm[slot] (F32
// records of 48 words; padding words and slots >= n_leaves are zero).
__global__ __launch_bounds__(kBlock) void pack_coeffs_kernel(const float* src, const int64_t* perm,
                                                             int64_t n_leaves, int64_t stride, float4* dst,
                                                             int R, int n_coeff)
{
    const int64_t id = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (id >= R * stride) return;
    const int64_t slot = id / R;
    const int g = (int)(id - slot * R);
    float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (slot < n_leaves) {
        const int64_t p = perm[slot];
        if (p >= 0 && p < n_leaves) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int q = 4 * g + e;
                if (q < n_coeff) v[e] = src[p * n_coeff + q];
            }
        }
    }
    dst[id] = make_float4(v[0], v[1], v[2], v[3]);
}

}  // namespace dev

// ---------------------------------------------------------------------------
// host helpers
// ---------------------------------------------------------------------------
using dev::tree_dev;

static int mode_of(const fpo_tree_view* t, const fpo_render_opts* o)
{
    if (o->snapshot) return 16 + (int)o->snapshot_dtype;
    return (int)t->dtype;
}

}  // namespace fpo

using namespace fpo;

// Share of an image inside the rectangle around the projection of the box
// [lo, hi] (the leaves' bounds): 0 where the box is out of view, 1 where it
// reaches the eye's plane.  fr as camera_frame gives it.
static double seen_share(const float fr[12], const float* lo, const float* hi)
{
    double x[2] = {1.0, -1.0}, y[2] = {1.0, -1.0};        // least and greatest, in half images
    int ahead = 0;
    for (int c = 0; c < 8; ++c) {
        double f = 0.0, r = 0.0, u = 0.0, rr = 0.0, uu = 0.0;
        for (int a = 0; a < 3; ++a) {
            const double v = (double)((c >> a) & 1 ? hi[a] : lo[a]) - fr[a];
            f += v * fr[3 + a];
            r += v * fr[6 + a];
            u += v * fr[9 + a];
            rr += (double)fr[6 + a] * fr[6 + a];
            uu += (double)fr[9 + a] * fr[9 + a];
        }
        if (f < 1e-3) continue;
        ++ahead;
        x[0] = std::min(x[0], r / (rr * f));
        x[1] = std::max(x[1], r / (rr * f));
        y[0] = std::min(y[0], u / (uu * f));
        y[1] = std::max(y[1], u / (uu * f));
    }
    if (ahead == 0) return 0.0;
    if (ahead < 8) return 1.0;
    const double w = std::min(x[1], 1.0) - std::max(x[0], -1.0), h = std::min(y[1], 1.0) - std::max(y[0], -1.0);
    return w > 0.0 && h > 0.0 ? 0.25 * w * h : 0.0;
}

// Pixels of a launch: all, and those that see the leaves' bounds, from outside
// the box of twice their size and from inside it.
struct LaunchPixels {
    double all, far, near;
};

static void count_view(LaunchPixels& n, const float fr[12], double pixels, const float* lo, const float* hi)
{
    bool near = true;
    for (int a = 0; a < 3; ++a) near = near && std::fabs(fr[a] - 0.5f * (lo[a] + hi[a])) <= hi[a] - lo[a];
    n.all += pixels;
    (near ? n.near : n.far) += pixels * seen_share(fr, lo, hi);
}

// Lanes per ray of a camera launch.  Parts shorten the longest rays, which a
// launch that does not fill the machine waits for, but cost work: a part's lanes
// idle where their stretch is empty, and the parts behind a ray's end are walked
// for nothing.  So they pay while few pixels see the scene, fewer from nearby or
// inside, where rays end early, and the longer the rays, in lattice cells, the
// more: the limits double per level.  us at depth 7 (60 k leaves) / 9 (2 M), one
// lane against 8 or 16, 40 degrees of view from 1.6, 0.8 and 0.15 cubes off the
// middle:
//   F32 snapshot 200x200   144 / 773 -> 39 / 133 (16), 130 / 696 -> 51 / 138 (16),
//                           87 / 444 -> 79 / 254 (16)
//     400x400              136 / 688 -> 66 / 149 (8, 16), 121 / 658 -> 91 / 241
//                          (8, 16), 87 / 461 -> 167 / 642 (8: not taken)
//     1920x1080            - / 690 -> 421 (8), - / 715 -> 1058 (8: not taken), - /
//                          1516 -> 4847 (8: not taken)
//   F32 coefficients 400x400  203 / 1020 -> 84 / 311 (16), 204 / 1078 -> 211 / 604
//                          (16, at depth 7 not taken), 159 / 852 -> 503 / 1694 (not taken)
//   BF16 200x200           181 / 823 -> 57 / 180 (16), 171 / 932 -> 95 / 270 (16),
//                          122 / 620 -> 171 / 659 (not taken)
//   FP8 200x200            293 / 1135 -> 81 / 239 (16), 276 / 1134 -> 123 / 299
//                          (16), 191 / 873 -> 251 / 808 (at depth 7 not taken)
static int ray_parts(int mode, int max_depth, const LaunchPixels& n)
{
    const auto within = [&](double all, double far, double near) {
        const double scale = std::ldexp(1.0, -max_depth);
        return n.all * scale <= all && n.far * scale / far + n.near * scale / near <= 1.0;
    };
    if (n.far + n.near == 0.0) return 1;                 // nothing to walk
    if (mode >= 16) return within(512, 512, 128) ? 16 : within(4096, 1024, 256) ? 8 : 1;
    if (mode == FPO_F32) return within(1536, 512, 160) ? 16 : 1;
    return within(1024, 300, mode == FPO_BF16 ? 64 : 96) ? 16 : 1;
}

template <int MODE, bool BUF = false>
static void launch_cam(const dev::CamLaunch& a, int grid, int skip, int parts, hipStream_t s)
{
    switch (parts) {              // 1 with a skip mode
#define FPO_PARTS(P) case P:                                                                                    \
        hipLaunchKernelGGL((dev::render_cam_kernel<MODE, false, FPO_N_SIGMA, FPO_N_SH_FOURIER, BUF, P>),         \
                           dim3(grid), dim3(64 * dev::cam_waves(MODE)), 0, s, a); return
        FPO_PARTS(8); FPO_PARTS(16);
#undef FPO_PARTS
        default: break;
    }
    if (skip != 0)
        hipLaunchKernelGGL((dev::render_cam_kernel<MODE, true, FPO_N_SIGMA, FPO_N_SH_FOURIER, BUF>), dim3(grid),
                           dim3(64 * dev::cam_waves(MODE)), 0, s, a);
    else
        hipLaunchKernelGGL((dev::render_cam_kernel<MODE, false, FPO_N_SIGMA, FPO_N_SH_FOURIER, BUF>), dim3(grid),
                           dim3(64 * dev::cam_waves(MODE)), 0, s, a);
}

// Fourier-mode render of another coefficient layout (n1, n2) = key / 100,
// key % 100 from a store of DT; false if the layout is not compiled.
template <int DT>
static bool launch_layout(const dev::CamLaunch& a, int key, int grid, hipStream_t s)
{
    switch (key) {
#define FPO_LAY(A, B) case A * 100 + B: \
        hipLaunchKernelGGL((dev::render_cam_kernel<DT, false, A, B>), dim3(grid), dim3(64 * dev::cam_waves(DT)), 0, s, a); return true
        FPO_LAY(11, 5); FPO_LAY(21, 5); FPO_LAY(11, 11); FPO_LAY(21, 11); FPO_LAY(31, 11);
#undef FPO_LAY
        default: return false;
    }
}

// The body of fpo_render: cameras go out in launches of at most
// cams_per_launch (<= 16); the skip modes' scratch (opts->workspace) holds
// one launch's pixels and is reused by every launch of the call.  snap_index:
// which of the snapshots each camera reads (null: its own).
static fpo_status render_impl(const fpo_tree_view* tree, const fpo_camera* cams, int32_t n_cams,
                              const fpo_render_opts* opts, float* rgb_out, float* T_out, void* stream,
                              int cams_per_launch, const int32_t* snap_index = nullptr)
{
    fpo_status st = check_tree(tree, opts == nullptr || opts->snapshot == nullptr, true);
    if (st != FPO_OK) return st;
    if ((st = check_opts(opts, tree, true)) != FPO_OK) return st;
    // the snapshot render does not read coefficients, so any compiled layout goes
    const bool variant = !default_layout(tree->layout) && !opts->snapshot;
    if (variant && opts->flags != 0)
        return fail(FPO_E_UNSUPPORTED, "layouts other than (31, 5) render without skipping only");
    if (!cams || n_cams < 1) return fail(FPO_E_INVALID, "cams is NULL or n_cams < 1");
    if (!rgb_out) return fail(FPO_E_INVALID, "rgb_out is NULL");
    const int W = cams[0].width, H = cams[0].height;
    for (int i = 0; i < n_cams; ++i)
        if (cams[i].width != W || cams[i].height != H)
            return fail(FPO_E_INVALID, "all cameras of one call must share width and height");
    if ((int64_t)W * H > (1ll << 30)) return fail(FPO_E_INVALID, "image too large");
    const int skip = force_fallback() ? 0 : opts->flags;     // FPO_FORCE_FALLBACK=1: plain traversal
    const int per_launch = std::max(1, std::min(cams_per_launch, dev::kCamsPerLaunch));
    if (skip != 0) {
        const int64_t need = (int64_t)std::min(n_cams, per_launch) * W * H * 8;
        if (opts->workspace_bytes < need)
            return fail(FPO_E_INVALID, "opts->workspace_bytes < min(n_cams, 16) * W * H * 8");
    }
    // Validate every camera before launching anything.
    static thread_local dev::CamLaunch a;
    static thread_local dev::SkipLaunch sk;
    std::memset(&a, 0, sizeof(a));
    a.tree = tree_dev(tree);
    LaunchPixels seen{0.0, 0.0, 0.0};
    for (int i = 0; i < n_cams; ++i) {
        float fr[12];
        if ((st = camera_frame(cams[i], fr)) != FPO_OK) return st;
        if (i < per_launch) count_view(seen, fr, (double)W * H, a.tree.box_lo, a.tree.box_hi);
    }
    a.W = W;
    a.H = H;
    a.bx_per_cam = (W + 15) / 16;
    a.blocks_per_cam = a.bx_per_cam * ((H + 15) / 16);
    for (int c = 0; c < 3; ++c) a.bg[c] = opts->bg[c];
    a.stop_T = opts->stop_T;
    const int mode = mode_of(tree, opts);
    const int parts = variant || skip ? 1 : ray_parts(mode, tree->max_depth, seen);   // by the first launch
    {
        const int waves = variant ? dev::cam_waves(tree->dtype) : dev::cam_waves(mode);
        const int tw = dev::cam_tile_w(waves, parts), th = dev::cam_tile_h(waves, parts);
        a.cbx_per_cam = (W + tw - 1) / tw;
        a.crows_per_cam = (H + th - 1) / th;
    }
    const size_t snap_rec = opts->snapshot_dtype == FPO_F32 ? 128 : 64;   // bytes per leaf record
    // snapshot records within 4 GiB per camera are read with 32-bit offsets
    const bool snap_buf = opts->snapshot && (uint64_t)tree->n_leaves * snap_rec <= 0xFFFFFFFFull;
    a.snap_bytes = snap_buf ? (uint32_t)((uint64_t)tree->n_leaves * snap_rec) : 0u;
    hipStream_t s = static_cast<hipStream_t>(stream);
    for (int c0 = 0; c0 < n_cams; c0 += per_launch) {
        const int nc = std::min(per_launch, n_cams - c0);
        a.n_cams = nc;
        for (int i = 0; i < nc; ++i) {
            const fpo_camera& cam = cams[c0 + i];
            camera_frame(cam, a.cam[i].frame);
            basis_row(cam.time, (double)tree->layout.period, tree->layout.n_sigma, a.cam[i].basis);
            a.cam[i].snap = opts->snapshot
                ? static_cast<const char*>(opts->snapshot) +
                      (size_t)(snap_index ? snap_index[c0 + i] : c0 + i) * (size_t)opts->snapshot_cam_stride * snap_rec
                : nullptr;
        }
        a.rgb = rgb_out + (int64_t)c0 * W * H * 3;
        a.Tout = T_out ? T_out + (int64_t)c0 * W * H : nullptr;
        const int64_t total = (int64_t)nc * a.blocks_per_cam;
        const int64_t crows = (int64_t)nc * a.crows_per_cam;
        // Which tiles an XCD takes.  Where the cameras read the same records,
        // single rows in turn, all cameras' middle rows first.  Cameras with
        // records of their own go one after another, a multiple of 8 as bands of
        // rows (whole cameras per XCD), others in single rows.  2 M leaves at
        // 1080p, bands of rows / single rows in order / as chosen: 16 cameras of
        // one pruned snapshot (ten launches and their bake) 29.9 / 30.2 / 28.4 ms,
        // 12 cameras - / 2.52 / 2.24 ms a launch, four 1.00 / 1.03 / 0.88, one
        // 0.79 / 0.60 / 0.60; 16 cameras of 16 snapshots with their decode 4.84 /
        // 4.97 / 4.80 ms, five (500x500, depth 8) - / 0.52 / 0.50.  Bands leave the
        // rows through the scene's middle to a few XCDs and the longest rays to
        // the end; views from near, whose rows are all alike, gain from neighbours
        // in one L2 (800x800 inside the 2 M leaves 730 us in rows, 705 in bands).
        a.mix_cams = 1;
        for (int i = 1; i < nc; ++i) a.mix_cams = a.mix_cams && a.cam[i].snap == a.cam[0].snap;
        const bool bands = (!a.mix_cams && nc % 8 == 0) || seen.near > seen.far;
        a.group_rows = bands ? (int)((crows + 7) / 8) : 1;
        const int64_t groups = (crows + a.group_rows - 1) / a.group_rows;
        const int64_t ctotal = (groups + 7) / 8 * 8 * a.group_rows * a.cbx_per_cam;
        if (ctotal > INT32_MAX - 8) return fail(FPO_E_INVALID, "launch too large");
        const int grid = (int)((total + 7) / 8 * 8);           // skip pre-pass: 16x16 tiles
        const int cam_grid = (int)ctotal;                       // camera kernel tiles
        if (skip != 0) {
            sk.n_cams = nc;
            sk.W = W;
            sk.H = H;
            sk.bx_per_cam = a.bx_per_cam;
            sk.blocks_per_cam = a.blocks_per_cam;
            for (int i = 0; i < nc; ++i) {
                for (int q = 0; q < 12; ++q) sk.frame[i][q] = a.cam[i].frame[q];
                const double per = (double)tree->layout.period;
                double tau = std::fmod(cams[c0 + i].time / per, 1.0);
                if (tau < 0.0) tau += 1.0;
                sk.tau[i] = (float)tau;
            }
            sk.bits = opts->coarse_bits;
            sk.packed = static_cast<const unsigned char*>(opts->proposal);
            sk.skip = static_cast<float2*>(opts->workspace);
            a.skip = sk.skip;
            a.bits = opts->coarse_bits;
            if (skip == FPO_RENDER_SKIP_PROPOSAL) {
                hipLaunchKernelGGL(dev::proposal_infer_kernel, dim3(std::min(grid, 1024)), dim3(dev::kBlock), 0, s, sk);
                hipLaunchKernelGGL(dev::skip_scan_kernel<true>, dim3(grid), dim3(dev::kBlock), 0, s, sk);
            } else {
                hipLaunchKernelGGL(dev::skip_scan_kernel<false>, dim3(grid), dim3(dev::kBlock), 0, s, sk);
            }
            if ((st = launch_status("fpo_render (skip pre-pass)")) != FPO_OK) return st;
        }
        if (variant) {
            const int key = tree->layout.n_sigma * 100 + tree->layout.n_sh_fourier;
            bool ok = false;
            switch (tree->dtype) {
                case FPO_F32: ok = launch_layout<FPO_F32>(a, key, cam_grid, s); break;
                case FPO_BF16: ok = launch_layout<FPO_BF16>(a, key, cam_grid, s); break;
                default: ok = launch_layout<FPO_FP8_E4M3>(a, key, cam_grid, s); break;
            }
            if (!ok) return fail(FPO_E_UNSUPPORTED, "layout (n1, n2) not compiled");
            if ((st = launch_status("fpo_render")) != FPO_OK) return st;
            continue;
        }
        switch (mode) {
            case FPO_F32: launch_cam<FPO_F32>(a, cam_grid, skip, parts, s); break;
            case FPO_BF16: launch_cam<FPO_BF16>(a, cam_grid, skip, parts, s); break;
            case FPO_FP8_E4M3: launch_cam<FPO_FP8_E4M3>(a, cam_grid, skip, parts, s); break;
            case dev::kSnapF32:
                if (snap_buf) launch_cam<dev::kSnapF32, true>(a, cam_grid, skip, parts, s);
                else launch_cam<dev::kSnapF32>(a, cam_grid, skip, parts, s);
                break;
            case dev::kSnapBF16:
                if (snap_buf) launch_cam<dev::kSnapBF16, true>(a, cam_grid, skip, parts, s);
                else launch_cam<dev::kSnapBF16>(a, cam_grid, skip, parts, s);
                break;
            default: return fail(FPO_E_INVALID, "unknown render mode");
        }
        if ((st = launch_status("fpo_render")) != FPO_OK) return st;
    }
    return FPO_OK;
}

extern "C" fpo_status fpo_render(const fpo_tree_view* tree, const fpo_camera* cams, int32_t n_cams,
                                 const fpo_render_opts* opts, float* rgb_out, float* T_out, void* stream)
{
    ApiRange api_range_("fpo_render");
    return render_impl(tree, cams, n_cams, opts, rgb_out, T_out, stream, dev::kCamsPerLaunch);
}

// ---------------------------------------------------------------------------
// fpo_render_decoded: evaluate every leaf at the cameras' times first
// (fpo_bake_times into F32 records), then render those.
//
// A Fourier-mode ray reads 128 (transparent) to 672 bytes of coefficients and
// spends 64 to 409 flop per segment; the decoded record is one 128-byte line
// and 2 to 77 flop, and costs one pass over the store.
// ---------------------------------------------------------------------------
namespace fpo {
constexpr int64_t kDecodeHead = (int64_t)dev::kDecodeTimes * FPO_BASIS_STRIDE * sizeof(float);
constexpr int64_t kDecodeMaxBytes = 4ll << 30;

// The cameras from c0 on whose distinct times (in times[], at most max_t) fit
// one decode; returns the camera after them.
static int decode_group(const fpo_camera* cams, int c0, int n_cams, int max_t, double* times, int& n_t)
{
    n_t = 0;
    int c = c0;
    for (; c < n_cams; ++c) {
        int j = 0;
        while (j < n_t && times[j] != cams[c].time) ++j;
        if (j == n_t) {
            if (n_t == max_t) break;
            times[n_t++] = cams[c].time;
        }
    }
    return c;
}
}  // namespace fpo

extern "C" int64_t fpo_render_decode_bytes(const fpo_tree_view* tree, const fpo_camera* cams, int32_t n_cams,
                                           const fpo_render_opts* opts)
{
    if (check_tree(tree, true) != FPO_OK || check_opts(opts, tree, true) != FPO_OK) return 0;
    if (opts->snapshot || opts->flags != 0 || !cams || n_cams < 1) return 0;
    const dev::TreeDev td = dev::tree_dev(tree);
    double px = 0.0;              // of the images that the leaves' bounds are in
    for (int i = 0; i < n_cams; ++i) {
        float fr[12];
        if (cams[i].width != cams[0].width || cams[i].height != cams[0].height || camera_frame(cams[i], fr) != FPO_OK)
            return 0;
        if (seen_share(fr, td.box_lo, td.box_hi) > 0.0) px += (double)cams[i].width * cams[i].height;
    }
    const int64_t rec = tree->n_leaves * 128;
    if ((kDecodeMaxBytes - kDecodeHead) / rec < 1) return 0;
    const int cap = (int)std::min<int64_t>((kDecodeMaxBytes - kDecodeHead) / rec, dev::kDecodeTimes);
    int groups = 0, most = 0;
    int64_t decoded = 0;
    for (int c0 = 0; c0 < n_cams; ++groups) {
        double times[dev::kDecodeTimes];
        int n_t;
        c0 = decode_group(cams, c0, n_cams, cap, times, n_t);
        decoded += n_t;
        most = std::max(most, n_t);
    }
    // Where decoding pays, in us.  A decode streams the store and its records
    // at 5 TB/s, plus two launches.  What it saves at 2 M leaves of depth 9:
    // 9.4 ms for 16 views of 1920x1080 (33 Mpixel; 12.6 ms from F32
    // coefficients, 3.2 ms from decoded records), 930 us for one, 640 us at
    // 800x800, 290 us at 400x400; at depth 8 (300 k leaves) 240 us at 800x800,
    // at depth 7 (60 k leaves) 130 us at 800x800 and 67 us at 400x400.  A view
    // that the scene is not in is rendered in 20 us either way.
    const double saved = std::ldexp(2.85e-4 * px + 4e-4 * std::min(px, 1048576.0), tree->max_depth - 9);
    const double bytes = (double)tree->n_leaves * 16 * record_words(tree->dtype, FPO_N_SIGMA, FPO_N_SH_FOURIER) * groups +
                         (double)rec * decoded;
    if (saved <= bytes / 5e6 + 12.0 * groups) return 0;
    return kDecodeHead + most * rec;
}

extern "C" fpo_status fpo_render_decoded(const fpo_tree_view* tree, const fpo_camera* cams, int32_t n_cams,
                                         const fpo_render_opts* opts, float* rgb_out, float* T_out, void* workspace,
                                         int64_t workspace_bytes, void* stream)
{
    ApiRange api_range_("fpo_render_decoded");
    fpo_status st = check_tree(tree, true);
    if (st != FPO_OK) return st;
    if ((st = check_opts(opts, tree, true)) != FPO_OK) return st;
    if (opts->snapshot || opts->flags != 0)
        return fail(FPO_E_UNSUPPORTED, "fpo_render_decoded renders coefficients without skipping");
    if (!cams || n_cams < 1) return fail(FPO_E_INVALID, "cams is NULL or n_cams < 1");
    if (!rgb_out) return fail(FPO_E_INVALID, "rgb_out is NULL");
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 127) != 0)
        return fail(FPO_E_INVALID, "fpo_render_decoded needs a 128-byte aligned workspace");
    const int64_t rec = tree->n_leaves * 128;
    const int cap = (int)std::min<int64_t>((workspace_bytes - kDecodeHead) / rec, dev::kDecodeTimes);
    if (workspace_bytes < kDecodeHead || cap < 1)
        return fail(FPO_E_INVALID, "workspace_bytes below the basis rows and one time's records");
    const int W = cams[0].width, H = cams[0].height;
    if ((int64_t)W * H > (1ll << 30)) return fail(FPO_E_INVALID, "image too large");
    for (int i = 0; i < n_cams; ++i) {
        float fr[12];
        if (cams[i].width != W || cams[i].height != H)
            return fail(FPO_E_INVALID, "all cameras of one call must share width and height");
        if ((st = camera_frame(cams[i], fr)) != FPO_OK) return st;
    }
    float* basis = static_cast<float*>(workspace);
    char* recs = static_cast<char*>(workspace) + kDecodeHead;
    fpo_tree_view view = *tree;
    view.leaf_stride = tree->n_leaves;
    fpo_render_opts o = *opts;
    o.snapshot = recs;
    o.snapshot_dtype = FPO_F32;
    o.snapshot_cam_stride = tree->n_leaves;
    o.workspace = nullptr;
    o.workspace_bytes = 0;
    hipStream_t s = static_cast<hipStream_t>(stream);
    for (int c0 = 0; c0 < n_cams;) {
        double times[dev::kDecodeTimes];
        int n_t;
        const int end = decode_group(cams, c0, n_cams, cap, times, n_t);
        dev::BasisRows rows;
        std::memset(&rows, 0, sizeof(rows));
        for (int j = 0; j < n_t; ++j)
            basis_row(times[j], (double)tree->layout.period, tree->layout.n_sigma, rows.row + j * FPO_BASIS_STRIDE);
        hipLaunchKernelGGL(dev::basis_rows_kernel, dim3(1), dim3(dev::kBlock), 0, s, rows, basis);
        if ((st = launch_status("fpo_render_decoded")) != FPO_OK) return st;
        if ((st = fpo_bake_times(&view, basis, n_t, FPO_F32, recs, nullptr, stream)) != FPO_OK) return st;
        // 16 cameras of the group at a time, each with its time's records
        for (int a = c0; a < end; a += dev::kCamsPerLaunch) {
            const int n = std::min(end - a, dev::kCamsPerLaunch);
            int32_t index[dev::kCamsPerLaunch];
            for (int i = 0; i < n; ++i) {
                int j = 0;
                while (times[j] != cams[a + i].time) ++j;
                index[i] = j;
            }
            st = render_impl(&view, cams + a, n, &o, rgb_out + (int64_t)a * W * H * 3,
                             T_out ? T_out + (int64_t)a * W * H : nullptr, stream, dev::kCamsPerLaunch, index);
            if (st != FPO_OK) return st;
        }
        c0 = end;
    }
    return FPO_OK;
}

// ---------------------------------------------------------------------------
// fpo_render_noalloc: fpo_render whose skip-mode scratch is a file-scope
// device array instead of a caller workspace.  Each device that loads the
// library holds its own copy (kNoallocScratchBytes) until the process ends.
// Host code never passes the array's name to a kernel: its device address
// comes from hipGetSymbolAddress, once per device, with that device current.
// ---------------------------------------------------------------------------
namespace fpo {
namespace dev {
constexpr int64_t kNoallocScratchBytes = FPO_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];
}  // namespace dev

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices];

// Device address of `scratch` on the current device (looked up on the first
// call from that device).
static fpo_status scratch_address(void** out)
{
    int d = -1;
    if (hipGetDevice(&d) != hipSuccess || d < 0 || d >= kMaxDevices)
        return fail(FPO_E_DEVICE, "fpo_render_noalloc: no current HIP device");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[d]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(dev::scratch));
        if (e != hipSuccess || !p)
            return fail(FPO_E_DEVICE, std::string("fpo_render_noalloc: hipGetSymbolAddress failed: ") +
                                          hipGetErrorString(e));
        g_scratch_ptr[d] = p;
    }
    *out = g_scratch_ptr[d];
    return FPO_OK;
}
}  // namespace fpo

extern "C" fpo_status fpo_render_noalloc(const fpo_tree_view* tree, const fpo_camera* cams, int32_t n_cams,
                                         const fpo_render_opts* opts, float* rgb_out, float* T_out, void* stream)
{
    ApiRange api_range_("fpo_render_noalloc");
    // every host-side check before the device is touched
    fpo_status st = check_tree(tree, opts == nullptr || opts->snapshot == nullptr, true);
    if (st != FPO_OK) return st;
    if ((st = check_opts(opts, tree, true, false, false)) != FPO_OK) return st;
    if (opts->flags == 0) return render_impl(tree, cams, n_cams, opts, rgb_out, T_out, stream, dev::kCamsPerLaunch);
    if (!cams || n_cams < 1) return fail(FPO_E_INVALID, "cams is NULL or n_cams < 1");
    const int64_t per_cam = (int64_t)cams[0].width * cams[0].height * 8;
    if (cams[0].width < 1 || cams[0].height < 1) return fail(FPO_E_INVALID, "bad image size");
    if (per_cam > FPO_NOALLOC_SCRATCH_BYTES)
        return fail(FPO_E_CAPACITY, "fpo_render_noalloc: one camera's skip scratch (8 W H bytes) exceeds "
                                    "FPO_NOALLOC_SCRATCH_BYTES; use fpo_render with a workspace");
    void* ptr = nullptr;
    if ((st = scratch_address(&ptr)) != FPO_OK) return st;
    fpo_render_opts o = *opts;
    o.workspace = ptr;
    o.workspace_bytes = FPO_NOALLOC_SCRATCH_BYTES;
    const int per_launch = (int)std::min<int64_t>(dev::kCamsPerLaunch, FPO_NOALLOC_SCRATCH_BYTES / per_cam);
    return render_impl(tree, cams, n_cams, &o, rgb_out, T_out, stream, per_launch);
}

// Lanes per ray of a batch of n rays (see ray_parts; batch rays seldom miss the
// scene, and share no leaves).  us for 32, 16 and 1 lanes, rays from outside
// through the middle, at depths 7 (60 k leaves) / 9 (2 M): F32 coefficients 4000
// rays 39 55 203 / 89 151 703, 16,000 rays 108 103 197 / 229 286 796, 64,000
// rays 364 330 266 / 775 880 1051, 128,000 rays 707 626 331 / 1490 1677 1271;
// BF16 64,000 rays 338 296 242 / 708 758 953, 128,000 rays 654 547 270 / 1364
// 1419 1016; F32 snapshots 16,000 rays 63 46 127 / 115 124 522, 64,000 rays 192
// 121 155 / 341 277 612, 128,000 rays 363 212 175 / 640 481 649, 256,000 rays
// 713 396 217 / 1241 890 727.
static int batch_parts(int mode, int max_depth, int64_t n)
{
    if (mode == FPO_F32 && n <= FPO_RECORD_MAX_RAYS) return record_parts(max_depth, n);
    if (n <= (64ll << max_depth)) return 32;
    return n <= (mode >= 16 ? std::min<int64_t>(320ll << max_depth, 163840) : std::min<int64_t>(200ll << max_depth, 81920))
               ? 16 : 1;
}

template <int MODE>
static void launch_rays(const dev::RaysLaunch& a, int parts, hipStream_t s)
{
    const dim3 grid((unsigned)((a.n * parts + dev::kWave - 1) / dev::kWave)), block(dev::kWave);
    if (parts == 32) hipLaunchKernelGGL((dev::render_rays_kernel<MODE, 32>), grid, block, 0, s, a);
    else if (parts == 16) hipLaunchKernelGGL((dev::render_rays_kernel<MODE, 16>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((dev::render_rays_kernel<MODE, 1>), grid, block, 0, s, a);
}

extern "C" fpo_status fpo_render_rays(const fpo_tree_view* tree, const float* o, const float* d,
                                      const int32_t* t_idx, const float* basis, int32_t n_t, int64_t n_rays,
                                      const fpo_render_opts* opts, float* rgb_out, float* T_out, void* stream)
{
    ApiRange api_range_("fpo_render_rays");
    fpo_status st = check_tree(tree, opts == nullptr || opts->snapshot == nullptr);
    if (st != FPO_OK) return st;
    const bool record = opts && opts->flags == FPO_RAYS_RECORD;
    if ((st = check_opts(opts, tree, false, true)) != FPO_OK) return st;
    if (n_rays < 0) return fail(FPO_E_INVALID, "n_rays < 0");
    if (n_rays == 0) return FPO_OK;
    RecordLayout rl;
    if (record) {
        if (mode_of(tree, opts) != FPO_F32 || n_rays > FPO_RECORD_MAX_RAYS)
            return fail(FPO_E_UNSUPPORTED, "FPO_RAYS_RECORD needs F32 Fourier mode and at most 32768 rays");
        if ((st = record_layout(opts, n_rays, rl)) != FPO_OK) return st;
    }
    if (!o || !d || !t_idx || !basis || !rgb_out) return fail(FPO_E_INVALID, "NULL device pointer");
    if (n_t < 1) return fail(FPO_E_INVALID, "n_t must be >= 1");
    if (n_rays > (int64_t)INT32_MAX * dev::kBlock) return fail(FPO_E_INVALID, "too many rays");
    dev::RaysLaunch a;
    std::memset(&a, 0, sizeof(a));
    a.tree = tree_dev(tree);
    a.o = o; a.d = d; a.t_idx = t_idx; a.basis = basis; a.n_t = n_t; a.n = n_rays;
    a.snap = opts->snapshot;
    a.snap_stride = opts->snapshot_cam_stride;
    a.rgb = rgb_out; a.Tout = T_out;
    for (int c = 0; c < 3; ++c) a.bg[c] = opts->bg[c];
    a.stop_T = opts->stop_T;
    if (record) {
        a.rec_count = rl.count;
        a.rec = reinterpret_cast<float4*>(rl.records);
        a.rec_cap = rl.cap;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int mode = mode_of(tree, opts);
    const int parts = batch_parts(mode, tree->max_depth, n_rays);
    if (record) {
        const dim3 grid((unsigned)((n_rays * parts + dev::kWave - 1) / dev::kWave)), block(dev::kWave);
        if (parts == 32) hipLaunchKernelGGL(dev::render_rays_record_kernel<32>, grid, block, 0, s, a);
        else hipLaunchKernelGGL(dev::render_rays_record_kernel<16>, grid, block, 0, s, a);
        return launch_status("fpo_render_rays");
    }
    switch (mode) {
        case FPO_F32: launch_rays<FPO_F32>(a, parts, s); break;
        case FPO_BF16: launch_rays<FPO_BF16>(a, parts, s); break;
        case FPO_FP8_E4M3: launch_rays<FPO_FP8_E4M3>(a, parts, s); break;
        case dev::kSnapF32: launch_rays<dev::kSnapF32>(a, parts, s); break;
        case dev::kSnapBF16: launch_rays<dev::kSnapBF16>(a, parts, s); break;
        default: return fail(FPO_E_INVALID, "unknown render mode");
    }
    return launch_status("fpo_render_rays");
}

extern "C" fpo_status fpo_trace_rays(const fpo_tree_view* tree, const float* o, const float* d, int64_t n_rays,
                                     int32_t max_visits, int32_t* leaf_ids, float* t01, int32_t* n_visits,
                                     void* stream)
{
    ApiRange api_range_("fpo_trace_rays");
    fpo_status st = check_tree(tree, false);
    if (st != FPO_OK) return st;
    if (n_rays < 0 || max_visits < 0) return fail(FPO_E_INVALID, "negative size");
    if (n_rays == 0) return FPO_OK;
    if (!o || !d || !n_visits || (max_visits > 0 && (!leaf_ids || !t01)))
        return fail(FPO_E_INVALID, "NULL device pointer");
    if (n_rays > (int64_t)INT32_MAX * dev::kBlock) return fail(FPO_E_INVALID, "too many rays");
    dev::TraceLaunch a;
    a.tree = tree_dev(tree);
    a.o = o; a.d = d; a.n = n_rays; a.cap = max_visits; a.ids = leaf_ids; a.t01 = t01; a.n_visits = n_visits;
    const int64_t grid = (n_rays + dev::kBlock - 1) / dev::kBlock;
    hipLaunchKernelGGL(dev::trace_rays_kernel, dim3((unsigned)grid), dim3(dev::kBlock), 0,
                       static_cast<hipStream_t>(stream), a);
    return launch_status("fpo_trace_rays");
}

extern "C" fpo_status fpo_camera_rays(const float* cam_table, int32_t n_cams, const int32_t* cam,
                                      const int32_t* py, const int32_t* px, int64_t n,
                                      float* o_out, float* d_out, void* stream)
{
    ApiRange api_range_("fpo_camera_rays");
    if (n < 0) return fail(FPO_E_INVALID, "n < 0");
    if (n == 0) return FPO_OK;
    if (!cam_table || !cam || !py || !px || !o_out || !d_out) return fail(FPO_E_INVALID, "NULL device pointer");
    if (n_cams < 1) return fail(FPO_E_INVALID, "n_cams must be >= 1");
    if (n > (int64_t)INT32_MAX * dev::kBlock) return fail(FPO_E_INVALID, "too many rays");
    const int64_t grid = (n + dev::kBlock - 1) / dev::kBlock;
    hipLaunchKernelGGL(dev::camera_rays_kernel, dim3((unsigned)grid), dim3(dev::kBlock), 0,
                       static_cast<hipStream_t>(stream), cam_table, n_cams, cam, py, px, n, o_out, d_out);
    return launch_status("fpo_camera_rays");
}

extern "C" fpo_status fpo_pack_coeffs(const float* src, const int64_t* perm, int64_t n_leaves,
                                      int64_t leaf_stride, const fpo_layout* layout, float* dst, void* stream)
{
    ApiRange api_range_("fpo_pack_coeffs");
    if (!src || !perm || !dst) return fail(FPO_E_INVALID, "NULL device pointer");
    if (n_leaves < 1 || leaf_stride < n_leaves) return fail(FPO_E_INVALID, "bad n_leaves / leaf_stride");
    const int n1 = layout ? layout->n_sigma : FPO_N_SIGMA;
    const int n2 = layout ? layout->n_sh_fourier : FPO_N_SH_FOURIER;
    if (!layout_supported(n1, n2)) return fail(FPO_E_UNSUPPORTED, "layout (n1, n2) not compiled");
    const int n_coeff = n1 + 3 * FPO_N_SH * n2;
    const int R = record_words(FPO_F32, n1, n2);
    const int64_t total = (int64_t)R * leaf_stride;
    if (total > (int64_t)INT32_MAX * dev::kBlock) return fail(FPO_E_INVALID, "too many leaves");
    const int64_t grid = (total + dev::kBlock - 1) / dev::kBlock;
    hipLaunchKernelGGL(dev::pack_coeffs_kernel, dim3((unsigned)grid), dim3(dev::kBlock), 0,
                       static_cast<hipStream_t>(stream), src, perm, n_leaves, leaf_stride,
                       reinterpret_cast<float4*>(dst), R, n_coeff);
    return launch_status("fpo_pack_coeffs");
}
