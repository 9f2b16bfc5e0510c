// libfpo construction entry points (Sec. 4.2): per-frame values on the
// union leaves, and the per-leaf DFT of Eq. 10-12 that turns them into
// Fourier coefficients.
//
// Values of one frame and one leaf travel as snapshot records (32 F32 values:
// 0 = sigma, 1 + c*9 + j = z_{c,j}, 28..31 zero), the same records a time bake
// produces, so that the DFT of T records sampled at t = 0 .. T-1 is the exact
// inverse of fpo_bake_times for band-limited leaves.
//
// DFT kernel.  8 lanes take a leaf, a lane one 16-byte word of its record in every
// frame, and sum the terms of that word's values and a share of the density's 31
// (dft_kernel).  The weighted basis c_i IDFT_i(t) of all frames sits in LDS
// (c_0 = 1/T, c_i = 2/T, or 1/T for every i with the printed weights), computed
// from exact integer phases (i t mod 2T) with sinpi / cospi.  The kernel streams
// T records per leaf and is bound by HBM.
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

// Union leaf `slot` (cell d, i, j, k) in the frame's octree: the frame leaf that
// is the cell or contains it, else empty.  A frame node that is still internal
// at the cell's depth means the cell list does not refine the frame.
__global__ __launch_bounds__(kBlock) void frame_values_kernel(TreeDev ft, const int64_t* __restrict__ perm,
                                                              const float4* __restrict__ vals,
                                                              const int4* __restrict__ cells, int64_t n,
                                                              float4* __restrict__ out, int* __restrict__ n_bad)
{
    const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (s >= n) return;
    const int4 c = cells[s];
    const int D = ft.max_depth;
    int leaf = -1;
    bool bad = c.x < 1 || c.x > D;
    if (!bad) {
        const int sh = D - c.x;
        const int x = c.y << sh, y = c.z << sh, z = c.w << sh;
        int node = 0;
        for (int lvl = 0; lvl < c.x; ++lvl) {
            const int b = D - 1 - lvl;
            const int oct = ((x >> b) & 1) | (((y >> b) & 1) << 1) | (((z >> b) & 1) << 2);
            const int ch = ft.children[node * 8 + oct];
            if (ch < 0) {
                leaf = -ch - 1;
                break;
            }
            if (ch == 0) break;
            if (ch >= ft.n_nodes || lvl + 1 >= c.x) {
                bad = true;
                break;
            }
            node = ch;
        }
    }
    if (bad) atomicAdd(n_bad, 1);
    float4* o = out + s * 8;
    if (leaf >= 0 && leaf < ft.n_leaves && !bad) {
        const float4* v = vals + perm[leaf] * 8;
#pragma unroll
        for (int w = 0; w < 7; ++w) o[w] = v[w];
        o[7] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    } else {
#pragma unroll
        for (int w = 0; w < 8; ++w) o[w] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
}


struct DftLaunch {
    const float* frames;     // [T][stride][32]
    float* coeffs;           // [stride][192]
    float* sigma_max;        // [stride] or null
    int64_t n_leaves, stride;
    int32_t T;
    int32_t literal;
};

constexpr int kDftLeaves = 8 * kBlock / kWave;   // leaves of a block at a time: 8 per wave
constexpr int kDftOutPad = 200;                  // LDS floats per staged output record (192 + 8: spreads banks)
constexpr int kDftFrames = 4;                    // frames whose loads a wave has in flight

// Forward DFT of every leaf.  HBM-bound: T records of 128 bytes read and 768
// bytes written per leaf.  8 lanes take one leaf, lane w the 16-byte word w of
// its record in every frame, so a wave reads 1 KB of consecutive records per
// frame, the block's four waves 4 KB, with nothing staged and no barrier.  The
// lane sums the 5 terms of its (up to) four SH values and 4 of the density's
// 31 terms, for which the density is passed from lane w = 0 to the other
// seven.  The frames are read once (non-temporal loads), the next kDftFrames
// frames' loads in flight.  The coefficients leave through LDS as whole lines.
// 2 M leaves x 60 frames: 3.27 ms; without the stores the reads alone take
// 2.31 ms (6.6 TB/s): stores between reads cost HBM more than their bytes.
// One wave per output group with the records of 4 frames staged in LDS by the
// block took 3.58 ms, behind a zero fill of the output (0.21 ms).
__global__ __launch_bounds__(kBlock) void dft_kernel(DftLaunch a)
{
    // dynamic LDS: basis [T][32]
    extern __shared__ __align__(16) float lds[];
    __shared__ __align__(16) float s_out[kBlock / kWave][4 * kDftOutPad];
    const int T = a.T;
    float (*B)[FPO_BASIS_STRIDE] = reinterpret_cast<float (*)[FPO_BASIS_STRIDE]>(lds);
    for (int e = threadIdx.x; e < T * FPO_BASIS_STRIDE; e += kBlock) {
        const int t = e / FPO_BASIS_STRIDE, i = e % FPO_BASIS_STRIDE;
        // Eq. 8 at t: cos(i pi t / T) (even i), sin((i + 1) pi t / T) (odd i), exact phase
        const int m = (i & 1) ? i + 1 : i;
        const int ph = (int)(((int64_t)m * t) % (2 * T));
        const float x = (float)ph / (float)T;
        const float v = (i & 1) ? sinpif(x) : cospif(x);
        const float c = (i == 0 || a.literal) ? 1.0f / (float)T : 2.0f / (float)T;
        B[t][i] = i < FPO_N_SIGMA ? c * v : 0.0f;
    }
    __syncthreads();
    typedef float vec4 __attribute__((ext_vector_type(4)));
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int ln = threadIdx.x % kWave;
    const int w = ln & 7;                    // word of the record
    const int ll = ln >> 3;                  // leaf of the wave's eight
    float* out = s_out[wv];
    // loads of kDftFrames frames from t on of the leaves l0 .. l0 + 7; past the
    // last frame or leaf the last one is read again
    auto fetch = [&](int64_t l0, int t, vec4* v) {
        const int nl = (int)min<int64_t>(8, a.n_leaves - l0);
        const int off = min(ll, nl - 1) * 8 + w;
#pragma unroll
        for (int f = 0; f < kDftFrames; ++f) {
            const vec4* src = reinterpret_cast<const vec4*>(a.frames + (min(t + f, T - 1) * a.stride + l0) * 32);
            v[f] = __builtin_nontemporal_load(src + off);
        }
    };
    const int64_t hop = (int64_t)gridDim.x * kDftLeaves;
    int64_t l0 = ((int64_t)blockIdx.x * (kBlock / kWave) + wv) * 8;
    if (l0 >= a.n_leaves) return;
    vec4 x[kDftFrames], nx[kDftFrames];
    fetch(l0, 0, x);
    for (; l0 < a.n_leaves; l0 += hop) {
        const int nl = (int)min<int64_t>(8, a.n_leaves - l0);
        const bool in = ll < nl;
        float sg[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        float z[4][FPO_N_SH_FOURIER];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < FPO_N_SH_FOURIER; ++i) z[e][i] = 0.0f;
        float smax = -__builtin_inff();
        auto add = [&](int t, const vec4 x) {
            const float* bt = B[t];
            // the density to the leaf's 8 lanes: lane 0 of each quad's pair
            // (w & ~3 == 0), then quads 4 .. 7 from four lanes below
            const float q0 = dpp_move<0x00>(x.x);                 // quad_perm [0, 0, 0, 0]
            const float up = dpp_move<0x114>(q0);                 // row_shr 4
            const float sv = (w & 4) ? up : q0;
            const vec4 bs = *reinterpret_cast<const vec4*>(bt + 4 * w);
            smax = fmaxf(smax, sv);
#pragma unroll
            for (int e = 0; e < 4; ++e) sg[e] = fmaf(sv, bs[e], sg[e]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < FPO_N_SH_FOURIER; ++i) z[e][i] = fmaf(x[e], bt[i], z[e][i]);
        };
        // the next loads (at the end those of the next leaves) are in flight
        // while these frames are summed
        for (int t = 0; t < T; t += kDftFrames) {
            if (t + kDftFrames < T) fetch(l0, t + kDftFrames, nx);
            else if (l0 + hop < a.n_leaves) fetch(l0 + hop, 0, nx);
#pragma unroll
            for (int f = 0; f < kDftFrames; ++f)
                if (t + f < T) add(t + f, x[f]);
#pragma unroll
            for (int f = 0; f < kDftFrames; ++f) x[f] = nx[f];
        }
        if (a.sigma_max && w == 0 && in) a.sigma_max[l0 + ll] = smax;
        // records through LDS, four leaves at a time: lane w holds density
        // terms 4 w .. 4 w + 3 and SH values m = 4 w - 1 .. 4 w + 2 (value 0 of
        // word 0 is the density)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float* rec = out + (ll & 3) * kDftOutPad;
            if ((ll >> 2) == h) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (4 * w + e < FPO_N_SIGMA) rec[4 * w + e] = sg[e];
                    const int m = 4 * w - 1 + e;
                    if (m >= 0 && m < 3 * FPO_N_SH) {
#pragma unroll
                        for (int i = 0; i < FPO_N_SH_FOURIER; ++i)
                            rec[FPO_N_SIGMA + FPO_N_SH_FOURIER * m + i] = z[e][i];
                    }
                }
                for (int e = FPO_N_COEFF + w; e < 192; e += 8) rec[e] = 0.0f;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            vec4* dst = reinterpret_cast<vec4*>(a.coeffs + (l0 + 4 * h) * 192);
            const int words = min(max(nl - 4 * h, 0), 4) * 48;
#pragma unroll
            for (int k = 0; k < 4 * 48 / kWave; ++k) {
                const int e = k * kWave + ln;
                const vec4* from = reinterpret_cast<const vec4*>(out + e / 48 * kDftOutPad) + e % 48;
                if (e < words) __builtin_nontemporal_store(*from, dst + e);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }
}

}  // namespace dev
}  // namespace fpo

using namespace fpo;

extern "C" fpo_status fpo_frame_values(const fpo_tree_view* frame_tree, const int64_t* frame_perm,
                                       const float* frame_values, const int32_t* union_cells, int64_t n_union,
                                       float* out, int32_t* n_bad, void* stream)
{
    ApiRange api_range_("fpo_frame_values");
    fpo_status st = check_tree(frame_tree, false);
    if (st != FPO_OK) return st;
    if (n_union < 0) return fail(FPO_E_INVALID, "n_union < 0");
    if (n_union == 0) return FPO_OK;
    if (!frame_perm || !frame_values || !union_cells || !out || !n_bad) return fail(FPO_E_INVALID, "NULL device pointer");
    if (n_union > (int64_t)INT32_MAX * dev::kBlock) return fail(FPO_E_INVALID, "too many union leaves");
    const int64_t grid = (n_union + dev::kBlock - 1) / dev::kBlock;
    hipLaunchKernelGGL(dev::frame_values_kernel, dim3((unsigned)grid), dim3(dev::kBlock), 0,
                       static_cast<hipStream_t>(stream), dev::tree_dev(frame_tree), frame_perm,
                       reinterpret_cast<const float4*>(frame_values), reinterpret_cast<const int4*>(union_cells),
                       n_union, reinterpret_cast<float4*>(out), n_bad);
    return launch_status("fpo_frame_values");
}

extern "C" fpo_status fpo_dft_frames(const float* frames, int32_t n_frames, int64_t n_leaves, int64_t leaf_stride,
                                     int32_t literal, float* coeffs_out, float* sigma_max_out, void* stream)
{
    ApiRange api_range_("fpo_dft_frames");
    if (!frames || !coeffs_out) return fail(FPO_E_INVALID, "NULL device pointer");
    if (n_frames < 1 || n_frames > FPO_MAX_FRAMES) return fail(FPO_E_INVALID, "n_frames must be in 1..FPO_MAX_FRAMES");
    if (n_leaves < 0 || leaf_stride < n_leaves) return fail(FPO_E_INVALID, "need 0 <= n_leaves <= leaf_stride");
    if ((reinterpret_cast<uintptr_t>(frames) & 15) != 0 || (reinterpret_cast<uintptr_t>(coeffs_out) & 15) != 0)
        return fail(FPO_E_INVALID, "frames and coeffs_out must be 16-byte aligned");
    if (n_leaves == 0) return FPO_OK;
    dev::DftLaunch a;
    a.frames = frames;
    a.coeffs = coeffs_out;
    a.sigma_max = sigma_max_out;
    a.n_leaves = n_leaves;
    a.stride = leaf_stride;
    a.T = n_frames;
    a.literal = literal ? 1 : 0;
    // blocks loop over their leaves, so that the basis table is built 8 times per CU
    const int64_t tiles = (n_leaves + dev::kDftLeaves - 1) / dev::kDftLeaves;
    const unsigned grid = (unsigned)std::min<int64_t>(tiles, 2048);
    const size_t lds = sizeof(float) * (size_t)n_frames * FPO_BASIS_STRIDE;
    hipLaunchKernelGGL(dev::dft_kernel, dim3(grid), dim3(dev::kBlock), lds, static_cast<hipStream_t>(stream), a);
    return launch_status("fpo_dft_frames");
}
