// Device helpers shared by the rasteriser kernels: the pair arithmetic's
// building blocks and the lane exchanges of the transpose-reduces.
#pragma once

#include "vgr_internal.h"

namespace vgr {

namespace {

__device__ __forceinline__ float fast_rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// Near-plane segment factor Phi(eta) of a flagged record (K' < 0):
// eta = (gamma - t_n) / beta = mz (v0 . w) / |w| - zn |w| for the pixel's
// w = L u, t_n = zn |u| the near-plane crossing of the ray (Sec. 4.2, the
// integral from t_n on).  qw = |w|^2, rq = 1 / |w|.
__device__ __forceinline__ float near_eta(float v0x, float v0y, float v0z, float mz, float w0,
                                          float w1, float w2, float qw, float rq, float zn)
{
    const float vw = __fmaf_rn(v0x, w0, __fmaf_rn(v0y, w1, v0z * w2));
    return __fmaf_rn(mz, vw, -zn * qw) * rq;
}
__device__ __forceinline__ float norm_cdf(float e) { return 0.5f * erfcf(-0.70710678f * e); }

// Profile factor of the line integral at D^2 = se num rq2 (with se from the
// record): exp2(-(log2 e / 2) D^2) for the Gaussian, (1 - D^2)^(3/2) (0 past
// the support) for the Epanechnikov kernel.
template <bool EPAN>
__device__ __forceinline__ float profile(float se, float num, float rq2)
{
    if constexpr (EPAN) {
        const float h2 = fmaxf(1.0f - se * num * rq2, 0.0f);
        return h2 * __builtin_sqrtf(h2);
    } else {
        return fast_exp2(-(se * num * rq2));
    }
}

// h^(3/2) for h = 1 - d2, 0 past the support: the square root from its reciprocal and a
// Newton step, rounded correctly (checked on every float from 2^-24, the smallest h, to
// 1) in half the instructions of the compiler's.  X-ray rasterisers with this kernel, 16
// views of 200k at 512x512, forward and backward: 0.60 / 0.82 ms, 0.68 / 0.90 with the
// compiler's, 0.58 / 0.78 with v_sqrt_f32 alone, which is an ulp off on every seventh
// value.
__device__ __forceinline__ float epan_ray(float d2)
{
    const float h = fmaxf(1.0f - d2, 1e-37f);   // (its power underflows to 0)
    const float r = fast_rsq(h), s = h * r;
    return h * __fmaf_rn(__fmaf_rn(-s, s, h), 0.5f * r, s);
}

// Timed runs (b.wg_time set) record for each workgroup the constant-rate
// realtime counter difference between start and end, and a key of the compute unit it ran on (XCC id, then the
// shader engine, array and CU fields of HW_ID), so that the host can sum the
// busy time per compute unit (load balance).
__device__ __forceinline__ uint64_t wg_clock() { return __builtin_amdgcn_s_memrealtime(); }
__device__ __forceinline__ uint32_t cu_key()
{
    const uint32_t hw = __builtin_amdgcn_s_getreg(4 | (31 << 11));    // HW_ID
    const uint32_t xcc = __builtin_amdgcn_s_getreg(20 | (3 << 11));   // XCC_ID[3:0]
    return (xcc << 8) | ((hw >> 8) & 0xFFu);
}

// True if p holds on any active lane: a ballot of the predicate's lane mask,
// which the branch tests directly.
__device__ __forceinline__ bool wave_any(bool p) { return __builtin_amdgcn_ballot_w64(p) != 0; }

// Whether products of two such triples stay finite, so that a weight of 0 takes them
// out of a sum.
__device__ __forceinline__ bool ordinary(float x, float y, float z)
{
    return fabsf(x) + fabsf(y) + fabsf(z) < 1e18f;
}

__device__ __forceinline__ int find_view(const ViewInfo *views, int n_views, int gt)
{
    int v = 0;
    for (int k = 1; k < n_views; ++k)
        if (views[k].tile_off <= gt) v = k;
    return v;
}

__device__ __forceinline__ float swap_add32(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ float swap_add16(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// LDS stores of this wave visible to its own lanes.
__device__ __forceinline__ void lds_wave_sync()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// DPP lane moves (gfx9 encodings): row rotate right by 8, quad permutations
// [2,3,0,1] and [1,0,3,2].
constexpr int kDppRowRor8 = 0x128;
constexpr int kDppQuadXor2 = 0x4E;
constexpr int kDppQuadXor1 = 0xB1;

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move_u(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}

// With N13 only v[0..12] are summed (v[13..15] are zero): step 1 pairs
// (v[k], v[k+8]) for k < 5, then (v[5], v[6]) and (v[7], 0), leaving seven
// slots.  Slot s and the lane bit h that picked the pair member give the
// index of the total a lane ends with, n13_index(s, h); -1: the lane holds
// no total.
__device__ __forceinline__ int n13_index(int s, int h)
{
    return s < 5 ? s + 8 * h : (s == 5 ? 5 + h : ((s == 6 && h == 0) ? 7 : -1));
}

template <bool N13, class SWAP>
__device__ __forceinline__ void pair_step1(float (&v)[16], SWAP swap_add)
{
    if constexpr (N13) {
#pragma unroll
        for (int k = 0; k < 5; ++k) v[k] = swap_add(v[k], v[k + 8]);
        v[5] = swap_add(v[5], v[6]);
        v[6] = swap_add(v[7], 0.0f);
        v[7] = 0.0f;
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = swap_add(v[k], v[k + 8]);
    }
}

// Step 2 for the pairs (v[k], v[k+4]), k < 3: lanes with bit 3 clear (banks
// 0-1 of each row) add slot k across l ^ 8, the others slot k + 4, each lane
// writing the sum of the slot it keeps with one bank-masked DPP add (the
// compiler forms DPP adds only with every bank enabled, and then needs two
// selects to route the slots).  The s_nop gives the two wait states a DPP read
// needs after a VALU write of its source VGPR.
#define VGR_PAIR_ADD8(D, A, C)                                                   \
    "v_add_f32_dpp " D ", " A ", " A " row_ror:8 row_mask:0xf bank_mask:0x3\n\t" \
    "v_add_f32_dpp " D ", " C ", " C " row_ror:8 row_mask:0xf bank_mask:0xc\n\t"

__device__ __forceinline__ void pair_add8x3(float (&v)[16])
{
    float r0, r1, r2;
    asm volatile("s_nop 1\n\t" VGR_PAIR_ADD8("%0", "%3", "%6") VGR_PAIR_ADD8("%1", "%4", "%7")
                     VGR_PAIR_ADD8("%2", "%5", "%8")
                 : "=&v"(r0), "=&v"(r1), "=&v"(r2)
                 : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[4]), "v"(v[5]), "v"(v[6]));
    v[0] = r0;
    v[1] = r1;
    v[2] = r2;
}

// The same for the four pairs k < 4.
__device__ __forceinline__ void pair_add8x4(float (&v)[16])
{
    float r0, r1, r2, r3;
    asm volatile("s_nop 1\n\t" VGR_PAIR_ADD8("%0", "%4", "%8") VGR_PAIR_ADD8("%1", "%5", "%9")
                     VGR_PAIR_ADD8("%2", "%6", "%10") VGR_PAIR_ADD8("%3", "%7", "%11")
                 : "=&v"(r0), "=&v"(r1), "=&v"(r2), "=&v"(r3)
                 : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]),
                   "v"(v[6]), "v"(v[7]));
    v[0] = r0;
    v[1] = r1;
    v[2] = r2;
    v[3] = r3;
}
#undef VGR_PAIR_ADD8

// Sum v[0..15] over the 64 lanes (transpose-reduce).  Afterwards lane l with
// (l & 3) == 0 holds the total of index l / 4.
//   step 1: v_permlane32_swap pairs (v[k], v[k+8]); after the add, lanes 0-31
//           hold index k and lanes 32-63 index k + 8;
//   step 2: v_permlane16_swap pairs (v[k], v[k+4]); row r (16 lanes) now
//           holds indices 4 r + k, k = 0..3;
//   step 3: lanes l and l ^ 8 (DPP row rotate by 8) keep one pair of indices
//           each and send the other;
//   step 4: lanes l and 7 - l of each 8-lane half row (DPP half mirror) keep
//           one index each and send the other;
//   step 5: sums within each quad (DPP quad permutations).
// Index of the total lane l holds after wave_reduce16 (lanes l & 3 == 0).
template <bool N13>
__device__ __forceinline__ int wave_index(int lane)
{
    return N13 ? n13_index((lane >> 2) & 7, (lane >> 5) & 1) : lane >> 2;
}

// Steps 3 and 4 of wave_reduce16 as DPP adds with bank masks, each lane
// writing the sum of the slot it keeps: across l ^ 8 the lanes of banks 0-1 of
// each row keep slot 0 or 1 and those of banks 2-3 slot 2 or 3; across the
// half-row mirror (7 - i within each 8 lanes) banks 0 and 2 keep the first
// and banks 1 and 3 the second.  The compiler forms DPP adds only with every
// bank enabled and then routes the slots with selects.  The s_nops give the
// two wait states a DPP read needs after a VALU write of its source VGPR.
__device__ __forceinline__ float wave_steps34(float v0, float v1, float v2, float v3)
{
    float r0, r1, out;
    asm volatile(
        "s_nop 1\n\t"
        "v_add_f32_dpp %1, %3, %3 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %1, %5, %5 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %4, %4 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %2, %6, %6 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %0, %1, %1 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "s_nop 0\n\t"
        "v_add_f32_dpp %0, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xa"
        : "=&v"(out), "=&v"(r0), "=&v"(r1)
        : "v"(v0), "v"(v1), "v"(v2), "v"(v3));
    return out;
}

template <bool N13>
__device__ __forceinline__ float wave_reduce16(float (&v)[16], int lane)
{
    (void)lane;
    pair_step1<N13>(v, [](float a, float b) { return swap_add32(a, b); });
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = swap_add16(v[k], v[k + 4]);
    v[0] = wave_steps34(v[0], v[1], v[2], v[3]);
    v[0] += dpp_move<kDppQuadXor2>(v[0]);
    v[0] += dpp_move<kDppQuadXor1>(v[0]);
    return v[0];
}

constexpr int kBlock = 4;        // pixel block side
constexpr int kRegion = 8;       // region side: four blocks
// Position in its tile of block q: the blocks go region by region, four per region.
__device__ __forceinline__ int block_x(int q, int tile_w)
{
    return ((q >> 2) & (tile_w / kRegion - 1)) * kRegion + (q & 1) * kBlock;
}
__device__ __forceinline__ int block_y(int q, int tile_w)
{
    return (q >> 2) / (tile_w / kRegion) * kRegion + ((q >> 1) & 1) * kBlock;
}

// Whether the culling ellipse (c6, c7: record g6, g7) reaches the pixel centres
// of the SIDE x SIDE square at (bx, by): the test of the tile culling (cull_row in
// the preprocess source) for one square, with the rows cut to whole pixels first.  1-ulp square roots: their error is far below kCullPad.
template <int SIDE>
__device__ __forceinline__ bool reaches(const float4 &c6, const float4 &c7, float bx, float by)
{
    const float cx = c6.x, cy = c6.y, a = c6.z, P = c6.w;
    const float R = c7.x, ymax = c7.y, yl = c7.z;
    const float ya = fmaxf(by, ceilf(cy - ymax - kCullPad)) - cy;
    const float yb = fminf(by + (SIDE - 1), floorf(cy + ymax + kCullPad)) - cy;
    const float yla = fminf(fmaxf(yl, ya), yb), yra = fminf(fmaxf(-yl, ya), yb);
    const float left = __fmaf_rn(a, yla, -__builtin_amdgcn_sqrtf(fmaxf(P - R * yla * yla, 0.0f)));
    const float right = __fmaf_rn(a, yra, __builtin_amdgcn_sqrtf(fmaxf(P - R * yra * yra, 0.0f)));
    const float lo = fmaxf(ceilf(cx + left - kCullPad), bx);
    const float hi = fminf(floorf(cx + right + kCullPad), bx + (SIDE - 1));
    return !(c7.w > 0.0f) || (ya <= yb && lo <= hi);
}

}  // namespace

}  // namespace vgr
