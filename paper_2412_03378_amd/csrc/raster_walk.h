// One wave per tile: the staged records, the pair arithmetic and the forward
// walk (see the header comment of raster.hip), for the rasteriser kernels that
// include it.
#pragma once

#include <type_traits>

#include "raster_common.h"

namespace vgr {

namespace {

constexpr int kStageVec = 6;   // record float4 the rasteriser uses (g0..g5)

template <int B>
struct Stage {
    float4 g[kStageVec][B];
    uint32_t item[B];
};

// Word of the kept pre-test mask of lane `lane` for the batch that starts at
// list position bs of global tile gt (layout: pmask_words).
template <int B>
__device__ __forceinline__ size_t mask_word(uint32_t bs, int gt, int lane)
{
    return (size_t)bs * (64 / B) + 64 * (size_t)gt + lane;
}

// Fields of the bound pre-test (g0..g2) and of the full evaluation (g3..g5).
struct PreRec {
    float hx, hy, lx, ly, Q00, Q01x2, l0x2, l1x2, Q11, A00, A10, A20;
};
struct FullRec {
    float A01, A11, A21, v0x, v0y, v0z, K, se, c0, c1, c2, mz;
};

template <class ST>
__device__ __forceinline__ PreRec load_pre(const ST &st, int q)
{
    const float4 a = st.g[0][q], b = st.g[1][q], c = st.g[2][q];
    PreRec r;
    r.hx = a.x; r.hy = a.y; r.lx = a.z; r.ly = a.w;
    r.Q00 = b.x; r.Q01x2 = b.y; r.l0x2 = b.z; r.l1x2 = b.w;
    r.Q11 = c.x; r.A00 = c.y; r.A10 = c.z; r.A20 = c.w;
    return r;
}

template <class ST>
__device__ __forceinline__ FullRec load_full(const ST &st, int q)
{
    const float4 a = st.g[3][q], b = st.g[4][q], c = st.g[5][q];
    FullRec r;
    r.A01 = a.x; r.A11 = a.y; r.A21 = a.z; r.v0x = a.w;
    r.v0y = b.x; r.v0z = b.y; r.K = b.z; r.se = b.w;
    r.c0 = c.x; r.c1 = c.y; r.c2 = c.z; r.mz = c.w;
    return r;
}

// One staged record in registers, read at a per-lane index.
struct RecRegs {
    float4 g[kStageVec];
};

template <class ST>
__device__ __forceinline__ RecRegs load_regs(const ST &st, int q)
{
    RecRegs r;
#pragma unroll
    for (int v = 0; v < kStageVec; ++v) r.g[v] = st.g[v][q];
    return r;
}

__device__ __forceinline__ PreRec pre_of4(const float4 &a, const float4 &b, const float4 &c)
{
    PreRec r;
    r.hx = a.x; r.hy = a.y; r.lx = a.z; r.ly = a.w;
    r.Q00 = b.x; r.Q01x2 = b.y; r.l0x2 = b.z; r.l1x2 = b.w;
    r.Q11 = c.x; r.A00 = c.y; r.A10 = c.z; r.A20 = c.w;
    return r;
}

__device__ __forceinline__ PreRec pre_of(const RecRegs &x)
{
    return pre_of4(x.g[0], x.g[1], x.g[2]);
}

__device__ __forceinline__ FullRec full_of(const RecRegs &x)
{
    FullRec r;
    r.A01 = x.g[3].x; r.A11 = x.g[3].y; r.A21 = x.g[3].z; r.v0x = x.g[3].w;
    r.v0y = x.g[4].x; r.v0z = x.g[4].y; r.K = x.g[4].z; r.se = x.g[4].w;
    r.c0 = x.g[5].x; r.c1 = x.g[5].y; r.c2 = x.g[5].z; r.mz = x.g[5].w;
    return r;
}

// Stage one record; returns its g5 (the colour).  wild: a field of the pre-test is not
// finite.
template <class ST>
__device__ __forceinline__ float4 stage_record(ST &st, const Buffers &b, int lane, uint32_t item,
                                               bool &wild)
{
    const float4 *gp = b.geom + (size_t)item * kRecVec;
    RecRegs r;
#pragma unroll
    for (int v = 0; v < kStageVec; ++v) r.g[v] = gp[v];
#pragma unroll
    for (int v = 0; v < kStageVec; ++v) st.g[v][lane] = r.g[v];
    st.item[lane] = item;
    float sum = fabsf(r.g[2].x);
    sum += fabsf(r.g[0].x) + fabsf(r.g[0].y) + fabsf(r.g[0].z) + fabsf(r.g[0].w);
    sum += fabsf(r.g[1].x) + fabsf(r.g[1].y) + fabsf(r.g[1].z) + fabsf(r.g[1].w);
    wild = !(sum < INFINITY);
    return r.g[5];
}

template <class ST>
__device__ __forceinline__ float4 stage_record(ST &st, const Buffers &b, int lane, uint32_t item)
{
    bool wild;
    return stage_record(st, b, lane, item, wild);
}

// Per-lane terms of the pre-test shared by the lane's pixels (pxc = px + 0.5).
struct ColTerms {
    float dx, f0, f1;
};

__device__ __forceinline__ ColTerms col_terms(const PreRec &r, float pxc)
{
    ColTerms c;
    c.dx = (pxc - r.hx) - r.lx;
    c.f0 = __fmaf_rn(c.dx, __fmaf_rn(r.Q00, c.dx, r.l0x2), -1.0f);
    c.f1 = __fmaf_rn(r.Q01x2, c.dx, r.l1x2);
    return c;
}

// Bound pre-test of one pixel (pyc = py + 0.5): true if alpha >= alpha_min is
// possible.  Writes the row offset.
__device__ __forceinline__ bool pre_test(const PreRec &r, const ColTerms &c, float pyc, float &dy)
{
    dy = (pyc - r.hy) - r.ly;
    const float f = __fmaf_rn(dy, __fmaf_rn(r.Q11, dy, c.f1), c.f0);
    return !(f > kConicMargin);
}

// Margin left by the pre-test at one pixel (pyc = py + 0.5): negative where alpha <
// alpha_min for sure.  A NaN made here is positive; the negated factors are finite
// (records with fields that are not skip the pre-test).
__device__ __forceinline__ float pre_margin(const PreRec &r, float pxc, float pyc)
{
    const float dx = (pxc - r.hx) - r.lx, dy = (pyc - r.hy) - r.ly;
    const float g0 = __fmaf_rn(-dx, __fmaf_rn(r.Q00, dx, r.l0x2), 1.0f + kConicMargin);
    const float f1 = __fmaf_rn(r.Q01x2, dx, r.l1x2);
    return __fmaf_rn(-dy, __fmaf_rn(r.Q11, dy, f1), g0);
}

// Index of the lowest bit of m (31 for m = 0: the caller sees to what it reads there).
__device__ __forceinline__ int lowest_bit(uint64_t m)
{
    uint32_t lo, hi;
    asm("v_ffbl_b32 %0, %1" : "=v"(lo) : "v"((uint32_t)m));
    asm("v_ffbl_b32 %0, %1" : "=v"(hi) : "v"((uint32_t)(m >> 32)));
    return (int)min(lo, hi + 32u);
}

struct PairGeom {
    float a0, a1, a2, w0, w1, w2, n0, n1, n2, num, qw;
};

__device__ __forceinline__ void pair_geom(const PreRec &p, const FullRec &r, float dx, float dy,
                                          PairGeom &g)
{
    g.a0 = __fmaf_rn(r.A01, dy, p.A00 * dx);
    g.a1 = __fmaf_rn(r.A11, dy, p.A10 * dx);
    g.a2 = __fmaf_rn(r.A21, dy, p.A20 * dx);
    g.w0 = r.v0x + g.a0;
    g.w1 = r.v0y + g.a1;
    g.w2 = r.v0z + g.a2;
    g.n0 = __fmaf_rn(r.v0y, g.a2, -r.v0z * g.a1);
    g.n1 = __fmaf_rn(r.v0z, g.a0, -r.v0x * g.a2);
    g.n2 = __fmaf_rn(r.v0x, g.a1, -r.v0y * g.a0);
    g.num = __fmaf_rn(g.n0, g.n0, __fmaf_rn(g.n1, g.n1, g.n2 * g.n2));
    g.qw = __fmaf_rn(g.w0, g.w0, __fmaf_rn(g.w1, g.w1, g.w2 * g.w2));
}

template <int TW, int TH>
struct TileMap {
    static constexpr int PPL = TW * TH / 64;
    static constexpr int RS = 64 / TW;
    static_assert(TW * TH % 64 == 0 && 64 % TW == 0, "tile shape");
};

// Word of qmask, within a region, of the pixel of lane l (column l % 8, row l / 8):
// block by block.
__device__ __forceinline__ uint32_t block_word(int l)
{
    return (uint32_t)((((l >> 5) & 1) * 2 + ((l >> 2) & 1)) * 16 + ((l >> 3) & 3) * 4 + (l & 3));
}

// Pair counts (per lane) and wave-level visit counts (kept by lane 0): a
// visit is one Gaussian against one slot of the wave's pixels; a full visit
// is one that takes the evaluation branch.
struct Counts {
    uint32_t test = 0, full = 0, blend = 0, visits = 0, visits_full = 0;
};

// The forward by one wave (header comment of raster.hip) of tile gt, or in colour
// with the volumetric opacity of its 8x8 region rgn (TW = TH = 8; CULL: the tile is
// larger than the region, so the list's entries that do not reach the region are left
// out first).  wg: the workgroup's record for the load balance.
template <int TW, int TH, int MODE, bool COUNT, int B, bool CULL = false>
__device__ __forceinline__ void walk_tile_fwd(const RenderParams &rp, const Buffers &b,
                                              Stage<B> &st, int gt, int rgn, int64_t wg)
{
    static_assert(B == 32 || B == 64, "records per batch");
    constexpr int PPL = TileMap<TW, TH>::PPL;
    constexpr int RS = TileMap<TW, TH>::RS;
    constexpr bool SPLAT = MODE == kModeSplat;   // colour with the 3DGS splatting alpha
    constexpr bool NEAR = MODE == kModeColorNear;
    constexpr bool EPAN = MODE == kModeColorEpan;
    // the backward runs in 4x4 pixel blocks from the pairs blended here (qmask)
    constexpr bool BLOCKS = !SPLAT;
    static_assert(!BLOCKS || (B == 64 && TW == 8 && TH == 8), "a region, 64 entries per batch");
    static_assert(BLOCKS || !CULL, "tiles are culled already");
    const bool timed = b.wg_time != nullptr;   // uniform
    const uint64_t t_start = timed ? wg_clock() : 0;
    const int v = find_view(b.views, rp.n_views, gt);
    const ViewInfo &vi = b.views[v];
    const int lt = gt - vi.tile_off;
    const int tx = lt % vi.tiles_x, ty = lt / vi.tiles_x;
    const int lane = threadIdx.x;
    const int bx = BLOCKS ? tx * rp.tile_w + block_x(4 * rgn, rp.tile_w) : tx * TW;
    const int by = BLOCKS ? ty * rp.tile_h + block_y(4 * rgn, rp.tile_w) : ty * TH;
    const int px = bx + lane % TW;
    const int py0 = by + lane / TW;
    const int W = vi.width, H = vi.height;
    const float pxc = (float)px + 0.5f;
    const float ux = (pxc - vi.cx) / vi.fx;
    uint32_t used = 0;   // batches up to the last that blended (uniform)

    float pyc[PPL], un[PPL], T[PPL], C0[PPL], C1[PPL], C2[PPL];
    int last[PPL];
    uint64_t alive[PPL];   // lanes whose pixel in slot k is in the image and has not stopped (uniform)
    Counts n;
#pragma unroll
    for (int k = 0; k < PPL; ++k) {
        const int py = py0 + k * RS;
        pyc[k] = (float)py + 0.5f;
        const float uyn = (pyc[k] - vi.cy) / vi.fy;
        un[k] = sqrtf(ux * ux + uyn * uyn + 1.0f);
        alive[k] = __builtin_amdgcn_ballot_w64(px < W && py < H);
        T[k] = 1.0f;
        C0[k] = C1[k] = C2[k] = 0.0f;
        last[k] = -1;
    }
    const uint2 range = b.ranges[gt];
    const float tau2 = rp.tau2, ymax = rp.ymax, Tmin = rp.T_min;
    const float amin = rp.amin, amax = rp.amax;
    const float zn = vi.znear;

    // A lane with no record left steps on slot 31 (lowest_bit), which a batch of fewer
    // records has not written: its weight is 0, so the colour there has to be finite.
    // Once a colour is not, every step takes the colour by whether the lane blends.
    if (lane < B) st.g[5][lane] = make_float4(0, 0, 0, 0);
    bool anyodd = false;   // of the list so far (uniform)

    // the staged records' items, a batch ahead
    uint32_t item = 0;
    if (lane < B && range.x + lane < range.y) item = b.inst_val[range.x + lane];
    for (uint32_t bs = range.x; bs < range.y; bs += B) {
        const uint32_t j = bs + lane;
        bool odd = false;   // a colour that is not finite, or huge
        bool wild = false;  // a pre-test field that is not
        int nb = (int)min((uint32_t)B, range.y - bs);
        bool keep = lane < B && j < range.y;
        int at = lane;      // where the lane's record goes
        if constexpr (CULL) {
            keep = keep && reaches<kRegion>(b.geom[(size_t)item * kRecVec + 6],
                                            b.geom[(size_t)item * kRecVec + 7], (float)bx, (float)by);
            const uint64_t km = __builtin_amdgcn_ballot_w64(keep);
            nb = __builtin_popcountll(km);
            at = __builtin_popcountll(km & ((1ull << lane) - 1ull));
        }
        if (keep) {
            const float4 c = stage_record(st, b, at, item, wild);
            odd = !ordinary(c.x, c.y, c.z);
            if constexpr (CULL) st.item[at] = (uint32_t)lane;   // its entry in the batch
        }
        if (lane < B && j + B < range.y) item = b.inst_val[j + B];
        const bool bad = wave_any(wild);   // the batch's records pass the pre-test untested
        const bool oddb = wave_any(odd);
        anyodd = anyodd || oddb;
        __syncthreads();
        {
            // Phase 1: bound pre-test of the whole batch (broadcast records);
            // bit q of mask[k] marks record q as passing for the lane's slot k.
            // The two 32-record halves fill 32-bit words with the sign bits of the
            // margins, one shift a record (so they come in reverse): one instruction
            // after the margin, where a compare and an add of its lane mask take two
            // and two wait states between them (476 -> 450 us at 3M Gaussians,
            // 1600x1064).
            uint32_t mhalf[2][PPL];
    #pragma unroll
            for (int k = 0; k < PPL; ++k) mhalf[1][k] = 0u;   // B = 32: one half
    #pragma unroll
            for (int h = 0; h < B / 32; ++h) {
    #pragma unroll
                for (int k = 0; k < PPL; ++k) mhalf[h][k] = 0u;
                const int qend = min(nb, 32 * h + 32);
                for (int qi = 32 * h; qi < qend; ++qi) {
                    const PreRec pr = pre_of4(st.g[0][qi], st.g[1][qi], st.g[2][qi]);
    #pragma unroll
                    for (int k = 0; k < PPL; ++k) {
                        mhalf[h][k] = __builtin_amdgcn_alignbit(
                            mhalf[h][k], __float_as_uint(pre_margin(pr, pxc, pyc[k])), 31);
                        if (COUNT) {
                            n.test += __builtin_amdgcn_inverse_ballot_w64(alive[k]) ? 1u : 0u;
                            n.visits += (lane == 0 && alive[k] != 0) ? 1u : 0u;
                        }
                    }
                }
                const int m = qend - 32 * h;   // uniform
    #pragma unroll
                for (int k = 0; k < PPL; ++k)
                    mhalf[h][k] = m > 0 ? (bad ? ~0u : ~__builtin_bitreverse32(mhalf[h][k])) >> (32 - m)
                                        : 0u;
            }
            uint64_t mask[PPL];
    #pragma unroll
            for (int k = 0; k < PPL; ++k)
                mask[k] = __builtin_amdgcn_inverse_ballot_w64(alive[k])
                              ? ((uint64_t)mhalf[1][k] << 32) | mhalf[0][k] : 0ull;
            // kept for the backward (layout: pmask_words)
            if constexpr (!BLOCKS) {
    #pragma unroll
                for (int k = 0; k < PPL; ++k)
                    b.pmask[mask_word<B>(bs, gt, lane) * PPL + k] = mask[k];
            }
            const size_t bq = BLOCKS ? ((quad_batch(range.x, gt) + (bs - range.x) / B) *
                                        (size_t)quad_blocks(rp.tile_w, rp.tile_h) + 4 * rgn) : 0;
            const uint32_t word = BLOCKS ? block_word(lane) : 0;   // of the lane's pixel
            // Phase 2: every lane evaluates and blends its own passing records in
            // list order, one per step (records read from LDS at per-lane
            // addresses), so a step does useful work on every lane that still has
            // a record left instead of only on those that pass one shared record.
    #pragma unroll
            for (int k = 0; k < PPL; ++k) {
                uint64_t mk = mask[k];
                uint64_t mine = 0, over = 0;   // entries the pixel blends; clamped ones (BLOCKS)
                // lanes with a record left (the loop and its masks are wave-uniform)
                uint64_t left = __builtin_amdgcn_ballot_w64(mk != 0) & alive[k];
                // ODD: some colour of the list so far is not finite
                auto blend = [&](auto ODD) {
                do {
                    const bool has = __builtin_amdgcn_inverse_ballot_w64(left);
                    const int qi = lowest_bit(mk);   // 31 if none
                    const uint32_t entry = CULL ? st.item[qi] : (uint32_t)qi;
                    mk &= mk - 1;
                    if (COUNT) {
                        n.full += has ? 1u : 0u;
                        n.visits_full += lane == 0 ? 1u : 0u;
                    }
                    const RecRegs rr = load_regs(st, qi);
                    const PreRec pr = pre_of(rr);
                    const FullRec fr = full_of(rr);
                    const float dx = (pxc - pr.hx) - pr.lx;
                    const float dy = (pyc[k] - pr.hy) - pr.ly;
                    float y, om, wa;   // log2(e) x (volumetric), 1 - alpha, alpha
                    uint64_t blm;      // lanes that reach the threshold
                    if constexpr (SPLAT) {
                        // alpha = o exp(-1/2 d^T C d) (the 3DGS splat)
                        const float e = __fmaf_rn(dx, __fmaf_rn(fr.A01, dx, fr.A11 * dy),
                                                  fr.A21 * (dy * dy));
                        const float al = fr.K * fast_exp2(-e);
                        blm = __builtin_amdgcn_ballot_w64(!(al < amin)) & left;
                        wa = al > amax ? amax : al;
                        om = 1.0f - wa;
                        y = 0.0f;
                    } else {
                        PairGeom g;
                        pair_geom(pr, fr, dx, dy, g);
                        const float rq = fast_rsq(g.qw);
                        const float ex = profile<EPAN>(fr.se, g.num, rq * rq);
                        y = (NEAR ? fabsf(fr.K) : fr.K) * un[k] * rq * ex;
                        if constexpr (NEAR) {
                            if (fr.K < 0.0f)
                                y *= norm_cdf(near_eta(fr.v0x, fr.v0y, fr.v0z, fr.mz, g.w0, g.w1,
                                                       g.w2, g.qw, rq, zn));
                        }
                        blm = __builtin_amdgcn_ballot_w64(!(y < tau2)) & left;
                        om = fast_exp2(-(y > ymax ? ymax : y));
                        wa = 1.0f - om;
                    }
                    const float Tn = T[k] * om;
                    const uint64_t low = __builtin_amdgcn_ballot_w64(Tn < Tmin);
                    const uint64_t dom = blm & ~low;
                    const bool dob = __builtin_amdgcn_inverse_ballot_w64(dom);
                    const float wgt = dob ? wa * T[k] : 0.0f;
                    float c0 = fr.c0, c1 = fr.c1, c2 = fr.c2;
                    if constexpr (ODD) {
                        c0 = dob ? c0 : 0.0f;
                        c1 = dob ? c1 : 0.0f;
                        c2 = dob ? c2 : 0.0f;
                    }
                    C0[k] = __fmaf_rn(c0, wgt, C0[k]);
                    C1[k] = __fmaf_rn(c1, wgt, C1[k]);
                    C2[k] = __fmaf_rn(c2, wgt, C2[k]);
                    T[k] = dob ? Tn : T[k];
                    alive[k] &= ~(blm & low);
                    if constexpr (BLOCKS) {
                        mine |= (uint64_t)(dob ? 1u : 0u) << (entry & 63u);
                        const uint64_t cl = __builtin_amdgcn_ballot_w64(y > ymax) & dom;
                        if (__builtin_expect(cl != 0, 0)) {
                            // (the empty asm keeps this a branch)
                            uint32_t one = __builtin_amdgcn_inverse_ballot_w64(cl) ? 1u : 0u;
                            asm volatile("" : "+v"(one));
                            over |= (uint64_t)one << (entry & 63u);
                        }
                    } else {
                        last[k] = dob ? (int)(bs + qi) : last[k];
                    }
                    if (COUNT) n.blend += dob ? 1u : 0u;
                    left = __builtin_amdgcn_ballot_w64(mk != 0) & alive[k];
                } while (left != 0);
                };
                if (left != 0) {
                    if (anyodd) blend(std::true_type{});
                    else blend(std::false_type{});
                }
                if constexpr (BLOCKS) {
                    const bool anyclamp = wave_any(over != 0);
                    b.qmask[bq * 16 + word] = mine;
                    if (anyclamp) b.qclamp[bq * 16 + word] = over;
                    if (wave_any(mine != 0)) used = (bs - range.x) / B + 1;
                    last[k] = mine != 0 ? (int)bs + 63 - (int)__builtin_clzll(mine) : last[k];
                    const uint32_t flag = (anyclamp ? kFlagClamp : 0u) | (oddb ? kFlagOdd : 0u);
                    if (lane < 4) b.qflag[bq + lane] = flag;
                }
            }
        }
        __syncthreads();
        uint64_t any = 0;
#pragma unroll
        for (int k = 0; k < PPL; ++k) any |= alive[k];
        if (any == 0) break;                          // every pixel has stopped
    }

    const int64_t HW = (int64_t)W * H;
#pragma unroll
    for (int k = 0; k < PPL; ++k) {
        const int py = py0 + k * RS;
        if (px < W && py < H) {
            const int64_t idx = (int64_t)py * W + px;
            const int64_t pidx = vi.pix_off + idx;
            vi.out[idx] = __fmaf_rn(T[k], rp.bg[0], C0[k]);
            vi.out[HW + idx] = __fmaf_rn(T[k], rp.bg[1], C1[k]);
            vi.out[2 * HW + idx] = __fmaf_rn(T[k], rp.bg[2], C2[k]);
            b.T_final[pidx] = T[k];
            if (!BLOCKS) b.last_pos[pidx] = last[k];
            b.last_id[pidx] = last[k] >= 0
                ? (int32_t)((int64_t)b.inst_val[last[k]] - (int64_t)v * rp.n) : -1;
        }
    }
    if (BLOCKS && lane < 4)
        b.qused[(size_t)gt * quad_blocks(rp.tile_w, rp.tile_h) + 4 * rgn + lane] = used;
    if (COUNT) {
        atomicAdd(&b.counters[0], (unsigned long long)n.test);
        atomicAdd(&b.counters[1], (unsigned long long)n.full);
        atomicAdd(&b.counters[2], (unsigned long long)n.blend);
        atomicAdd(&b.counters[3], (unsigned long long)n.visits);
        atomicAdd(&b.counters[4], (unsigned long long)n.visits_full);
    }
    if (timed && lane == 0)
        b.wg_time[wg] = make_uint2(cu_key(), (uint32_t)(wg_clock() - t_start));
}

}  // namespace

}  // namespace vgr
