// Colour rasteriser with the volumetric opacity, forward and backward, for
// gfx950 (wave64).
//
// Both are bound by VALU issue (85 to 92 % busy), in two ways that ask for two
// splits: a large frame by the work of all its pairs, a small one by its longest
// lists, whose composition is serial.  So the tiles are split in two by the length
// of their lists (d_total[3], rule at kLongShare in the preprocess source).
//
// The long ones, one wave per 4x4 pixel block (block_fwd, blocks_bwd): lane l holds
// pixel l >> 2 of the block and Gaussian l & 3 of a step of four.
//   - The list is culled per block before any pair is evaluated: 64 candidates at a
//     time, one per lane, test their bound ellipse against the block (about 25
//     instructions per 64 candidates, where a per-pixel pre-test takes 12 for each),
//     and the survivors are packed in LDS.
//   - A step reads four consecutive packed records at lane-uniform addresses.
//   - Only the composition is serial in the list: T goes through the step's four
//     Gaussians by four multiplications with quad broadcasts, in list order, so that
//     every transmittance and decision is the same as with one Gaussian at a time.
//   - The loads of the next batches are in flight during a batch's steps.
// A list takes a quarter of the steps of one wave per tile, and a frame has four
// times the waves, but 64-thread workgroups cost about 0.3 ns each to launch and the
// four waves cull the same list: a third more time once the chip is full.
//
// The others, one wave per 8x8 region: forward as in raster.hip's header (walk),
// backward the region's four blocks side by side (blocks_bwd with BPW = 4).
//
// The forward keeps, per pixel and 64 list entries, the entries the pixel blended as
// one 64-bit word (and those whose alpha was clamped, where there are any).  The
// backward packs the entries that some pixel of its block blended and takes every
// decision from the words, so it evaluates no threshold and can use a shorter form
// of the pair arithmetic (below) without ever disagreeing with the forward.  With
// four blocks per wave the records' sums are collected in LDS and added to memory
// once per batch: one block's 7 to 8 million visits x 13 atomics are bound by the
// device's 190 G float atomics/s (0.57 ms at 1M Gaussians, 1080p).
//
// Forward / backward in us, one wave per tile with a per-lane walk and quarter-wave
// backward (before) -> this split; in brackets all tiles as regions, as blocks:
//   333x250, 20k, 8x8 tiles     138 / 335  ->  54 / 69   (155 / 230,   54 / 68)
//   640x480, 100k               238 / 380  ->  93 / 92   (271 / 263,   93 / 93)
//   1280x720, 300k              141 / 251  ->  82 / 123  (156 / 169,   79 / 110)
//   1920x1080, 300k             128 / 238  -> 112 / 163  (140 / 163,  146 / 209)
//   1920x1080, 1M               249 / 596  -> 257 / 438  (259 / 440,  337 / 528)
//   1920x1080, 3M               493 / 1172 -> 511 / 834  (509 / 832,  636 / 984)
//   4 x 640x480, 300k, 16x16   1696 / 1998 -> 235 / 314  (345 / 460,  208 / 282)
//   1920x1080, 1M, 16x16        605 / 811  -> 275 / 463  (263 / 452,  356 / 558)
// (Full-size 8x8 forwards pay 3 % for the words.)
//
// Backward frame.  In an orthonormal basis (e0, e1, e2 = v0/|v0|) of the L-frame
// (ray_frame), scaled by 1/|v0|, a pixel offset d gives w = L u = (a0, a1, w2):
//   a0 = r00 dx + r01 dy,  a1 = r10 dx + r11 dy,  w2 = 1 + s0 dx + s1 dy,
//   p = w/|w|,  hp = p0^2 + p1^2,  D^2 = E hp  with  E = mz^2 |v0|^2,
//   z = sqrt(E) (-p2 p0, -p2 p1, hp),
// so the moments  M = sum t (p p^T + z z^T),  Z = sum t z  are products of p,
// hp and q = D^2 (18 operations, 45 with z and M formed in the L-frame):
//   M_ij = sum t p_i p_j (1 + E - q)  (i, j < 2),  M_i2 = sum t p_i p2 (1 - q),
//   M_22 = sum t - sum t hp (1 - q),  Z = sqrt(E) sum t (-p2 p0, -p2 p1, hp).
// The preprocess backward turns them back to the L-frame.
#include <type_traits>

#include "raster_walk.h"

namespace vgr {

namespace {

// LDS float4 between the arrays of a staged record's fields (records side by side
// in each; the pad moves the arrays to other banks)
constexpr int kStride = 64 + 1;

// Which tile slot (position in tile_order) workgroup g of a run of slots has, with
// 2^lnp workgroups per slot, and which of them it is.  The workgroups of a slot sit 8
// apart, so that they run on one XCD (workgroups go to the 8 XCDs in turn) and share
// its L2 copy of the tile's records.
__device__ __forceinline__ int part_of(uint32_t g, int lnp, uint32_t &slot)
{
    slot = (g >> (3 + lnp)) * 8 + (g & 7u);
    return (int)((g >> 3) & ((1u << lnp) - 1u));
}

__device__ __forceinline__ int log2_regions(const RenderParams &rp)
{
    return 31 - __builtin_clz((uint32_t)(rp.tile_w * rp.tile_h / (kRegion * kRegion)));
}

// Quad lane J's value on the quad's four lanes.  (bound_ctrl: every lane of the
// permutation is valid, and with it the compiler folds the move into the user.)
template <int J>
__device__ __forceinline__ float quad_bcast(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), J * 0x55, 0xF, 0xF, true));
}

// Lanes of odd r, and of r >= 2 (the asm keeps the constants in SGPR pairs).
struct QuadMasks {
    uint64_t odd = 0xAAAAAAAAAAAAAAAAull, high = 0xCCCCCCCCCCCCCCCCull;
    __device__ __forceinline__ QuadMasks() { asm volatile("" : "+s"(odd), "+s"(high)); }
};

// x[r] for quad lane r, as three selects on constant lane masks.
__device__ __forceinline__ float quad_pick(const QuadMasks &m, float x0, float x1, float x2, float x3)
{
    const bool odd = __builtin_amdgcn_inverse_ballot_w64(m.odd);
    const bool high = __builtin_amdgcn_inverse_ballot_w64(m.high);
    const float a = odd ? x1 : x0, b = odd ? x3 : x2;
    return high ? b : a;
}

__device__ __forceinline__ int quad_max(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(0, v, kDppQuadXor1, 0xF, 0xF, false));
    return max(v, __builtin_amdgcn_update_dpp(0, v, kDppQuadXor2, 0xF, 0xF, false));
}

// Lane `from`'s value.
__device__ __forceinline__ uint64_t lane_from(uint64_t v, int from)
{
    const uint32_t lo = __builtin_amdgcn_ds_bpermute(4 * from, (int)(uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_ds_bpermute(4 * from, (int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// OR over the four lanes of each quad.
__device__ __forceinline__ uint64_t quad_or(uint64_t m)
{
    uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
    lo |= dpp_move_u<kDppQuadXor1>(lo);
    hi |= dpp_move_u<kDppQuadXor1>(hi);
    lo |= dpp_move_u<kDppQuadXor2>(lo);
    hi |= dpp_move_u<kDppQuadXor2>(hi);
    return ((uint64_t)hi << 32) | lo;
}

// OR over the 16 lanes of each row (on lane 0 of the row at least).
__device__ __forceinline__ uint32_t row_or(uint32_t m)
{
    m |= dpp_move_u<kDppRowRor8>(m);
    m |= dpp_move_u<0x124>(m);   // row_ror:4
    m |= dpp_move_u<kDppQuadXor2>(m);
    return m | dpp_move_u<kDppQuadXor1>(m);
}

// Pair counts per lane; steps and (Gaussian, block) visits on lane 0.
struct QuadCounts {
    uint32_t test = 0, full = 0, blend = 0, steps = 0, visits = 0;
};

__device__ __forceinline__ void add_counts(unsigned long long *c, const QuadCounts &n)
{
    atomicAdd(c + 0, (unsigned long long)n.test);
    atomicAdd(c + 1, (unsigned long long)n.full);
    atomicAdd(c + 2, (unsigned long long)n.blend);
    atomicAdd(c + 3, (unsigned long long)n.steps);
    atomicAdd(c + 4, (unsigned long long)n.visits);
}

// Packed records of the forward: the fields of g0 and g2..g5 that a pair reads,
// at the survivor's rank.  c holds the colours per step and channel (float4 4 s + ch:
// channel ch of the step's four Gaussians), since lane r of a quad composites
// channel r of its pixel.  Up to three slots past the survivors pad the last step.
template <bool NEAR>
struct FwdStage {
    float4 h[68];                    // hx, hy, lx, ly
    float4 a[68];                    // A00, A10, A20, A01
    float4 v[68];                    // A11, A21, v0x, v0y
    float4 k[68];                    // v0z, K', se, list position
    float4 c[64];
    float mz[NEAR ? 68 : 1];
};

// One candidate's record in registers.
struct Rec {
    float4 h, g3, g4, g5;
    float a00, a10, a20;             // g2.yzw
};

__device__ __forceinline__ void load_rec(Rec &x, const Buffers &b, uint32_t item)
{
    const float4 *gp = b.geom + (size_t)item * kRecVec;
    x.h = gp[0];
    const float4 g2 = gp[2];
    x.a00 = g2.y;
    x.a10 = g2.z;
    x.a20 = g2.w;
    x.g3 = gp[3];
    x.g4 = gp[4];
    x.g5 = gp[5];
}

// C + c.x w0 + c.y w1 + c.z w2 + c.w w3 in this order, w_j quad lane j's w.  Written
// out, since the compiler leaves the quad broadcasts of a multiply-add apart.
// The s_nop: two wait states before a DPP read of a VGPR just written.
__device__ __forceinline__ float add_colors(float w, const float4 &c, float C)
{
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f32_dpp %0, %1, %2 quad_perm:[0,0,0,0] row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %0, %1, %3 quad_perm:[1,1,1,1] row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %0, %1, %4 quad_perm:[2,2,2,2] row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %0, %1, %5 quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf"
                 : "+v"(C)
                 : "v"(w), "v"(c.x), "v"(c.y), "v"(c.z), "v"(c.w));
    return C;
}

// The forward of block q of tile gt by one wave.
template <int MODE, bool COUNT>
__device__ __forceinline__ void block_fwd(const RenderParams &rp, const Buffers &b,
                                          FwdStage<MODE == kModeColorNear> &st, int gt, int q,
                                          int64_t wg)
{
    constexpr bool NEAR = MODE == kModeColorNear;
    constexpr bool EPAN = MODE == kModeColorEpan;
    const int lnb = log2_regions(rp) + 2;
    const bool timed = b.wg_time != nullptr;        // uniform
    const uint64_t t_start = timed ? wg_clock() : 0;
    const int v = find_view(b.views, rp.n_views, gt);
    const ViewInfo &vi = b.views[v];
    const int lt = gt - vi.tile_off;
    const int ty = lt / vi.tiles_x, tx = lt - ty * vi.tiles_x;
    const int lane = threadIdx.x, r = lane & 3, p = lane >> 2;
    const int bx = tx * rp.tile_w + block_x(q, rp.tile_w);
    const int by = ty * rp.tile_h + block_y(q, rp.tile_w);
    const int px = bx + (p & 3), py = by + (p >> 2);
    const int W = vi.width, H = vi.height;
    const float pxc = (float)px + 0.5f, pyc = (float)py + 0.5f;
    const float ux = (pxc - vi.cx) / vi.fx;
    const float uyn = (pyc - vi.cy) / vi.fy;
    const float un = sqrtf(ux * ux + uyn * uyn + 1.0f);
    const bool inside = px < W && py < H;
    const uint2 range = b.ranges[gt];
    const float tau2 = rp.tau2, ymax = rp.ymax, Tmin = rp.T_min;
    const float zn = vi.znear;
    const uint64_t below = (1ull << lane) - 1ull;
    const QuadMasks qm;

    float T = 1.0f, C = 0.0f;   // C: channel r
    int last = -1;
    // colours past a batch's survivors are read (with no lane blending), so they
    // have to be finite: they are zeros or an earlier batch's, and zeros again after a
    // batch with one that is not finite
    st.c[lane] = make_float4(0, 0, 0, 0);
    uint64_t alive = __builtin_amdgcn_ballot_w64(inside);   // uniform
    uint32_t used = 0;                                      // batches up to the last that blended
    QuadCounts n;

    // Candidates (one per lane) move through three batches: item, culling ellipse,
    // record; each load is issued a batch before its use and is in flight during
    // the steps of the batch before.
    uint32_t it1 = 0, it2 = 0;       // items of the next batch, of the one after
    float4 c6 = make_float4(0, 0, 0, 0), c7 = c6;   // ellipses of the next batch
    Rec rec;                         // records of the next batch's survivors
    uint64_t km1 = 0;                // the next batch's survivors
    auto load_item = [&](uint32_t j, uint32_t &it) {
        if (j < range.y) it = b.inst_val[j];
    };
    auto load_ellipse = [&](uint32_t j, uint32_t it) {
        if (j < range.y) {
            c6 = b.geom[(size_t)it * kRecVec + 6];
            c7 = b.geom[(size_t)it * kRecVec + 7];
        }
    };
    auto cull = [&](uint32_t j, uint32_t it) {
        const bool keep = j < range.y && reaches<kBlock>(c6, c7, (float)bx, (float)by);
        km1 = __builtin_amdgcn_ballot_w64(keep);
        if (keep) load_rec(rec, b, it);
    };
    if (alive != 0 && range.x < range.y) {
        const uint32_t j = range.x + lane;
        load_item(j, it1);
        load_item(j + 64, it2);
        load_ellipse(j, it1);
        cull(j, it1);
        load_ellipse(j + 64, it2);
        it1 = it2;
        load_item(j + 128, it2);
    }
    size_t batch = quad_batch(range.x, gt);
    for (uint32_t bs = range.x; bs < range.y && alive != 0; bs += 64, ++batch) {
        const uint32_t j = bs + lane;
        const uint64_t km = km1;
        const int cnt = __builtin_popcountll(km);
        bool odd = false;   // a colour that is not finite, or huge
        if (__builtin_amdgcn_inverse_ballot_w64(km)) {
            const int at = __builtin_popcountll(km & below);
            st.h[at] = rec.h;
            st.a[at] = make_float4(rec.a00, rec.a10, rec.a20, rec.g3.x);
            st.v[at] = make_float4(rec.g3.y, rec.g3.z, rec.g3.w, rec.g4.x);
            st.k[at] = make_float4(rec.g4.y, rec.g4.z, rec.g4.w, __uint_as_float(j - range.x));
            float *c = reinterpret_cast<float *>(st.c) + (at >> 2) * 16 + (at & 3);
            c[0] = rec.g5.x;
            c[4] = rec.g5.y;
            c[8] = rec.g5.z;
            if constexpr (NEAR) st.mz[at] = rec.g5.w;
            odd = !ordinary(rec.g5.x, rec.g5.y, rec.g5.z);
        }
        if (lane < 4) {   // the pad: |w| = 1 and K' = 0, which blends nowhere
            st.h[cnt + lane] = st.a[cnt + lane] = st.v[cnt + lane] = make_float4(0, 0, 0, 0);
            st.k[cnt + lane] = make_float4(1.0f, 0, 0, 0);
        }
        const bool anyodd = wave_any(odd);
        cull(j + 64, it1);
        load_ellipse(j + 128, it2);
        it1 = it2;
        load_item(j + 192, it2);
        if (COUNT) {
            const uint32_t nb = min(64u, range.y - bs);
            n.test += (r == 0 && __builtin_amdgcn_inverse_ballot_w64(alive)) ? nb : 0u;
            n.steps += lane == 0 ? nb : 0u;
            n.visits += lane == 0 ? (uint32_t)cnt : 0u;
        }
        __syncthreads();
        // entries of the batch that the lane blended, and of those it clamped
        uint64_t mine = 0, over = 0;
        // ODD: some colour of the batch is not ordinary; it reaches only the pixels
        // that blend it
        auto steps = [&](auto ODD) {
            int lim = cnt;
            for (int s = 0; 4 * s < lim; ++s) {
                const int at = 4 * s + r;
                const float4 h = st.h[at], ra = st.a[at], rv = st.v[at], rk = st.k[at];
                float4 c = st.c[at];
                const float dx = (pxc - h.x) - h.z, dy = (pyc - h.y) - h.w;
                const float a0 = __fmaf_rn(ra.w, dy, ra.x * dx);
                const float a1 = __fmaf_rn(rv.x, dy, ra.y * dx);
                const float a2 = __fmaf_rn(rv.y, dy, ra.z * dx);
                const float v0 = rv.z, v1 = rv.w, v2 = rk.x;
                const float w0 = v0 + a0, w1 = v1 + a1, w2 = v2 + a2;
                const float n0 = __fmaf_rn(v1, a2, -v2 * a1);
                const float n1 = __fmaf_rn(v2, a0, -v0 * a2);
                const float n2 = __fmaf_rn(v0, a1, -v1 * a0);
                const float num = __fmaf_rn(n0, n0, __fmaf_rn(n1, n1, n2 * n2));
                const float qw = __fmaf_rn(w0, w0, __fmaf_rn(w1, w1, w2 * w2));
                const float rq = fast_rsq(qw);
                const float ex = profile<EPAN>(rk.z, num, rq * rq);
                float y = (NEAR ? fabsf(rk.y) : rk.y) * un * rq * ex;
                if constexpr (NEAR) {
                    if (rk.y < 0.0f)
                        y *= norm_cdf(near_eta(v0, v1, v2, st.mz[at], w0, w1, w2, qw, rq, zn));
                }
                // lanes that blend, unless the pixel stops in this step
                uint64_t bm = __builtin_amdgcn_ballot_w64(!(y < tau2)) & alive;
                const bool clamped = y > ymax;
                const float om = fast_exp2(-(clamped ? ymax : y));
                const float wa = 1.0f - om;
                const float oe = __builtin_amdgcn_inverse_ballot_w64(bm) ? om : 1.0f;
                // T in front of each of the four, in list order
                const float T1 = T * quad_bcast<0>(oe), T2 = T1 * quad_bcast<1>(oe);
                const float T3 = T2 * quad_bcast<2>(oe), T4 = T3 * quad_bcast<3>(oe);
                const float Tb = quad_pick(qm, T, T1, T2, T3);
                const uint64_t stop = __builtin_amdgcn_ballot_w64(!(T4 >= Tmin));
                if (__builtin_expect(stop == 0, 1)) {
                    T = T4;
                } else {
                    // T keeps the last value before the first one below Tmin, where the
                    // pixel stops: what is behind it, NaN (a line integral of Inf * 0)
                    // included, does not count
                    const bool s1 = T1 < Tmin, s2 = s1 || T2 < Tmin, s3 = s2 || T3 < Tmin;
                    const bool s4 = s3 || T4 < Tmin;
                    bm &= __builtin_amdgcn_ballot_w64(!(r == 0 ? s1 : (r == 1 ? s2 : (r == 2 ? s3 : s4))));
                    T = s1 ? T : (s2 ? T1 : (s3 ? T2 : (s4 ? T3 : T4)));
                    alive &= ~__builtin_amdgcn_ballot_w64(s4);
                    if (alive == 0) lim = 0;   // every pixel has stopped
                }
                const bool dob = __builtin_amdgcn_inverse_ballot_w64(bm);
                const float wgt = dob ? wa * Tb : 0.0f;
                if constexpr (ODD) {
                    c.x = quad_bcast<0>(wgt) != 0.0f ? c.x : 0.0f;
                    c.y = quad_bcast<1>(wgt) != 0.0f ? c.y : 0.0f;
                    c.z = quad_bcast<2>(wgt) != 0.0f ? c.z : 0.0f;
                    c.w = quad_bcast<3>(wgt) != 0.0f ? c.w : 0.0f;
                }
                // in list order, so that the image does not depend on the tile shape
                C = add_colors(wgt, c, C);
                last = dob ? (int)__float_as_uint(rk.w) : last;
                const uint64_t bit = dob ? 1ull << (__float_as_uint(rk.w) & 63u) : 0ull;
                mine |= bit;
                over |= clamped ? bit : 0ull;
                if (COUNT) {
                    // (the per-pixel form of the bound, as the pair count past it)
                    const uint32_t jt = range.x + __float_as_uint(rk.w);
                    if (at < cnt && inside) {
                        const float4 *gp = b.geom + (size_t)b.inst_val[jt] * kRecVec;
                        const float4 g1 = gp[1], g2 = gp[2];
                        const float e0 = __fmaf_rn(dx, __fmaf_rn(g1.x, dx, g1.z), -1.0f);
                        const float e1 = __fmaf_rn(g1.y, dx, g1.w);
                        const float f = __fmaf_rn(dy, __fmaf_rn(g2.x, dy, e1), e0);
                        n.full += (dob || (((alive >> lane) & 1) && !(f > kConicMargin))) ? 1u : 0u;
                    }
                    n.blend += dob ? 1u : 0u;
                }
            }
        };
        if (anyodd) steps(std::true_type{});
        else steps(std::false_type{});
        const size_t bq = (batch << lnb) + q;
        mine = quad_or(mine);
        over = quad_or(over);
        if (wave_any(mine != 0)) used = (bs - range.x) / 64 + 1;
        const bool anyclamp = wave_any(over != 0);
        if (r == 0) {
            b.qmask[bq * 16 + p] = mine;
            if (anyclamp) b.qclamp[bq * 16 + p] = over;
        }
        if (lane == 0) b.qflag[bq] = (anyclamp ? kFlagClamp : 0u) | (anyodd ? kFlagOdd : 0u);
        if (anyodd) st.c[lane] = make_float4(0, 0, 0, 0);
        __syncthreads();
    }

    if (lane == 0) b.qused[((size_t)gt << lnb) + q] = used;
    last = quad_max(last);
    if (inside) {
        const int64_t HW = (int64_t)W * H;
        const int64_t idx = (int64_t)py * W + px;
        const int64_t pidx = vi.pix_off + idx;
        if (r < 3) {
            const float bg = r == 0 ? rp.bg[0] : (r == 1 ? rp.bg[1] : rp.bg[2]);
            vi.out[r * HW + idx] = __fmaf_rn(T, bg, C);
        } else {
            b.T_final[pidx] = T;
            b.last_id[pidx] = last >= 0
                ? (int32_t)((int64_t)b.inst_val[range.x + last] - (int64_t)v * rp.n) : -1;
        }
    }
    if (COUNT) add_counts(b.counters, n);
    if (timed && lane == 0)
        b.wg_time[wg] = make_uint2(cu_key(), (uint32_t)(wg_clock() - t_start));
}

// Workgroups g = 0 .. color_workgroups() - 1 lie in rows of 2^kGridRow: a grid
// dimension has fewer than 2^32 threads, and so fewer than 2^26 of these workgroups,
// the regions of 16 views of 16384x16384.
constexpr int kGridRow = 20;
__device__ __forceinline__ uint32_t workgroup() { return (blockIdx.y << kGridRow) + blockIdx.x; }

// First the long tiles, one wave per block, then the others, one wave per region
// (CULL: tiles are larger than a region).
template <bool CULL, int MODE, bool COUNT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(6))) void color_fwd_kernel(
    RenderParams rp, Buffers b)
{
    using Block = FwdStage<MODE == kModeColorNear>;
    using Walk = Stage<64>;
    __shared__ __align__(16) unsigned char lds[sizeof(Block) > sizeof(Walk) ? sizeof(Block) : sizeof(Walk)];
    const int lnr = log2_regions(rp);
    const uint32_t nlong = b.d_total[3];
    const uint32_t wlong = ((nlong + 7u) / 8u * 8u) << (lnr + 2);   // their workgroups
    const uint32_t g = workgroup();
    uint32_t slot;
    if (g < wlong) {
        const int q = part_of(g, lnr + 2, slot);
        if (slot < nlong)
            block_fwd<MODE, COUNT>(rp, b, *reinterpret_cast<Block *>(lds), (int)b.tile_order[slot], q, g);
    } else {
        const int rgn = part_of(g - wlong, lnr, slot);
        slot += nlong;
        if (slot < (uint32_t)rp.total_tiles)
            walk_tile_fwd<8, 8, MODE, COUNT, 64, CULL>(rp, b, *reinterpret_cast<Walk *>(lds),
                                                       (int)b.tile_order[slot], rgn, g);
    }
}

// Slots a and c summed across lanes l ^ 8 of each row, then across l ^ 4: banks
// 0-1 (0 and 2) of a row keep a, banks 2-3 (1 and 3) keep c, one bank-masked DPP
// add each (the compiler forms DPP adds only with every bank enabled and then
// routes the slots with selects).  s_nop 1: a DPP read of a VGPR that a VALU
// instruction wrote needs two wait states; s_nop 2: a lane swap likewise.
#define VGR_ADD8(D, A, C)                                                             \
    "v_add_f32_dpp " D ", " A ", " A " row_ror:8 row_mask:0xf bank_mask:0x3\n\t"      \
    "v_add_f32_dpp " D ", " C ", " C " row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
#define VGR_ADD4(D, A, C)                                                             \
    "v_add_f32_dpp " D ", " A ", " A " row_shl:4 row_mask:0xf bank_mask:0x5\n\t"      \
    "v_add_f32_dpp " D ", " C ", " C " row_shr:4 row_mask:0xf bank_mask:0xa\n\t"

// Sum v[0..15] (v[0..12] if N13) over the 16 lanes of the same l & 3: across
// l ^ 8 and l ^ 4 by bank-masked DPP adds, then across l ^ 16 and l ^ 32 by lane
// swaps (which take twice the issue time of a DPP add, so the levels with many
// slots go first to DPP), each level halving the slots.  Lane l ends with index
// quad_index(l) of its Gaussian (-1: none).
template <bool N13>
__device__ __forceinline__ float quad_reduce16(float (&v)[16])
{
    float a0, a1, a2, a3, a4, a5, a6, b0, b1, b2, b3;
    if constexpr (N13) {
        // pairs (k, k + 8) for k < 5, (5, 6), and 7 alone; then (k, k + 4), k < 3,
        // and 3 alone
        asm volatile("s_nop 1\n\t" VGR_ADD8("%0", "%7", "%15") VGR_ADD8("%1", "%8", "%16")
                         VGR_ADD8("%2", "%9", "%17") VGR_ADD8("%3", "%10", "%18")
                         VGR_ADD8("%4", "%11", "%19") VGR_ADD8("%5", "%12", "%13")
                     "v_add_f32_dpp %6, %14, %14 row_ror:8 row_mask:0xf bank_mask:0xf"
                     : "=&v"(a0), "=&v"(a1), "=&v"(a2), "=&v"(a3), "=&v"(a4), "=&v"(a5), "=&v"(a6)
                     : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]),
                       "v"(v[7]), "v"(v[8]), "v"(v[9]), "v"(v[10]), "v"(v[11]), "v"(v[12]));
        asm volatile("s_nop 1\n\t" VGR_ADD4("%0", "%4", "%8") VGR_ADD4("%1", "%5", "%9")
                         VGR_ADD4("%2", "%6", "%10")
                     "v_add_f32_dpp %3, %7, %7 row_shl:4 row_mask:0xf bank_mask:0x5\n\t"
                     "s_nop 2"
                     : "=&v"(b0), "=&v"(b1), "=&v"(b2), "=&v"(b3)
                     : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "v"(a4), "v"(a5), "v"(a6));
    } else {
        float a7;
        asm volatile("s_nop 1\n\t" VGR_ADD8("%0", "%8", "%16") VGR_ADD8("%1", "%9", "%17")
                         VGR_ADD8("%2", "%10", "%18") VGR_ADD8("%3", "%11", "%19")
                         VGR_ADD8("%4", "%12", "%20") VGR_ADD8("%5", "%13", "%21")
                         VGR_ADD8("%6", "%14", "%22") VGR_ADD8("%7", "%15", "%23")
                     : "=&v"(a0), "=&v"(a1), "=&v"(a2), "=&v"(a3), "=&v"(a4), "=&v"(a5),
                       "=&v"(a6), "=&v"(a7)
                     : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]),
                       "v"(v[7]), "v"(v[8]), "v"(v[9]), "v"(v[10]), "v"(v[11]), "v"(v[12]),
                       "v"(v[13]), "v"(v[14]), "v"(v[15]));
        asm volatile("s_nop 1\n\t" VGR_ADD4("%0", "%4", "%8") VGR_ADD4("%1", "%5", "%9")
                         VGR_ADD4("%2", "%6", "%10") VGR_ADD4("%3", "%7", "%11") "s_nop 2"
                     : "=&v"(b0), "=&v"(b1), "=&v"(b2), "=&v"(b3)
                     : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "v"(a4), "v"(a5), "v"(a6), "v"(a7));
    }
    return swap_add32(swap_add16(b0, b2), swap_add16(b1, b3));
}
#undef VGR_ADD8
#undef VGR_ADD4

template <bool N13>
__device__ __forceinline__ int quad_index(int lane)
{
    // level by level: bit 3 picks the pair member, bits 2, 4 and 5 the slot
    const int s = ((lane >> 2) & 1) * 4 + ((lane >> 4) & 1) * 2 + (lane >> 5);
    const int h = (lane >> 3) & 1;
    return N13 ? n13_index(s, h) : s + 8 * h;
}

// Candidates of the backward in the ray frame (see the header comment), the
// survivors' offsets of the current block, and with four blocks per wave the blocks'
// pixels and the sums of the batch's records over the region.  Those leave the wave
// once per batch: the global atomics (about one float per clock and L2 channel) else
// bound the kernel.
template <bool NEAR, int BPW>
struct BwdStage {
    float4 h[kStride];               // hx, hy, lx, ly
    float4 r[kStride];               // r00, r01, r10, r11
    float4 s[kStride];               // s0, s1, K'/|v0|, E
    float4 c[kStride];               // r, g, b, item
    float4 e[NEAR ? kStride : 1];    // mz |v0|, |v0| (near-plane segment)
    uint16_t off[64];
    // [record][slot]; an odd number of floats apart, to spread the four records of a
    // step over the banks
    static constexpr int kAcc = NEAR ? 17 : 13;
    float acc[BPW == 4 ? 65 * kAcc : 1];
    float4 pix[BPW == 4 ? 64 : 1];   // per pixel of the region: |u|, dL/dC
    float2 run[BPW == 4 ? 64 : 1];   // T in front of, and GB behind, what was replayed
};
constexpr uint32_t kPad = 64 * 16;   // offset of record 64, which no lane blends

// The backward of BPW blocks of tile gt from q0 on (a region's four, or one) by one
// wave.
template <int MODE, bool COUNT, int BPW>
__device__ __forceinline__ void blocks_bwd(const RenderParams &rp, const Buffers &b,
                                           BwdStage<MODE == kModeColorNear, BPW> &st, int gt,
                                           int q0, int64_t wg)
{
    constexpr bool NEAR = MODE == kModeColorNear;
    constexpr bool EPAN = MODE == kModeColorEpan;
    constexpr int NS = NEAR ? 16 : 13;   // slots
    constexpr int kAcc = BwdStage<NEAR, BPW>::kAcc;
    const int lnb = log2_regions(rp) + 2;
    const bool timed = b.wg_time != nullptr;        // uniform
    const uint64_t t_start = timed ? wg_clock() : 0;
    const int lane = threadIdx.x, r = lane & 3, p = lane >> 2;
    int used[BPW], top = 0;
#pragma unroll
    for (int k = 0; k < BPW; ++k) {
        used[k] = (int)b.qused[((size_t)gt << lnb) + q0 + k];
        top = max(top, used[k]);
    }
    QuadCounts n;
    if (top != 0) {   // uniform
        const int v = find_view(b.views, rp.n_views, gt);
        const ViewInfo &vi = b.views[v];
        const int lt = gt - vi.tile_off;
        const int ty = lt / vi.tiles_x, tx = lt - ty * vi.tiles_x;
        const int bx = tx * rp.tile_w + block_x(q0, rp.tile_w);
        const int by = ty * rp.tile_h + block_y(q0, rp.tile_w);
        const int W = vi.width, H = vi.height;
        const uint2 range = b.ranges[gt];
        const float ymax = rp.ymax, zn = vi.znear;
        const uint64_t below = (1ull << lane) - 1ull;
        const QuadMasks qm;
        const int e = quad_index<!NEAR>(lane);
        const uint64_t emask = __builtin_amdgcn_ballot_w64(e >= 0);
        float *rg = reinterpret_cast<float *>(b.rgrad) + (e >= 0 ? e : 0);

        // GB: dL/dC . (colour composited behind the current Gaussian)
        float un, T = 1.0f, GB, g0 = 0.0f, g1 = 0.0f, g2 = 0.0f;
        {
            // one block: the lane's pixel; four: pixel `lane` of the region, block by
            // block, which goes to LDS
            const int pl = BPW == 4 ? lane & 15 : p, bl = BPW == 4 ? lane >> 4 : 0;
            const int x = bx + (bl & 1) * kBlock + (pl & 3), y = by + (bl >> 1) * kBlock + (pl >> 2);
            const float ux = ((float)x + 0.5f - vi.cx) / vi.fx;
            const float uyn = ((float)y + 0.5f - vi.cy) / vi.fy;
            un = sqrtf(ux * ux + uyn * uyn + 1.0f);
            if (x < W && y < H) {
                const int64_t HW = (int64_t)W * H;
                const int64_t idx = (int64_t)y * W + x;
                T = b.T_final[vi.pix_off + idx];
                g0 = vi.dL[idx];
                g1 = vi.dL[HW + idx];
                g2 = vi.dL[2 * HW + idx];
            }
            GB = T * __fmaf_rn(g2, rp.bg[2], __fmaf_rn(g1, rp.bg[1], g0 * rp.bg[0]));
        }
        if constexpr (BPW == 4) {
            st.pix[lane] = make_float4(un, g0, g1, g2);
            st.run[lane] = make_float2(T, GB);
            // the sums of the entries that a batch has, to the end of their last four,
            // which leave together below (the pad's are never read)
            const int sums = ((int)min(range.y - range.x, 64u) + 3) / 4 * 4 * kAcc;
            for (int i = lane; i < sums; i += 64) st.acc[i] = 0.0f;
        }
        // record 64, named by the slots past a block's survivors, is read with no
        // lane blending: it has to hold finite values
        if (lane == 0) {
            st.h[64] = st.r[64] = st.s[64] = st.c[64] = make_float4(0, 0, 0, 0);
            if constexpr (NEAR) st.e[64] = make_float4(0, 0, 0, 0);
        }

        // Batches move through two stages, from the last to the first: masks and
        // items, then the records some pixel blended; each load is issued a batch
        // before its use and is in flight during the steps of the batch after.
        const size_t bq0 = (quad_batch(range.x, gt) << lnb) + q0;
        uint64_t mask1 = 0;                    // of the next batch: lane's pixel (as above)
        uint32_t flag1 = 0, it1 = 0, itr = 0;  // its flags (lane k: block k) and items; items of rec
        Rec rec;
        const int ml = BPW == 4 ? lane : p, mk = BPW == 4 ? lane >> 4 : 0;
        auto load_masks = [&](int k) {
            if (k < 0) return;   // uniform
            const size_t bq = bq0 + ((size_t)k << lnb);
            // (a block the forward had left by then has written none)
            const bool on = k < (BPW == 1 ? used[0] : (mk == 0 ? used[0] : (mk == 1 ? used[1 % BPW] : (mk == 2 ? used[2 % BPW] : used[3 % BPW]))));
            mask1 = on ? b.qmask[bq * 16 + ml] : 0ull;
            flag1 = on ? b.qflag[bq + mk] : 0u;
            const uint32_t j = range.x + 64u * (uint32_t)k + lane;
            if (j < range.y) it1 = b.inst_val[j];
        };
        uint64_t mask = 0, cmask = 0;          // entries the lane's pixel blended; clamped
        uint32_t klo = 0, khi = 0, flags = 0;  // entries some pixel of the lane's row blended
        uint64_t kany = 0;                     // of the wave (uniform)
        // the next batch becomes the current one: its records are loaded
        auto advance = [&](int k) {
            if (k < 0) return;   // uniform
            mask = mask1;
            klo = row_or((uint32_t)mask);
            khi = row_or((uint32_t)(mask >> 32));
            kany = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                kany |= ((uint64_t)__builtin_amdgcn_readlane(khi, 16 * u) << 32) |
                        (uint32_t)__builtin_amdgcn_readlane(klo, 16 * u);
            flags = (wave_any((flag1 & kFlagClamp) != 0) ? kFlagClamp : 0u) |
                    (wave_any((flag1 & kFlagOdd) != 0) ? kFlagOdd : 0u);
            cmask = 0;
            if ((flags & kFlagClamp) != 0 && (flag1 & kFlagClamp) != 0)
                cmask = b.qclamp[(bq0 + ((size_t)k << lnb)) * 16 + ml];
            itr = it1;
            if (__builtin_amdgcn_inverse_ballot_w64(kany)) load_rec(rec, b, itr);
            load_masks(k - 1);
        };
        load_masks(top - 1);
        advance(top - 1);
        // (after the batch's loads are under way)
        bool wild = wave_any(!ordinary(g0, g1, g2) || !(fabsf(GB) < INFINITY));   // uniform
        for (int kb = top - 1; kb >= 0; --kb) {
            if (__builtin_amdgcn_inverse_ballot_w64(kany)) {
                const float vx = rec.g3.w, vy = rec.g4.x, vz = rec.g4.y;
                const float V2 = __fmaf_rn(vx, vx, __fmaf_rn(vy, vy, vz * vz));
                const float iV = fast_rsq(V2), mz = rec.g5.w;
                float B[9];
                ray_frame(vx * iV, vy * iV, vz * iV, B);
                float R[6];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const float ex = iV * B[3 * i], ey = iV * B[3 * i + 1], ez = iV * B[3 * i + 2];
                    R[2 * i] = __fmaf_rn(ex, rec.a00, __fmaf_rn(ey, rec.a10, ez * rec.a20));
                    R[2 * i + 1] = __fmaf_rn(ex, rec.g3.x, __fmaf_rn(ey, rec.g3.y, ez * rec.g3.z));
                }
                st.h[lane] = rec.h;
                st.r[lane] = make_float4(R[0], R[1], R[2], R[3]);
                st.s[lane] = make_float4(R[4], R[5], rec.g4.z * iV, mz * mz * V2);
                st.c[lane] = make_float4(rec.g5.x, rec.g5.y, rec.g5.z, __uint_as_float(itr));
                if constexpr (NEAR) st.e[lane] = make_float4(mz * (V2 * iV), V2 * iV, 0, 0);
            }
            // CLAMP: a pair of the batch was clamped.  WILD: a colour of the list so far or
            // an upstream gradient is not ordinary; what a pixel does not blend is left
            // out by selects, since a weight of 0 does not take it, or what its GB has
            // become, out
            wild = wild || (flags & kFlagOdd) != 0;
            const bool special = wild || flags != 0;   // uniform
            const uint64_t cur = mask, curc = cmask, touched = kany;
            const uint32_t clo = klo, chi = khi;
            advance(kb - 1);
            for (int k = 0; k < BPW; ++k) {
                const uint64_t km = ((uint64_t)__builtin_amdgcn_readlane(chi, 16 * k) << 32) |
                                    (uint32_t)__builtin_amdgcn_readlane(clo, 16 * k);
                if (BPW == 4 ? km == 0 : touched == 0) continue;   // uniform
                const uint64_t kk = BPW == 4 ? km : touched;       // the block's survivors
                const int cnt = __builtin_popcountll(kk);
                const int rank = __builtin_popcountll(kk & below);
                const bool keep = __builtin_amdgcn_inverse_ballot_w64(kk);
                // (in-order LDS: the previous block's reads have returned)
                st.off[keep ? rank : cnt + lane - rank] = (uint16_t)(keep ? lane * 16 : kPad);
                float pxk = (float)(bx + (p & 3)) + 0.5f, pyk = (float)(by + (p >> 2)) + 0.5f;
                uint64_t bmask = cur, cm = curc;
                if constexpr (BPW == 4) {
                    pxk += (float)((k & 1) * kBlock);
                    pyk += (float)((k >> 1) * kBlock);
                    const float4 px4 = st.pix[16 * k + p];
                    const float2 rn = st.run[16 * k + p];
                    un = px4.x; g0 = px4.y; g1 = px4.z; g2 = px4.w;
                    T = rn.x;
                    GB = rn.y;
                    bmask = lane_from(cur, 16 * k + p);
                    if (special) cm = lane_from(curc, 16 * k + p);
                }
                lds_wave_sync();
                auto steps = [&](auto CLAMP, auto WILD) {
                for (int s = (cnt + 3) / 4 - 1; s >= 0; --s) {
                    const uint32_t off = st.off[4 * s + r];
                    const char *rb = reinterpret_cast<const char *>(st.h) + off;
                    const float4 h = *reinterpret_cast<const float4 *>(rb);
                    const float4 rr = *reinterpret_cast<const float4 *>(rb + 16 * kStride);
                    const float4 rs = *reinterpret_cast<const float4 *>(rb + 32 * kStride);
                    const float4 rc = *reinterpret_cast<const float4 *>(rb + 48 * kStride);
                    // the lane's sum so far (the lanes of a step hold different ones, and
                    // this wave alone writes them)
                    const uint32_t sum_at = BPW == 4 ? (off >> 4) * kAcc + max(e, 0) : 0;
                    const float sum = BPW == 4 ? st.acc[sum_at] : 0.0f;
                    const uint32_t en = (off >> 4) & 63u;   // (the pad: any)
                    const bool bl = off != kPad && ((bmask >> en) & 1u) != 0;
                    const float dx = (pxk - h.x) - h.z, dy = (pyk - h.y) - h.w;
                    const float a0 = __fmaf_rn(rr.y, dy, rr.x * dx);
                    const float a1 = __fmaf_rn(rr.w, dy, rr.z * dx);
                    const float w2 = __fmaf_rn(rs.y, dy, __fmaf_rn(rs.x, dx, 1.0f));
                    const float qw = __fmaf_rn(w2, w2, __fmaf_rn(a0, a0, a1 * a1));
                    const float rq = fast_rsq(qw);
                    const float p0 = a0 * rq, p1 = a1 * rq, p2 = w2 * rq;
                    const float hp = __fmaf_rn(p0, p0, p1 * p1);
                    const float E = rs.w, D2 = E * hp;
                    float ex;
                    if constexpr (EPAN) ex = epan_ray(D2);
                    else ex = fast_exp2(-(0.5f * kLog2e) * D2);
                    float y = (NEAR ? fabsf(rs.z) : rs.z) * un * rq * ex;
                    // near-plane segment: y *= Phi(eta); hn = h (eta + 2 zn |w|) and
                    // h = phi(eta) / Phi(eta) enter the moments below
                    float hh = 0.0f, hn = 0.0f;
                    if constexpr (NEAR) {
                        if (rs.z < 0.0f) {
                            const float2 ev = *reinterpret_cast<const float2 *>(rb + 64 * kStride);
                            const float zw = zn * ev.y * (qw * rq);   // zn |w|
                            const float eta = __fmaf_rn(ev.x, p2, -zw);
                            const float Phi = norm_cdf(eta);
                            y *= Phi;
                            // far out in the lower tail Phi underflows and h tends to -eta
                            hh = Phi > 1e-30f ? 0.39894228f * fast_exp2(-0.72134752f * eta * eta) / Phi
                                              : -eta;
                            hn = hh * __fmaf_rn(2.0f, zw, eta);
                        }
                    }
                    y = bl ? y : 0.0f;
                    bool clamped = false;
                    float ye = y;
                    if constexpr (CLAMP) {
                        clamped = bl && ((cm >> en) & 1u) != 0;
                        ye = clamped ? ymax : y;
                    }
                    const float om = fast_exp2(-ye);
                    const float inv = fast_rcp(om);
                    // T in front of each of the four, from the last to the first
                    const float T3 = T * quad_bcast<3>(inv), T2 = T3 * quad_bcast<2>(inv);
                    const float T1 = T2 * quad_bcast<1>(inv), T0 = T1 * quad_bcast<0>(inv);
                    const float Tb = quad_pick(qm, T0, T1, T2, T3);
                    T = T0;
                    float gc = __fmaf_rn(g0, rc.x, __fmaf_rn(g1, rc.y, g2 * rc.z));
                    if constexpr (WILD) gc = bl ? gc : 0.0f;
                    const float wgt = (1.0f - om) * Tb;
                    const float gw = gc * wgt;
                    const float G2 = GB + quad_bcast<3>(gw), G1 = G2 + quad_bcast<2>(gw);
                    const float G0 = G1 + quad_bcast<1>(gw);
                    const float Gr = quad_pick(qm, G0, G1, G2, GB);
                    GB = G0 + quad_bcast<0>(gw);
                    // dL/dalpha = T_before (g.c) - (g.B) / (1 - alpha)
                    const float da = __fmaf_rn(Tb, gc, -(inv * Gr));
                    float t = da * (kLn2 * om) * y;             // dL/d(ln x)
                    if constexpr (CLAMP) t = clamped ? 0.0f : t;
                    float acc[16];
                    acc[10] = g0 * wgt;
                    acc[11] = g1 * wgt;
                    acc[12] = g2 * wgt;
                    if constexpr (WILD) {
                        acc[10] = bl ? acc[10] : 0.0f;
                        acc[11] = bl ? acc[11] : 0.0f;
                        acc[12] = bl ? acc[12] : 0.0f;
                        t = bl ? t : 0.0f;
                    }
                    acc[13] = acc[14] = acc[15] = 0.0f;
                    acc[9] = t;
                    if constexpr (!NEAR && !EPAN) {
                        const float kk = 1.0f - D2, k1 = kk + E;
                        const float tp0 = t * p0, tp1 = t * p1;
                        const float tk0 = tp0 * k1, tk1 = tp1 * k1;
                        acc[0] = tk0 * p0;
                        acc[1] = tk0 * p1;
                        acc[3] = tk1 * p1;
                        acc[6] = tp0 * p2;
                        acc[7] = tp1 * p2;
                        acc[2] = acc[6] * kk;
                        acc[4] = acc[7] * kk;
                        acc[8] = t * hp;
                        acc[5] = acc[8] * kk;
                    } else {
                        // weights of p p^T (tw) and of the z terms (tz)
                        float tw = t, tz = t;
                        if constexpr (EPAN) tz = t != 0.0f ? t * (3.0f * fast_rcp(1.0f - D2)) : 0.0f;
                        if constexpr (NEAR) {
                            tw = __fmaf_rn(t, hn, t);
                            const float th = t * hh;
                            acc[13] = th * p0;
                            acc[14] = th * p1;
                            acc[15] = th * p2;
                        }
                        const float kp = __fmaf_rn(tz, E - D2, tw), kq = __fmaf_rn(-tz, D2, tw);
                        const float z0 = tz * p0, z1 = tz * p1;
                        acc[0] = kp * p0 * p0;
                        acc[1] = kp * p0 * p1;
                        acc[3] = kp * p1 * p1;
                        acc[6] = z0 * p2;
                        acc[7] = z1 * p2;
                        acc[2] = kq * p0 * p2;
                        acc[4] = kq * p1 * p2;
                        acc[8] = tz * hp;
                        // sum t - M_22
                        acc[5] = __fmaf_rn(-tw, p2 * p2, __fmaf_rn(-acc[8], D2, t));
                    }
                    const float tot = quad_reduce16<!NEAR>(acc);
                if constexpr (BPW == 4) {
                        if (__builtin_amdgcn_inverse_ballot_w64(emask)) st.acc[sum_at] = sum + tot;
                    } else {
                        if (e >= 0 && off != kPad)
                            atomicAdd(rg + (size_t)__float_as_uint(rc.w) * kGradFloats, tot);
                    }
                    if (COUNT) {
                        const bool in = bx + (k & 1) * kBlock + (p & 3) < W &&
                                        by + (k >> 1) * kBlock + (p >> 2) < H;
                        n.steps += lane == 0 ? 1u : 0u;
                        n.visits += lane == 0 ? (uint32_t)min(4, cnt - 4 * s) : 0u;
                        n.full += (in && off != kPad) ? 1u : 0u;
                        n.blend += bl ? 1u : 0u;
                    }
                }
                };
                if (!special) steps(std::false_type{}, std::false_type{});
                else if (!wild) steps(std::true_type{}, std::false_type{});
                else steps(std::true_type{}, std::true_type{});
                if (BPW == 4 && r == 0) st.run[16 * k + p] = make_float2(T, GB);
            }
            if constexpr (BPW == 4) {
                // the region's sums: 16 lanes a record, four records at a time
                lds_wave_sync();
                const int f = lane & 15;
#pragma unroll 4
                for (int g = 0; g < 16; ++g) {
                    if (((touched >> (4 * g)) & 0xFull) == 0) continue;   // uniform
                    const int at = 4 * g + (lane >> 4);
                    if (f >= NS) continue;
                    const float sum = st.acc[at * kAcc + f];
                    const uint32_t it = __float_as_uint(st.c[at].w);
                    st.acc[at * kAcc + f] = 0.0f;
                    if (sum != 0.0f)
                        atomicAdd(reinterpret_cast<float *>(b.rgrad) + (size_t)it * kGradFloats + f, sum);
                }
            }
            __syncthreads();
        }
    }
    if (COUNT) add_counts(b.counters + 8, n);
    if (timed && lane == 0)
        b.wg_time[wg] = make_uint2(cu_key(), (uint32_t)(wg_clock() - t_start));
}

// First the long tiles, one wave per block, then the others, one wave per region.
template <int MODE, bool COUNT>
__global__ __launch_bounds__(64) void color_bwd_kernel(RenderParams rp, Buffers b, int64_t wg_half)
{
    constexpr bool NEAR = MODE == kModeColorNear;
    using One = BwdStage<NEAR, 1>;
    using Four = BwdStage<NEAR, 4>;
    __shared__ __align__(16) unsigned char lds[sizeof(Four)];
    static_assert(sizeof(One) <= sizeof(Four), "LDS");
    const int lnr = log2_regions(rp);
    const uint32_t nlong = b.d_total[3];
    const uint32_t wlong = ((nlong + 7u) / 8u * 8u) << (lnr + 2);   // their workgroups
    const uint32_t g = workgroup();
    uint32_t slot;
    if (g < wlong) {
        const int q = part_of(g, lnr + 2, slot);
        if (slot < nlong)
            blocks_bwd<MODE, COUNT, 1>(rp, b, *reinterpret_cast<One *>(lds), (int)b.tile_order[slot],
                                       q, wg_half + g);
    } else {
        const int rgn = part_of(g - wlong, lnr, slot);
        slot += nlong;
        if (slot < (uint32_t)rp.total_tiles)
            blocks_bwd<MODE, COUNT, 4>(rp, b, *reinterpret_cast<Four *>(lds),
                                       (int)b.tile_order[slot], rgn * 4, wg_half + g);
    }
}

}  // namespace

// Workgroups: one per region, and for up to long_tiles_max() tiles one per block.
int64_t color_workgroups(const RenderParams &rp)
{
    const int64_t cap = (long_tiles_max(rp.total_tiles, rp.tile_w, rp.tile_h) + 7) / 8 * 8;
    const int64_t blocks = quad_blocks(rp.tile_w, rp.tile_h);
    return cap * blocks + ((int64_t)rp.total_tiles + 7) / 8 * 8 * (blocks / 4);
}

static dim3 color_grid(const RenderParams &rp)
{
    const int64_t n = color_workgroups(rp), row = (int64_t)1 << kGridRow;
    return n <= row ? dim3((unsigned)n) : dim3((unsigned)row, (unsigned)((n + row - 1) / row));
}

hipError_t launch_color_fwd(const RenderParams &rp, const Buffers &b, bool count, hipStream_t s)
{
    const dim3 grid = color_grid(rp);
    const bool cull = rp.tile_w * rp.tile_h > 64;
#define VGR_FWD(M)                                                                        \
    do {                                                                                  \
        if (cull && count) color_fwd_kernel<true, M, true><<<grid, 64, 0, s>>>(rp, b);    \
        else if (cull) color_fwd_kernel<true, M, false><<<grid, 64, 0, s>>>(rp, b);       \
        else if (count) color_fwd_kernel<false, M, true><<<grid, 64, 0, s>>>(rp, b);      \
        else color_fwd_kernel<false, M, false><<<grid, 64, 0, s>>>(rp, b);                \
    } while (0)
    if (rp.kernel == VGR_KERNEL_EPANECHNIKOV) VGR_FWD(kModeColorEpan);
    else if (rp.near_segment) VGR_FWD(kModeColorNear);
    else VGR_FWD(VGR_MODE_COLOR);
#undef VGR_FWD
    return hipGetLastError();
}

hipError_t launch_color_bwd(const RenderParams &rp, const Buffers &b, bool count, hipStream_t s)
{
    const int64_t wg_half = color_workgroups(rp);
    const dim3 grid = color_grid(rp);
#define VGR_BWD(M)                                                                  \
    do {                                                                            \
        if (count) color_bwd_kernel<M, true><<<grid, 64, 0, s>>>(rp, b, wg_half);   \
        else color_bwd_kernel<M, false><<<grid, 64, 0, s>>>(rp, b, wg_half);        \
    } while (0)
    if (rp.kernel == VGR_KERNEL_EPANECHNIKOV) VGR_BWD(kModeColorEpan);
    else if (rp.near_segment) VGR_BWD(kModeColorNear);
    else VGR_BWD(VGR_MODE_COLOR);
#undef VGR_BWD
    return hipGetLastError();
}

}  // namespace vgr
