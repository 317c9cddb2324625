// X-ray rasteriser (sum of line integrals), forward and backward, for gfx950 (wave64).
//
// A tile of TW x TH pixels is a few 8x8 regions ("slots").  The sum has no order and no
// early stop, so a tile's list is split over the waves of a workgroup, 64 entries to a
// wave in turn (xray_waves).  Both kernels are bound by VALU issue; each holds in the
// lanes what it sums last.
//
// Ray frame.  In an orthonormal basis (e0, e1, e2 = v0/|v0|) of the L-frame, scaled by
// 1/|v0|, a pixel offset d gives w = L u = (a0, a1, w2) with
//   a0 = r00 dx + r01 dy,  a1 = r11 dy,  w2 = 1 + s0 dx + s1 dy
// (e0 is turned about e2 so that a1 does not depend on dx; ray_axes in the preprocess
// source, which writes the record so),
//   h = a0^2 + a1^2,  |w|^2 = h + w2^2,  D^2 = E h / |w|^2  with  E = mz^2 |v0|^2,
//   y = K'/|v0| |u| exp2(-(log2 e / 2) D^2) / |w|           (y = log2(e) x, Sec. 4.2):
// seven operations per pair up to |w|^2, 37 in the L-frame, and no cancellation is
// added, since a0 and a1 vanish at the mean's ray.  |u| is left out of the sums and
// multiplied in at the end; the cut compares with tau / |u|.
//
// Forward: lane l holds pixel (l & 7, l >> 3) of every slot; the waves' sums meet in
// LDS, in wave order.
//   - 64 entries at a time, one per lane, test their bound ellipse against each slot
//     (25 instructions per 64 entries and slot, where a pre-test of every pixel takes
//     seven per entry and slot); the ballots are scalars, and a scalar branch leaves
//     out the slots an entry does not reach.
//   - An entry's record is read with scalar loads, one entry ahead, and its fields are
//     scalar operands: no LDS staging, no per-lane copies.
//   - The number of terms of a pixel is an output, so the cut decides as the L-frame
//     formula does: a value within kTie of the cut (one visit in 200) is evaluated
//     again in the L-frame, from the rest of the record.
//
// Backward (it takes the forward's decisions, with the same band around the cut): lane l
// holds an entry.  Entries that reach a slot are packed in LDS, and 64
// of them run over the slot's 64 pixels, whose dL/dx and cut are broadcast from LDS; a
// lane sums its own record's moments, so nothing is reduced over lanes (a sum of ten
// values over a wave costs as much as a pair).  Along a row a1 is constant, so the
// moments need only sums of T = t / |w|^2 and (1 - D^2) T times 1, a0, a0^2, w2 and
// a0 w2, and the other factors come in per row.  With t = dL/d(ln x), p = w / |w| and
// z = sqrt(E) (-p2 p0, -p2 p1, h / |w|^2):
//   M_ij = sum t p_i p_j (1 + E - D^2)  (i, j < 2),  M_i2 = sum t p_i p2 (1 - D^2),
//   M_22 = sum t - sum t h/|w|^2 (1 - D^2),  Z = sqrt(E) sum t (-p2 p0, -p2 p1, h/|w|^2).
// The records' sums leave through LDS, 16 lanes a record.
//
// Forward / backward us, one wave per tile with a pre-test per pixel and slot, staged
// records and a transpose-reduce per record (before) -> this:
//   12 x 160x160, 8k Gaussians, 8x8 tiles         53 / 164 ->  50 / 70
//   8 x 256x256, 60k, 8x8                        355 / 1110 -> 295 / 332
//   64 x 512x512, 500k, 16x16 (371M instances) 56400 / 123600 -> 37700 / 59100
// (87 and 134 cycles per visit of 64 pairs; a backward that held pixels in its lanes took
// 68800, and one that decides by the ray frame also next to the cut 58500.)
#include "raster_common.h"

namespace vgr {

namespace {

typedef float vec4 __attribute__((ext_vector_type(4)));
// read with scalar loads (no kernel that reads records writes them)
typedef const __attribute__((address_space(4))) vec4 *RecPtr;

__device__ __forceinline__ RecPtr record_of(const Buffers &b, uint32_t item)
{
    return (RecPtr)(uintptr_t)(b.geom + (size_t)item * kRecVec);
}

// Fields of the ray frame: h (hx, hy, lx, ly), r (r00, r01, r11, unused), s (s0, s1,
// K'/|v0|, E scaled for the profile).
struct RayRec {
    vec4 h, r, s;
};

__device__ __forceinline__ RayRec load_ray(RecPtr p)
{
    return { p[0], p[1], p[2] };
}

// Relative band around the cut in which the L-frame decides: far above the rounding
// of either formula.
constexpr float kTie = 1.0f / 1024;
constexpr float kMost = (1.0f - kTie) / (1.0f + kTie);   // its lower end over its upper

template <int MODE>
struct Kind {
    static constexpr bool NEAR = MODE == kModeXrayNear;
    static constexpr bool EPAN = MODE == kModeXrayEpan;
};

template <int TW, int TH>
struct Slots {
    static constexpr int NX = TW / kRegion, NY = TH / kRegion, N = NX * NY;
};

// A pair's geometry.
struct RayPair {
    float a0, a1, w2, h, qw, rq, rq2;
};

__device__ __forceinline__ RayPair ray_pair(float a0, float a1, float a1sq, float w2)
{
    RayPair g;
    g.a0 = a0;
    g.a1 = a1;
    g.w2 = w2;
    g.h = __fmaf_rn(a0, a0, a1sq);
    g.qw = __fmaf_rn(w2, w2, g.h);
    g.rq = fast_rsq(g.qw);
    g.rq2 = g.rq * g.rq;
    return g;
}

// Near-plane segment (raster_common.h) in the ray frame: eta, and zn |w|.
// V = |v0|.
__device__ __forceinline__ float ray_eta(float V, float mz, const RayPair &g, float zn, float &zw)
{
    zw = zn * V * (g.qw * g.rq);
    return __fmaf_rn(mz * V, g.w2 * g.rq, -zw);
}
// |v0| of a record's g4, g5.
template <class V4>
__device__ __forceinline__ float length_v0(const V4 &g4, const V4 &g5)
{
    return __builtin_amdgcn_sqrtf(__fmaf_rn(g4.z, g4.z, __fmaf_rn(g4.w, g4.w, g5.x * g5.x)));
}

// log2(e) x of a pair by the L-frame formula of the colour kernels, from a record's g3
// to g5.
template <int MODE, class V4>
__device__ __forceinline__ float lframe_y(const V4 &g3, const V4 &g4, const V4 &g5, float dx,
                                          float dy, float un, float zn)
{
    const float A00 = g3.x, A10 = g3.y, A20 = g3.z, A01 = g3.w, A11 = g4.x, A21 = g4.y;
    const float v0x = g4.z, v0y = g4.w, v0z = g5.x, K = g5.y, se = g5.z, mz = g5.w;
    const float a0 = __fmaf_rn(A01, dy, A00 * dx);
    const float a1 = __fmaf_rn(A11, dy, A10 * dx);
    const float a2 = __fmaf_rn(A21, dy, A20 * dx);
    const float w0 = v0x + a0, w1 = v0y + a1, w2 = v0z + a2;
    const float n0 = __fmaf_rn(v0y, a2, -v0z * a1);
    const float n1 = __fmaf_rn(v0z, a0, -v0x * a2);
    const float n2 = __fmaf_rn(v0x, a1, -v0y * a0);
    const float num = __fmaf_rn(n0, n0, __fmaf_rn(n1, n1, n2 * n2));
    const float qw = __fmaf_rn(w0, w0, __fmaf_rn(w1, w1, w2 * w2));
    const float rq = fast_rsq(qw);
    const float ex = profile<Kind<MODE>::EPAN>(se, num, rq * rq);
    float y = (Kind<MODE>::NEAR ? fabsf(K) : K) * un * rq * ex;
    if constexpr (Kind<MODE>::NEAR) {
        if (K < 0.0f) y *= norm_cdf(near_eta(v0x, v0y, v0z, mz, w0, w1, w2, qw, rq, zn));
    }
    return y;
}

// What a wave knows of its tile; lane l as pixel (l & 7, l >> 3) of each slot.
template <int TW, int TH>
struct TileWave {
    using S = Slots<TW, TH>;
    const ViewInfo *vi;
    int bx, by, lane;

    __device__ __forceinline__ TileWave(const RenderParams &rp, const Buffers &b, int gt)
    {
        vi = &b.views[find_view(b.views, rp.n_views, gt)];
        const int lt = gt - vi->tile_off;
        const int ty = lt / vi->tiles_x, tx = lt - ty * vi->tiles_x;
        lane = threadIdx.x & 63;
        bx = tx * TW;
        by = ty * TH;
    }
    __device__ __forceinline__ int slot_x(int k) const { return bx + (k % S::NX) * kRegion; }
    __device__ __forceinline__ int slot_y(int k) const { return by + (k / S::NX) * kRegion; }
    __device__ __forceinline__ int x(int k) const { return slot_x(k) + (lane & 7); }
    __device__ __forceinline__ int y(int k) const { return slot_y(k) + (lane >> 3); }
    __device__ __forceinline__ bool in(int k) const { return x(k) < vi->width && y(k) < vi->height; }
    // slots outside the image hold no pixel
    __device__ __forceinline__ bool any(int k) const
    {
        return slot_x(k) < vi->width && slot_y(k) < vi->height;
    }
    __device__ __forceinline__ float unit(int px, int py) const   // |u| of a pixel
    {
        const float ux = ((float)px + 0.5f - vi->cx) / vi->fx;
        const float uy = ((float)py + 0.5f - vi->cy) / vi->fy;
        return sqrtf(ux * ux + uy * uy + 1.0f);
    }
    __device__ __forceinline__ float unit(int k) const { return unit(x(k), y(k)); }
};

// The lanes' candidates, a batch ahead: item and culling ellipse.
struct Candidate {
    uint32_t item = 0;
    float4 c6 = make_float4(0, 0, 0, 0), c7 = make_float4(0, 0, 0, 0);
    __device__ __forceinline__ void load(const Buffers &b, uint2 range, uint32_t j)
    {
        if (j < range.y) {
            item = b.inst_val[j];
            c6 = b.geom[(size_t)item * kRecVec + 6];
            c7 = b.geom[(size_t)item * kRecVec + 7];
        }
    }
};

// Lowest set bit (63 for 0); a lane mask added (one instruction where a select and an add
// take two; the mask comes over a branch, which gives the two wait states a VALU read
// needs after the VALU wrote it).
__device__ __forceinline__ int lowest(uint64_t m)
{
    int q;
    asm("s_ff1_i32_b64 %0, %1" : "=s"(q) : "s"(m));
    return q & 63;
}
__device__ __forceinline__ void add_mask(int &n, uint64_t m)
{
    uint64_t c;
    asm("v_addc_co_u32 %0, %1, 0, %0, %2" : "+v"(n), "=&s"(c) : "s"(m));
}

struct XrayCounts {
    uint32_t test = 0, full = 0, blend = 0, visits = 0, visits_full = 0;
};

__device__ __forceinline__ void add_counts(unsigned long long *c, const XrayCounts &n)
{
    atomicAdd(c + 0, (unsigned long long)n.test);
    atomicAdd(c + 1, (unsigned long long)n.full);
    atomicAdd(c + 2, (unsigned long long)n.blend);
    atomicAdd(c + 3, (unsigned long long)n.visits);
    atomicAdd(c + 4, (unsigned long long)n.visits_full);
}

// One workgroup of blockDim.x / 64 waves per tile.  LDS: (waves - 1) x slots x 64
// (sum, terms).
template <int TW, int TH, int MODE, bool COUNT>
__global__ __launch_bounds__(512) void xray_fwd_kernel(RenderParams rp, Buffers b)
{
    using S = Slots<TW, TH>;
    constexpr bool NEAR = Kind<MODE>::NEAR, EPAN = Kind<MODE>::EPAN;
    extern __shared__ float2 part[];
    const bool timed = b.wg_time != nullptr;   // uniform
    const uint64_t t_start = timed ? wg_clock() : 0;
    const int gt = (int)b.tile_order[blockIdx.x];
    const TileWave<TW, TH> t(rp, b, gt);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const uint2 range = b.ranges[gt];
    const float zn = t.vi->znear, tau2 = rp.tau2;

    // least sure term, and least possible one (infinite outside the image)
    float C[S::N], sure[S::N], most[S::N];
    int terms[S::N];
#pragma unroll
    for (int k = 0; k < S::N; ++k) {
        C[k] = 0.0f;
        terms[k] = 0;
        const float cut = t.in(k) ? tau2 / t.unit(k) : INFINITY;
        sure[k] = cut * (1.0f + kTie);
        most[k] = cut * (1.0f - kTie);
    }
    float pxc[S::NX], pyc[S::NY];
#pragma unroll
    for (int c = 0; c < S::NX; ++c) pxc[c] = (float)t.x(c) + 0.5f;
#pragma unroll
    for (int r = 0; r < S::NY; ++r) pyc[r] = (float)t.y(r * S::NX) + 0.5f;
    XrayCounts n;
    Candidate cand;
    const uint32_t first = range.x + 64u * (uint32_t)wv, step = 64u * (uint32_t)nw;
    cand.load(b, range, first + t.lane);
    for (uint32_t bs = first; bs < range.y; bs += step) {
        const uint32_t j = bs + t.lane;
        // bit k: the lane's candidate reaches slot k
        uint32_t reach = 0;
        if (j < range.y) {
#pragma unroll
            for (int k = 0; k < S::N; ++k)
                if (t.any(k) && reaches<kRegion>(cand.c6, cand.c7, (float)t.slot_x(k), (float)t.slot_y(k)))
                    reach |= 1u << k;
        }
        uint64_t u = __builtin_amdgcn_ballot_w64(reach != 0);
        const uint32_t items = cand.item;
        cand.load(b, range, j + step);
        if (COUNT) {
#pragma unroll
            for (int k = 0; k < S::N; ++k) {
                n.test += t.in(k) ? min(64u, range.y - bs) : 0u;
                n.visits += t.lane == 0 && t.any(k) ? min(64u, range.y - bs) : 0u;
            }
        }
        if (u == 0) continue;   // uniform
        int q = lowest(u);
        RecPtr rec = record_of(b, __builtin_amdgcn_readlane(items, q));
        RayRec c = load_ray(rec);
        do {
            // the next entry's record, in flight during this one (past the last entry
            // lane 63's: some item of the list, or item 0)
            u &= u - 1;
            const int qn = lowest(u);
            const RecPtr recn = record_of(b, __builtin_amdgcn_readlane(items, qn));
            const RayRec next = load_ray(recn);
            const uint32_t slots = S::N > 1 ? __builtin_amdgcn_readlane(reach, q) : 1u;
            float dx[S::NX], a0c[S::NX], wc[S::NX], dy[S::NY], a1[S::NY], a1sq[S::NY];
#pragma unroll
            for (int i = 0; i < S::NX; ++i) {
                dx[i] = (pxc[i] - c.h.x) - c.h.z;
                a0c[i] = c.r.x * dx[i];
                wc[i] = __fmaf_rn(c.s.x, dx[i], 1.0f);
            }
#pragma unroll
            for (int i = 0; i < S::NY; ++i) {
                dy[i] = (pyc[i] - c.h.y) - c.h.w;
                a1[i] = c.r.z * dy[i];
                a1sq[i] = a1[i] * a1[i];
            }
#pragma unroll
            for (int k = 0; k < S::N; ++k) {
                if ((slots & (1u << k)) == 0) continue;   // uniform
                const int ix = k % S::NX, iy = k / S::NX;
                const RayPair g = ray_pair(__fmaf_rn(c.r.y, dy[iy], a0c[ix]), a1[iy], a1sq[iy],
                                           __fmaf_rn(c.s.y, dy[iy], wc[ix]));
                const float d2 = c.s.w * (g.h * g.rq2);   // (log2 e / 2) D^2, or D^2 (EPAN)
                float ex;
                if constexpr (EPAN) ex = epan_ray(d2);
                else ex = fast_exp2(-d2);
                float y = (NEAR ? fabsf(c.s.z) : c.s.z) * (g.rq * ex);
                if constexpr (NEAR) {
                    if (c.s.z < 0.0f) {   // uniform
                        const vec4 g4 = rec[4], g5 = rec[5];
                        float zw;
                        y *= norm_cdf(ray_eta(length_v0(g4, g5), g5.w, g, zn, zw));
                    }
                }
                uint64_t on = __builtin_amdgcn_ballot_w64(y > sure[k]);
                const uint64_t may = __builtin_amdgcn_ballot_w64(!(y < most[k]));
                if (__builtin_expect(on != may, 0)) {
                    const float yl = lframe_y<MODE>(rec[3], rec[4], rec[5], dx[ix], dy[iy], t.unit(k), zn);
                    on |= __builtin_amdgcn_ballot_w64(!(yl < tau2)) & may &
                          __builtin_amdgcn_ballot_w64(t.in(k));
                }
                C[k] += __builtin_amdgcn_inverse_ballot_w64(on) ? y : 0.0f;
                add_mask(terms[k], on);
                if (COUNT) {
                    n.full += t.in(k) ? 1u : 0u;
                    n.blend += __builtin_amdgcn_inverse_ballot_w64(on) ? 1u : 0u;
                    n.visits_full += t.lane == 0 ? 1u : 0u;
                }
            }
            q = qn;
            rec = recn;
            c = next;
        } while (u != 0);
    }

    if (nw > 1) {   // uniform
        if (wv > 0) {
#pragma unroll
            for (int k = 0; k < S::N; ++k)
                part[((wv - 1) * S::N + k) * 64 + t.lane] = make_float2(C[k], __int_as_float(terms[k]));
        }
        __syncthreads();
        if (wv == 0) {
            for (int w = 0; w < nw - 1; ++w) {
#pragma unroll
                for (int k = 0; k < S::N; ++k) {
                    const float2 p = part[(w * S::N + k) * 64 + t.lane];
                    C[k] += p.x;
                    terms[k] += __float_as_int(p.y);
                }
            }
        }
    }
    if (wv == 0) {
#pragma unroll
        for (int k = 0; k < S::N; ++k) {
            if (t.in(k)) {
                const int64_t idx = (int64_t)t.y(k) * t.vi->width + t.x(k);
                const int64_t pidx = t.vi->pix_off + idx;
                const float y = C[k] * t.unit(k);
                t.vi->out[idx] = y * kLn2;
                b.T_final[pidx] = fast_exp2(-y);
                b.last_id[pidx] = terms[k];
            }
        }
    }
    if (COUNT) add_counts(b.counters, n);
    if (timed && threadIdx.x == 0)
        b.wg_time[blockIdx.x] = make_uint2(cu_key(), (uint32_t)(wg_clock() - t_start));
}

// One wave's LDS in the backward.
template <int N, int NSLOT>
struct BwdWave {
    static constexpr int kAcc = NSLOT == 16 ? 17 : 11;   // odd: rows on different banks
    uint32_t queue[N][128];    // entries that reach slot k and have not run
    float2 pix[N][64];         // dL/dx x / y, least sure y / |u|
    float acc[64 * kAcc];
    uint32_t item[64];
};

// Five waves per SIMD: left alone the compiler takes four (64 views of 16x16 tiles 2 %
// slower, 16x8 tiles 8 %).
template <int TW, int TH, int MODE, bool COUNT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(5))) void xray_bwd_kernel(
    RenderParams rp, Buffers b)
{
    using S = Slots<TW, TH>;
    constexpr bool NEAR = Kind<MODE>::NEAR, EPAN = Kind<MODE>::EPAN;
    constexpr bool PLAIN = !NEAR && !EPAN;
    constexpr int NSLOT = NEAR ? 16 : 10;
    using Wave = BwdWave<S::N, NSLOT>;
    extern __shared__ __align__(16) unsigned char lds[];
    const bool timed = b.wg_time != nullptr;   // uniform
    const uint64_t t_start = timed ? wg_clock() : 0;
    const int gt = (int)b.tile_order[blockIdx.x];
    const TileWave<TW, TH> t(rp, b, gt);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    Wave &st = reinterpret_cast<Wave *>(lds)[wv];
    const uint2 range = b.ranges[gt];
    const float zn = t.vi->znear, tau2 = rp.tau2;
    const int lane = t.lane;
    XrayCounts n;
    for (int k = 0; k < S::N; ++k) {
        const float un = t.unit(k);
        const float dL = t.in(k) ? t.vi->dL[(int64_t)t.y(k) * t.vi->width + t.x(k)] : 0.0f;
        st.pix[k][lane] = make_float2(dL * (kLn2 * un), tau2 / un * (1.0f + kTie));
    }

    // The first cnt entries of slot k's queue over its pixels.
    auto run = [&](int k, int cnt) {
        lds_wave_sync();
        const uint32_t it = st.queue[k][lane < cnt ? lane : 0];
        const float4 *gp = b.geom + (size_t)it * kRecVec;
        const float4 h = gp[0], r = gp[1], s = gp[2];
        const float E = EPAN ? s.w : s.w * (2.0f / kLog2e);
        float V = 0.0f, mz = 0.0f;
        if constexpr (NEAR) {
            const float4 g5 = gp[5];
            V = length_v0(gp[4], g5);
            mz = g5.w;
        }
        const int nx = min(kRegion, t.vi->width - t.slot_x(k));
        const int ny = min(kRegion, t.vi->height - t.slot_y(k));
        float dx[kRegion];
#pragma unroll
        for (int x = 0; x < kRegion; ++x) dx[x] = ((float)(t.slot_x(k) + x) + 0.5f - h.x) - h.z;
        // PLAIN: sums of T and (1 - D^2) T times a0^2, a0 a1, a1^2, a0 w2, a1 w2; else
        // the slots themselves
        float acc[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
        // A pair's geometry, D^2 (scaled, unless EPAN) and y / |u|.
        struct Term {
            RayPair g;
            float hp, d2, yy, hh, hn;   // hh, hn: as in raster_quad.hip
        };
        auto term = [&](float dxx, float a0r, float a1, float a1sq, float wr) {
            Term m;
            m.g = ray_pair(__fmaf_rn(r.x, dxx, a0r), a1, a1sq, __fmaf_rn(s.x, dxx, wr));
            m.hp = m.g.h * m.g.rq2;
            m.d2 = s.w * m.hp;   // (log2 e / 2) D^2, or D^2 (EPAN)
            float ex;
            if constexpr (EPAN) ex = epan_ray(m.d2);
            else ex = fast_exp2(-m.d2);
            m.yy = (NEAR ? fabsf(s.z) : s.z) * (m.g.rq * ex);
            m.hh = m.hn = 0.0f;
            if constexpr (NEAR) {
                if (s.z < 0.0f) {
                    float zw;
                    const float eta = ray_eta(V, mz, m.g, zn, zw);
                    const float Phi = norm_cdf(eta);
                    m.yy *= Phi;
                    m.hh = Phi > 1e-30f ? 0.39894228f * fast_exp2(-0.72134752f * eta * eta) / Phi : -eta;
                    m.hn = m.hh * __fmaf_rn(2.0f, zw, eta);
                }
            }
            return m;
        };
        // PLAIN: a row's sums, whose factors a1 and a1^2 come in at its end.
        struct Row {
            float S0 = 0.0f, S1 = 0.0f, SW = 0.0f, L0 = 0.0f, L1 = 0.0f, LW = 0.0f;
        };
        // tt: dL/d(ln x)
        auto add = [&](Row &q, const Term &m, float tt) {
            const RayPair &g = m.g;
            acc[9] += tt;
            if constexpr (PLAIN) {
                const float T = tt * g.rq2;
                const float L = T * __fmaf_rn(m.d2, -2.0f / kLog2e, 1.0f);
                const float T0 = T * g.a0, La = L * g.a0;
                q.S0 += T;
                q.S1 += T0;
                q.SW = __fmaf_rn(T, g.w2, q.SW);
                acc[0] = __fmaf_rn(T0, g.a0, acc[0]);
                acc[3] = __fmaf_rn(T0, g.w2, acc[3]);
                q.L0 += L;
                q.L1 += La;
                q.LW = __fmaf_rn(L, g.w2, q.LW);
                acc[5] = __fmaf_rn(La, g.a0, acc[5]);
                acc[8] = __fmaf_rn(La, g.w2, acc[8]);
            } else {
                // weights of p p^T (tw) and of the z terms (tz)
                const float D2 = EPAN ? m.d2 : m.d2 * (2.0f / kLog2e);
                const float p0 = g.a0 * g.rq, p1 = g.a1 * g.rq, p2 = g.w2 * g.rq;
                float tw = tt, tz = tt;
                if constexpr (EPAN) tz = tt != 0.0f ? tt * (3.0f * fast_rcp(1.0f - D2)) : 0.0f;
                if constexpr (NEAR) {
                    tw = __fmaf_rn(tt, m.hn, tt);
                    const float th = tt * m.hh;
                    acc[13] = __fmaf_rn(th, p0, acc[13]);
                    acc[14] = __fmaf_rn(th, p1, acc[14]);
                    acc[15] = __fmaf_rn(th, p2, acc[15]);
                }
                const float kp = __fmaf_rn(tz, E - D2, tw), kq = __fmaf_rn(-tz, D2, tw);
                const float z0 = tz * p0, z1 = tz * p1, zh = tz * m.hp;
                acc[0] = __fmaf_rn(kp * p0, p0, acc[0]);
                acc[1] = __fmaf_rn(kp * p0, p1, acc[1]);
                acc[2] = __fmaf_rn(kq * p0, p2, acc[2]);
                acc[3] = __fmaf_rn(kp * p1, p1, acc[3]);
                acc[4] = __fmaf_rn(kq * p1, p2, acc[4]);
                acc[5] += __fmaf_rn(-tw, p2 * p2, __fmaf_rn(-zh, D2, tt));   // sum t - M_22
                acc[6] = __fmaf_rn(z0, p2, acc[6]);
                acc[7] = __fmaf_rn(z1, p2, acc[7]);
                acc[8] += zh;
            }
        };
        auto end_row = [&](const Row &q, float a1, float a1sq) {
            if constexpr (PLAIN) {
                acc[1] = __fmaf_rn(q.S1, a1, acc[1]);
                acc[2] = __fmaf_rn(q.S0, a1sq, acc[2]);
                acc[4] = __fmaf_rn(q.SW, a1, acc[4]);
                acc[6] = __fmaf_rn(q.L1, a1, acc[6]);
                acc[7] = __fmaf_rn(q.L0, a1sq, acc[7]);
                acc[10] = __fmaf_rn(q.LW, a1, acc[10]);
            }
        };
        uint64_t tied = 0;   // bit 8 y + x: a pair within kTie of the cut (uniform)
        for (int y = 0; y < ny; ++y) {
            const float dy = ((float)(t.slot_y(k) + y) + 0.5f - h.y) - h.w;
            const float a0r = r.y * dy, a1 = r.z * dy, a1sq = a1 * a1;
            const float wr = __fmaf_rn(s.y, dy, 1.0f);
            const float2 *px = &st.pix[k][y * kRegion];
            Row q;
            uint32_t cols = 0;
#pragma unroll
            for (int x = 0; x < kRegion; ++x) {
                if (x >= nx) break;   // uniform
                const float2 gc = px[x];
                const Term m = term(dx[x], a0r, a1, a1sq, wr);
                const uint64_t on = __builtin_amdgcn_ballot_w64(m.yy > gc.y);
                const uint64_t may = __builtin_amdgcn_ballot_w64(!(m.yy < gc.y * kMost));
                cols |= on != may ? 1u << x : 0u;
                add(q, m, __builtin_amdgcn_inverse_ballot_w64(on) ? m.yy * gc.x : 0.0f);
                if (COUNT) {
                    n.full += lane < cnt ? 1u : 0u;
                    n.blend += m.yy > gc.y && lane < cnt ? 1u : 0u;
                }
            }
            tied |= (uint64_t)cols << (8 * y);
            end_row(q, a1, a1sq);
        }
        // their pairs, left out above, as the forward decides them
        while (__builtin_expect(tied != 0, 0)) {
            const int e = __builtin_ctzll(tied), x = t.slot_x(k) + (e & 7), y = t.slot_y(k) + (e >> 3);
            tied &= tied - 1;
            const float dxx = ((float)x + 0.5f - h.x) - h.z, dy = ((float)y + 0.5f - h.y) - h.w;
            const float a1 = r.z * dy, a1sq = a1 * a1;
            const Term m = term(dxx, r.y * dy, a1, a1sq, __fmaf_rn(s.y, dy, 1.0f));
            const float2 gc = st.pix[k][e];
            const float yl = lframe_y<MODE>(gp[3], gp[4], gp[5], dxx, dy, t.unit(x, y), zn);
            const bool on = !(m.yy < gc.y * kMost) && !(m.yy > gc.y) && !(yl < tau2);
            Row q;
            add(q, m, on ? m.yy * gc.x : 0.0f);
            end_row(q, a1, a1sq);
            if (COUNT) n.blend += on && lane < cnt ? 1u : 0u;
        }
        float out[NSLOT];
        if constexpr (PLAIN) {
            out[0] = __fmaf_rn(E, acc[0], acc[5]);
            out[1] = __fmaf_rn(E, acc[1], acc[6]);
            out[2] = acc[8];
            out[3] = __fmaf_rn(E, acc[2], acc[7]);
            out[4] = acc[10];
            out[5] = acc[5] + acc[7];
            out[6] = acc[3];
            out[7] = acc[4];
            out[8] = acc[0] + acc[2];
            out[9] = acc[9];
        } else {
#pragma unroll
            for (int e = 0; e < NSLOT; ++e) out[e] = acc[e];
        }
        st.item[lane] = it;
#pragma unroll
        for (int e = 0; e < NSLOT; ++e) st.acc[lane * Wave::kAcc + e] = out[e];
        lds_wave_sync();
        const int f = lane & 15;
        if (f < NSLOT) {
            for (int at = lane >> 4; at < cnt; at += 4) {
                const float sum = st.acc[at * Wave::kAcc + f];
                if (sum != 0.0f)
                    atomicAdd(reinterpret_cast<float *>(b.rgrad) + (size_t)st.item[at] * kGradFloats + f, sum);
            }
        }
        if (COUNT) n.visits_full += lane == 0 ? (uint32_t)cnt : 0u;
    };

    Candidate cand;
    uint32_t waiting = 0;   // 8 bits per slot: entries in its queue
    const uint64_t below = (1ull << lane) - 1ull;
    const uint32_t first = range.x + 64u * (uint32_t)wv, step = 64u * (uint32_t)nw;
    cand.load(b, range, first + lane);
    for (uint32_t bs = first; bs < range.y; bs += step) {
        const uint32_t j = bs + lane;
        const Candidate cur = cand;
        cand.load(b, range, j + step);
        for (int k = 0; k < S::N; ++k) {
            if (!t.any(k)) continue;   // uniform
            const uint64_t on = __builtin_amdgcn_ballot_w64(
                j < range.y &&
                reaches<kRegion>(cur.c6, cur.c7, (float)t.slot_x(k), (float)t.slot_y(k)));
            int w = (int)((waiting >> (8 * k)) & 255u);   // < 64
            if (__builtin_amdgcn_inverse_ballot_w64(on))
                st.queue[k][w + __builtin_popcountll(on & below)] = cur.item;
            w += __builtin_popcountll(on);
            if (COUNT) n.visits += lane == 0 ? min(64u, range.y - bs) : 0u;
            if (w >= 64) {
                run(k, 64);
                w -= 64;
                const uint32_t rest = st.queue[k][64 + lane];
                lds_wave_sync();
                if (lane < w) st.queue[k][lane] = rest;
            }
            waiting = (waiting & ~(255u << (8 * k))) | ((uint32_t)w << (8 * k));
        }
    }
    for (int k = 0; k < S::N; ++k) {
        const int w = (int)((waiting >> (8 * k)) & 255u);
        if (w > 0) run(k, w);
    }
    if (COUNT) add_counts(b.counters + 8, n);
    if (timed) {
        __syncthreads();
        if (threadIdx.x == 0)
            b.wg_time[rp.total_tiles + blockIdx.x] =
                make_uint2(cu_key(), (uint32_t)(wg_clock() - t_start));
    }
}

// Waves per tile: doubled while a launch has no more than `few` waves, at most 8 (4 for
// four slots: LDS).  Forward / backward us with 8x8 tiles at 1, 2, 4, 8 waves a tile:
//   12 x 160x160, 8k Gaussians   78 / 81   57 / 70   50 / 78   63 / 95
//   8 x 256x256, 60k            411 / 361  304 / 329  294 / 346  336 / 411
int xray_waves(const RenderParams &rp, bool fwd)
{
    const int most = rp.tile_w * rp.tile_h >= 4 * kRegion * kRegion ? 4 : 8;
    const int64_t few = fwd ? 16384 : 8192;
    int s = 1;
    while (s < most && (int64_t)rp.total_tiles * s <= few) s *= 2;
    return s;
}

template <int TW, int TH, int MODE>
hipError_t launch_shape(const RenderParams &rp, const Buffers &b, bool fwd, bool count, hipStream_t s)
{
    const int nw = xray_waves(rp, fwd);
    const dim3 grid(rp.total_tiles), block(64 * nw);
    constexpr int N = Slots<TW, TH>::N;
    const size_t lds = fwd ? (size_t)(nw - 1) * N * 64 * sizeof(float2)
                           : nw * sizeof(BwdWave<N, Kind<MODE>::NEAR ? 16 : 10>);
    if (fwd && count) xray_fwd_kernel<TW, TH, MODE, true><<<grid, block, lds, s>>>(rp, b);
    else if (fwd) xray_fwd_kernel<TW, TH, MODE, false><<<grid, block, lds, s>>>(rp, b);
    else if (count) xray_bwd_kernel<TW, TH, MODE, true><<<grid, block, lds, s>>>(rp, b);
    else xray_bwd_kernel<TW, TH, MODE, false><<<grid, block, lds, s>>>(rp, b);
    return hipGetLastError();
}

template <int TW, int TH>
hipError_t launch_mode(const RenderParams &rp, const Buffers &b, bool fwd, bool count, hipStream_t s)
{
    if (rp.kernel == VGR_KERNEL_EPANECHNIKOV)
        return launch_shape<TW, TH, kModeXrayEpan>(rp, b, fwd, count, s);
    if (rp.near_segment) return launch_shape<TW, TH, kModeXrayNear>(rp, b, fwd, count, s);
    return launch_shape<TW, TH, VGR_MODE_XRAY>(rp, b, fwd, count, s);
}

}  // namespace

hipError_t launch_xray(const RenderParams &rp, const Buffers &b, bool fwd, bool count, hipStream_t s)
{
    if (rp.tile_w == 8 && rp.tile_h == 8) return launch_mode<8, 8>(rp, b, fwd, count, s);
    if (rp.tile_w == 16 && rp.tile_h == 8) return launch_mode<16, 8>(rp, b, fwd, count, s);
    if (rp.tile_w == 32 && rp.tile_h == 8) return launch_mode<32, 8>(rp, b, fwd, count, s);
    return launch_mode<16, 16>(rp, b, fwd, count, s);
}

}  // namespace vgr
