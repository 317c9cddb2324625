// Device-wide exclusive scan and stable LSD radix sort of (u32 key, u32 value)
// pairs, written for wave64 gfx950.  The rasteriser uses them to order the
// (tile, depth) instance lists: the compositing assumes the Gaussians sorted
// front to back (Sec. 3.2), and the tile rasteriser sorts them per tile rather
// than per pixel (Sec. 7, Limitations).
//
// Radix pass = histogram kernel + per-digit exclusive scan of the digit-major
// table of per-block counts (one block per digit) + scatter kernel, which adds
// the digit starts (a scan of the 256 digit totals) itself.  The scatter ranks
// keys stably inside a tile of 1024, 2048 or 4096 keys (keys_per_thread): each wave owns
// a quarter of them, consecutive, ranks 64 keys at a time by matching digits with one
// ballot per digit bit, and keeps running per-digit counters in LDS.  The tile is then reordered by
// digit in LDS and written out run by run, so that neighbouring threads write
// neighbouring addresses.  Up to kOneMax pairs are sorted by one workgroup in one
// launch.
#include "block_scan.h"
#include "vgr_internal.h"

namespace vgr {

namespace {

constexpr int kThreads = 256;
constexpr int kItems = 16;
constexpr int kTile = kThreads * kItems;   // 4096
static_assert(kTile % kScanGrain == 0, "scan grain");
constexpr int kWaves = kThreads / 64;

__device__ inline uint32_t wave_inclusive_scan(uint32_t v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t t = __shfl_up(v, d, 64);
        if (lane >= d) v += t;
    }
    return v;
}

// Exclusive scan across the 256 threads of a block; *total gets the sum.
__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t *total)
{
    __shared__ uint32_t wsum[kWaves];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t inc = wave_inclusive_scan(v);
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
        uint32_t s = wsum[i];
        off += (i < w) ? s : 0u;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

// Single block: exclusive scan of the nb block sums in place (94k sums: 103 -> 26 us).
// With d_total, the total is also the instance count K: d_total[0] = K
// clamped to capacity, d_total[1] = overflow, d_total[5] set (sticky) on
// overflow, d_total[7] = 0 (the emission's mismatch counter).
template <int T>
__global__ __launch_bounds__(T) void scan_partials_kernel(uint32_t *__restrict__ partial, int64_t nb,
                                                          uint32_t *__restrict__ total_out,
                                                          uint32_t *__restrict__ d_total,
                                                          int64_t capacity)
{
    const uint32_t total = scan_in_place<T>(partial, nb);
    if (threadIdx.x == 0 && total_out) *total_out = total;
    if (threadIdx.x == 0 && d_total) {
        const bool over = (int64_t)total > capacity;
        d_total[0] = over ? (uint32_t)capacity : total;
        d_total[1] = over ? 1u : 0u;
        if (over) d_total[5] = 1u;   // sticky until the host clears it
        d_total[7] = 0u;
    }
}

// Also the first item of each wave of the emission (EmitSplit).
__global__ __launch_bounds__(kThreads) void scan_down_kernel(const uint32_t *__restrict__ in,
                                                             uint32_t *__restrict__ out,
                                                             int64_t n,
                                                             const uint32_t *__restrict__ partial,
                                                             uint32_t *__restrict__ starts,
                                                             EmitSplit split)
{
    __shared__ uint32_t tile[kTile];
    const int64_t base = (int64_t)blockIdx.x * kTile;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        int64_t idx = base + (int64_t)i * kThreads + threadIdx.x;
        tile[i * kThreads + threadIdx.x] = idx < n ? in[idx] : 0u;
    }
    __syncthreads();
    uint32_t v[kItems];
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        v[i] = tile[threadIdx.x * kItems + i];
        s += v[i];
    }
    uint32_t total;
    uint32_t off = block_exclusive_scan(s, &total) + partial[blockIdx.x * (kTile / kScanGrain)];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        tile[threadIdx.x * kItems + i] = off;
        off += v[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        int64_t idx = base + (int64_t)i * kThreads + threadIdx.x;
        if (idx < n) out[idx] = tile[i * kThreads + threadIdx.x];
    }
    // A wave of the emission begins with its group's first item, or with the item that
    // holds the instance at its cut; a cut at the group's end names the last item.
    // (Short loops: unrolled ones cost more in instruction fetches than they save.)
    auto put = [&](uint32_t i, uint32_t cut) {
        const uint32_t w = (uint32_t)((base + i) >> split.lg_items) + cut;
        if (w < split.waves) starts[w] = (uint32_t)base + i;
    };
    const uint32_t b0 = tile[0], b1 = b0 + total;
    const uint32_t nb = (uint32_t)min((int64_t)kTile, n - base);
    const uint32_t cmask = (1u << split.lg) - 1u;
    for (uint32_t i0 = threadIdx.x << split.lg_items; i0 < nb; i0 += kThreads << split.lg_items) {
        const uint32_t i1 = min(i0 + (1u << split.lg_items), nb);
        const uint32_t end = i1 < (uint32_t)kTile ? tile[i1] : b1;
        put(i0, tile[i0] >> split.lg);
        if ((end & cmask) == 0) put(i1 - 1u, end >> split.lg);
    }
    for (uint64_t x = (((uint64_t)b0 + cmask) >> split.lg) + threadIdx.x; x << split.lg < b1; x += kThreads) {
        // the last item that does not start behind the cut
        uint32_t lo = 0, hi = nb - 1u;
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1u) >> 1;
            if (tile[mid] <= x << split.lg) lo = mid;
            else hi = mid - 1u;
        }
        put(lo, (uint32_t)x);
    }
}

// ---------------------------------------------------------------- radix ---

// Whole tiles of aligned keys are read four at a time, all loads in flight before the
// first count (15.8M keys: 24.6 -> 19.9 us).
template <int IPT>
__global__ __launch_bounds__(kThreads) void radix_hist_kernel(const uint32_t *__restrict__ keys,
                                                              const uint32_t *__restrict__ d_n,
                                                              int shift, uint32_t mask,
                                                              uint32_t *__restrict__ hist, int stride)
{
    __shared__ uint32_t h[kWaves][256];
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) h[k][threadIdx.x] = 0;
    __syncthreads();
    const int64_t n = *d_n;
    const int64_t base = (int64_t)blockIdx.x * (kThreads * IPT);
    if (base + kThreads * IPT <= n && ((uintptr_t)keys & 15) == 0) {   // uniform
        uint4 k[IPT / 4];
#pragma unroll
        for (int i = 0; i < IPT / 4; ++i)
            k[i] = reinterpret_cast<const uint4 *>(keys + base)[i * kThreads + (int)threadIdx.x];
#pragma unroll
        for (int i = 0; i < IPT / 4; ++i) {
            atomicAdd(&h[w][(k[i].x >> shift) & mask], 1u);
            atomicAdd(&h[w][(k[i].y >> shift) & mask], 1u);
            atomicAdd(&h[w][(k[i].z >> shift) & mask], 1u);
            atomicAdd(&h[w][(k[i].w >> shift) & mask], 1u);
        }
    } else if (base < n) {
#pragma unroll 4
        for (int i = 0; i < IPT; ++i) {
            int64_t idx = base + (int64_t)i * kThreads + threadIdx.x;
            if (idx < n) atomicAdd(&h[w][(keys[idx] >> shift) & mask], 1u);
        }
    }
    __syncthreads();
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) s += h[k][threadIdx.x];
    hist[(int64_t)threadIdx.x * stride + blockIdx.x] = s;
}

// One block per digit: exclusive scan, in place, of that digit's row of the
// digit-major table (the per-block counts), and the row total into tot[d].  (3.9k
// entries a row: 8.2 -> 5.2 us.)
__global__ __launch_bounds__(kThreads) void radix_rowscan_kernel(uint32_t *__restrict__ table,
                                                                 int nb, int stride,
                                                                 uint32_t *__restrict__ tot)
{
    const uint32_t total = scan_in_place<kThreads>(table + (int64_t)blockIdx.x * stride, nb);
    if (threadIdx.x == 0) tot[blockIdx.x] = total;
}

template <int IPT>
__global__ __launch_bounds__(kThreads) void radix_scatter_kernel(
    const uint32_t *__restrict__ keys, const uint32_t *__restrict__ vals,
    uint32_t *__restrict__ keys_out, uint32_t *__restrict__ vals_out,
    const uint32_t *__restrict__ d_n, int shift, int dbits, const uint32_t *__restrict__ offs,
    const uint32_t *__restrict__ tot, int stride)
{
    __shared__ uint32_t cnt[kWaves][256];
    __shared__ uint32_t gdelta[256];   // global start minus block-local start
    constexpr int TILE = kThreads * IPT;
    __shared__ uint32_t sk[TILE], sv[TILE];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t mask = (1u << dbits) - 1u;
    const int64_t n = *d_n;
    const int64_t blk_base = (int64_t)blockIdx.x * TILE;
    if (blk_base >= n) return;   // uniform across the block
    // start of each digit = exclusive scan of the digit totals
    uint32_t tot_all;
    const uint32_t digit_start = block_exclusive_scan(tot[threadIdx.x], &tot_all);
#pragma unroll
    for (int k = 0; k < kWaves; ++k) cnt[k][threadIdx.x] = 0;
    __syncthreads();

    const int64_t wbase = blk_base + (int64_t)w * (TILE / kWaves);
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t k[IPT], v[IPT], r[IPT];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        int64_t idx = wbase + i * 64 + lane;
        bool valid = idx < n;
        k[i] = valid ? keys[idx] : 0u;
        v[i] = valid ? vals[idx] : 0u;
    }
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        int64_t idx = wbase + i * 64 + lane;
        bool valid = idx < n;
        uint32_t d = (k[i] >> shift) & mask;
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < dbits; ++b) {
            bool bit = (d >> b) & 1u;
            uint64_t bal = __ballot(bit);
            peers &= bit ? bal : ~bal;
        }
        uint32_t below = (uint32_t)__popcll(peers & lt_mask);
        uint32_t prev = valid ? cnt[w][d] : 0u;
        r[i] = prev + below;
        if (valid && below == 0) cnt[w][d] = prev + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    {
        // per digit: block-local start (scan over digits of the block's counts),
        // then each wave's start inside it; global start from the digit-major
        // table of block offsets
        const int d = threadIdx.x;
        uint32_t c_d = 0;
#pragma unroll
        for (int k2 = 0; k2 < kWaves; ++k2) c_d += cnt[k2][d];
        uint32_t blk_count;
        const uint32_t ls = block_exclusive_scan(c_d, &blk_count);
        gdelta[d] = digit_start + offs[(int64_t)d * stride + blockIdx.x] - ls;
        uint32_t run = ls;
#pragma unroll
        for (int k2 = 0; k2 < kWaves; ++k2) {
            uint32_t c = cnt[k2][d];
            cnt[k2][d] = run;
            run += c;
        }
    }
    __syncthreads();
    // reorder the tile by digit in LDS ...
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        int64_t idx = wbase + i * 64 + lane;
        if (idx < n) {
            uint32_t d = (k[i] >> shift) & mask;
            uint32_t lp = cnt[w][d] + r[i];
            sk[lp] = k[i];
            sv[lp] = v[i];
        }
    }
    __syncthreads();
    // ... and write it out in order: consecutive threads write consecutive
    // positions of the same digit run
    const int64_t cnt_blk = min((int64_t)TILE, n - blk_base);
    for (int e = threadIdx.x; e < cnt_blk; e += kThreads) {
        const uint32_t key = sk[e];
        const uint32_t d = (key >> shift) & mask;
        const uint32_t pos = gdelta[d] + (uint32_t)e;
        keys_out[pos] = key;
        vals_out[pos] = sv[e];
    }
}

// A sort of up to kOneMax pairs by one workgroup: every pass ranks as the scatter does
// (wave w owns 64 R consecutive keys, R rounds of 64) and exchanges the tile through
// LDS, keys and values in turn.  A pass skips the exchange if one digit has every key.
// Sorts this small are bound by their launches (three a pass) and by the passes' serial
// steps, not by the keys.  32 bits with the compaction before, many workgroups and one:
// 1k items 52 and 22 us, 4k 59 and 28, 8k 59 and 40, 12k 58 and 68.
constexpr int kOneThreads = 1024, kOneItems = 8;
constexpr int kOneMax = kOneThreads * kOneItems;

__global__ __launch_bounds__(kOneThreads) void radix_one_kernel(uint32_t *__restrict__ keys,
                                                                uint32_t *__restrict__ vals,
                                                                const uint32_t *__restrict__ d_n,
                                                                int bits, int passes)
{
    constexpr int W = kOneThreads / 64;
    __shared__ uint16_t cnt[W][256];
    __shared__ uint32_t tile[kOneMax];
    __shared__ uint32_t wsum[4], s_one;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int n = (int)min(*d_n, (uint32_t)kOneMax);
    const int rounds = (n + kOneThreads - 1) / kOneThreads;   // uniform
    const int base = w * 64 * rounds + lane;
    const uint64_t below = (1ull << lane) - 1ull;
    uint32_t k[kOneItems], v[kOneItems], r[kOneItems];
#pragma unroll
    for (int i = 0; i < kOneItems; ++i) {
        if (i >= rounds) break;   // uniform
        const int at = base + i * 64;
        k[i] = at < n ? keys[at] : 0u;
        v[i] = at < n ? vals[at] : 0u;
    }
    int shift = 0;
    for (int p = 0; p < passes; ++p) {
        const int dbits = (bits - shift + (passes - p) - 1) / (passes - p);
        const uint32_t mask = (1u << dbits) - 1u;
        for (int e = (int)threadIdx.x; e < W * 256; e += kOneThreads) (&cnt[0][0])[e] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kOneItems; ++i) {
            if (i >= rounds) break;   // uniform
            const bool valid = base + i * 64 < n;
            const uint32_t d = (k[i] >> shift) & mask;
            uint64_t peers = __ballot(valid);
            for (int b = 0; b < dbits; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t bal = __ballot(bit);
                peers &= bit ? bal : ~bal;
            }
            const uint32_t ahead = (uint32_t)__popcll(peers & below);
            const uint32_t prev = valid ? cnt[w][d] : 0u;
            r[i] = prev + ahead;
            if (valid && ahead == 0) cnt[w][d] = (uint16_t)(prev + (uint32_t)__popcll(peers));
        }
        __syncthreads();
        // per digit (threads 0..255): start of its keys, then of each wave's
        uint32_t c_d = 0, inc = 0;
        if (threadIdx.x < 256) {
#pragma unroll
            for (int q = 0; q < W; ++q) c_d += cnt[q][threadIdx.x];
            inc = wave_inclusive_scan(c_d);
            if (lane == 63) wsum[w] = inc;
            if (threadIdx.x == 0) s_one = 0u;
        }
        __syncthreads();
        if (threadIdx.x < 256) {
            uint32_t run = inc - c_d;
            for (int q = 0; q < w; ++q) run += wsum[q];
            if (c_d == (uint32_t)n) s_one = 1u;
#pragma unroll
            for (int q = 0; q < W; ++q) {
                const uint32_t c = cnt[q][threadIdx.x];
                cnt[q][threadIdx.x] = (uint16_t)run;
                run += c;
            }
        }
        __syncthreads();
        if (s_one == 0u) {   // uniform
#pragma unroll
            for (int i = 0; i < kOneItems; ++i) {
                if (i >= rounds) break;   // uniform
                r[i] += cnt[w][(k[i] >> shift) & mask];
                if (base + i * 64 < n) tile[r[i]] = k[i];
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kOneItems; ++i) {
                if (i >= rounds) break;   // uniform
                if (base + i * 64 < n) k[i] = tile[base + i * 64];
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kOneItems; ++i) {
                if (i >= rounds) break;   // uniform
                if (base + i * 64 < n) tile[r[i]] = v[i];
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kOneItems; ++i) {
                if (i >= rounds) break;   // uniform
                if (base + i * 64 < n) v[i] = tile[base + i * 64];
            }
        }
        __syncthreads();   // the next pass rewrites cnt, s_one and tile
        shift += dbits;
    }
#pragma unroll
    for (int i = 0; i < kOneItems; ++i) {
        if (i >= rounds) break;   // uniform
        const int at = base + i * 64;
        if (at < n) {
            keys[at] = k[i];
            vals[at] = v[i];
        }
    }
}

__global__ void copy_pairs_kernel(const uint32_t *__restrict__ k, const uint32_t *__restrict__ v,
                                  uint32_t *__restrict__ ko, uint32_t *__restrict__ vo,
                                  const uint32_t *__restrict__ d_n, int64_t bound)
{
    const int64_t n = *d_n;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n && i < bound;
         i += (int64_t)gridDim.x * blockDim.x) {
        ko[i] = k[i];
        vo[i] = v[i];
    }
}

inline int64_t blocks_for(int64_t n) { return (n + kTile - 1) / kTile; }

}  // namespace

int64_t scan_tmp_words(int64_t n)
{
    return (n + kScanGrain - 1) / kScanGrain + 1;
}

hipError_t launch_count_scan(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *tmp,
                             uint32_t *d_total, int64_t capacity, uint32_t *starts,
                             const EmitSplit &split, hipStream_t s)
{
    const int64_t ng = n > 0 ? (n + kScanGrain - 1) / kScanGrain : 0;
    // (one round of 256 threads, else many threads)
    if (ng <= kScanShort)
        scan_partials_kernel<kThreads><<<1, kThreads, 0, s>>>(tmp, ng, out + (n > 0 ? n : 0), d_total,
                                                              capacity);
    else
        scan_partials_kernel<kScanThreads><<<1, kScanThreads, 0, s>>>(tmp, ng, out + n, d_total,
                                                                      capacity);
    if (n > 0)
        scan_down_kernel<<<dim3((unsigned)blocks_for(n)), dim3(kThreads), 0, s>>>(in, out, n, tmp,
                                                                                 starts, split);
    return hipGetLastError();
}

// Keys per thread of a radix pass: 4 (1024-key tiles) up to 1M keys, so that small sorts
// still spread over all CUs, 8 up to 8M, then 16: a digit's run of a tile leaves as one
// piece, 16 bytes of a 1024-key tile on average.
// Depth sort and compaction at 4 and 8: 3M items (1.5M of them with instances) 177 and
// 143 us, 1.5M a call of two views 149 and 130; 0.8M instances 146 and 153 (too few
// blocks).  Tile sort of 4.9M instances at 8 and 16: 100 and 104 us.
constexpr int64_t kSmallSort = 1 << 20, kMediumSort = 1 << 23;
inline int keys_per_thread(int64_t n) { return n <= kSmallSort ? 4 : (n <= kMediumSort ? 8 : kItems); }

// Words between two digits' rows of the table: rows start at 16 bytes.
inline int64_t row_stride(int64_t nb) { return (nb + 3) & ~(int64_t)3; }

inline int64_t radix_blocks(int64_t n, int ipt) { return (n + kThreads * ipt - 1) / (kThreads * ipt); }

// Enough for a sort of any n <= n_bound (a smaller sort may use the smaller
// tiles and so more blocks).
int64_t radix_tmp_words(int64_t n_bound)
{
    const int64_t n = n_bound > 0 ? n_bound : 1;
    int64_t nb = radix_blocks(n, keys_per_thread(n));
    for (int64_t top : { kSmallSort, kMediumSort }) {
        const int64_t m = n < top ? n : top;
        const int64_t k = radix_blocks(m, keys_per_thread(m));
        nb = k > nb ? k : nb;
    }
    return 256 * row_stride(nb) + 256;
}

int radix_passes(int64_t n_bound, int bits)
{
    return n_bound <= kOneMax ? 0 : (bits + 7) / 8;
}

hipError_t launch_radix_sort(uint32_t *keys, uint32_t *vals, uint32_t *keys2, uint32_t *vals2,
                             const uint32_t *d_n, int64_t n_bound, int bits, uint32_t *tmp,
                             bool stay, hipStream_t s)
{
    if (n_bound <= 0 || bits <= 0) return hipSuccess;
    if (n_bound <= kOneMax) {
        radix_one_kernel<<<1, kOneThreads, 0, s>>>(keys, vals, d_n, bits, (bits + 7) / 8);
        return hipGetLastError();
    }
    const int ipt = keys_per_thread(n_bound);
    const int64_t nb = radix_blocks(n_bound, ipt);
    const int64_t table = 256 * row_stride(nb);
    uint32_t *hist = tmp;            // digit-major per-block counts, then their row scans
    uint32_t *tot = tmp + table;     // per-digit totals
    const int passes = radix_passes(n_bound, bits);
    // spread the bits evenly over the passes (each at most 8)
    int shift = 0;
    uint32_t *ki = keys, *vi = vals, *ko = keys2, *vo = vals2;
    for (int p = 0; p < passes; ++p) {
        const int dbits = (bits - shift + (passes - p) - 1) / (passes - p);
        const uint32_t mask = (1u << dbits) - 1u;
        const dim3 g((unsigned)nb), t(kThreads);
        const int stride = (int)row_stride(nb);
#define VGR_IPT(K) (ipt == 4 ? K<4> : (ipt == 8 ? K<8> : K<kItems>))
        VGR_IPT(radix_hist_kernel)<<<g, t, 0, s>>>(ki, d_n, shift, mask, hist, stride);
        radix_rowscan_kernel<<<256, kThreads, 0, s>>>(hist, (int)nb, stride, tot);
        VGR_IPT(radix_scatter_kernel)<<<g, t, 0, s>>>(ki, vi, ko, vo, d_n, shift, dbits, hist, tot, stride);
#undef VGR_IPT
        shift += dbits;
        uint32_t *tt;
        tt = ki; ki = ko; ko = tt;
        tt = vi; vi = vo; vo = tt;
    }
    if (ki != keys && !stay) {
        const int64_t grid = (n_bound + 255) / 256 < 65536 ? (n_bound + 255) / 256 : 65536;
        copy_pairs_kernel<<<dim3((unsigned)grid), 256, 0, s>>>(ki, vi, keys, vals, d_n, n_bound);
    }
    return hipGetLastError();
}

}  // namespace vgr
