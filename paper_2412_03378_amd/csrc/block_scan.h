// Exclusive scan of an array by one workgroup.
#pragma once

#include "vgr_internal.h"

namespace vgr {

namespace {

constexpr int kScanThreads = 1024;
// Longest array that 256 threads scan: one round.  (3k words by 256 and 1024 threads 4.4
// and 5.0 us, 200 words 2.1 and 4.7.)
constexpr int64_t kScanShort = 16 * 256;

// Exclusive scan, in place, of c[0..n) (16-byte aligned) by the T threads of the block;
// returns the total.  A serial chain of rounds, so a round takes 16 T words, four loads
// of four consecutive words a thread, all coalesced and in flight before the round's
// one scan.
template <int T = kScanThreads>
__device__ __forceinline__ uint32_t scan_in_place(uint32_t *__restrict__ c, int64_t n)
{
    constexpr int W = T / 64, Q = 4;
    __shared__ uint32_t wsum[Q][W];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (int64_t base = 0; base < n; base += Q * 4 * T) {   // uniform
        uint4 v[Q];
        uint32_t inc[Q];
        // quarters of the round that hold words (uniform): a short array fills one
        const int nq = (int)min((int64_t)Q, (n - base + 4 * T - 1) / (4 * T));
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (q >= nq) break;
            const int64_t k = base + 4 * ((int64_t)q * T + threadIdx.x);
            if (k + 3 < n) {
                v[q] = *reinterpret_cast<const uint4 *>(c + k);
            } else {
                v[q].x = k < n ? c[k] : 0u;
                v[q].y = k + 1 < n ? c[k + 1] : 0u;
                v[q].z = k + 2 < n ? c[k + 2] : 0u;
                v[q].w = 0u;
            }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (q >= nq) break;
            inc[q] = v[q].x + v[q].y + v[q].z + v[q].w;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t t = __shfl_up(inc[q], d, 64);
                if (lane >= d) inc[q] += t;
            }
            if (lane == 63) wsum[q][w] = inc[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (q >= nq) break;
            uint32_t off = carry;
#pragma unroll
            for (int i = 0; i < W; ++i) {
                const uint32_t s = wsum[q][i];
                off += i < w ? s : 0u;
                carry += s;
            }
            const int64_t k = base + 4 * ((int64_t)q * T + threadIdx.x);
            const uint32_t sum = v[q].x + v[q].y + v[q].z + v[q].w;
            uint4 o;
            o.x = off + inc[q] - sum;
            o.y = o.x + v[q].x;
            o.z = o.y + v[q].y;
            o.w = o.z + v[q].z;
            if (k + 3 < n) {
                *reinterpret_cast<uint4 *>(c + k) = o;
            } else {
                if (k < n) c[k] = o.x;
                if (k + 1 < n) c[k + 1] = o.y;
                if (k + 2 < n) c[k + 2] = o.z;
            }
        }
        __syncthreads();   // the next round rewrites wsum
    }
    return carry;
}

}  // namespace

}  // namespace vgr
