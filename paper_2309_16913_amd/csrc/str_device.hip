// Sort-Tile-Recursive bulk load on the device.
//
// The paper does not say how its trees are built; the library bulk-loads them
// with STR (Leutenegger, Lopez, Edgington 1997).  For a level of c items:
// P = ceil(c / F) nodes and S = ceil(sqrt(P)) vertical slices of S*F items.
// Items are ordered by x-center (ties by item index); the item at x-rank p
// belongs to slice p / (S*F); inside a slice items are ordered by y-center
// (ties by item index); consecutive runs of F items of that packing order
// form the level's nodes (every node full but the last).  The node MBRs are
// the next level's items.  Centers only decide the tree's shape, never a
// result: they are compared as order-preserving integers made from
// 0.5*lo + 0.5*hi with each operation rounded to f32.
//
// The packing order needs no full sort by x, only every item's slice.  By the
// size of the level:
//   large   items are bucketed by x-center on a linear grid; a bucket inside
//           one slice gives its items' slice at once, and only the buckets that
//           straddle a slice boundary are ranked.  The items then move to their
//           slices, and one block sorts each slice by (y, index) with radix
//           passes in its L2.  Straddling buckets too large to rank in LDS
//           (x-centers far from uniform, or all alike) set a flag, and the
//           build runs again with
//   any     stable LSD radix sorts of the whole level: by (y key, index), then
//           by slice from the x-rank;
//   small   (at most 16384 items) both ranks counted directly, every item
//           against every other;
//   top     the levels of at most 1024 items, all in one block.
// 10M rectangles: LSD sorts of every level 3.0 ms, this 1.15.
//
// Final numbering: breadth first from the root; the children of a node are
// stored contiguously in entry order, levels one after another.  pos[l][k]
// is the place of node k of level l (creation order) inside its level; it is
// computed from the root down: the children of the node stored at place g
// start at the sum of the entry counts of the nodes stored before g.
//
// Optionally (RT_BUILD_SORT_LX) the entries of every node are reordered by
// low x before the placement, which moves the children with their entries.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "rt_api_internal.h"

namespace rtk {

// Order-preserving integer of a center.  -0.0 counts as +0.0; a NaN center
// (an item spanning -inf..+inf) counts as larger than every number.
__device__ __forceinline__ uint32_t order_key(float c) {
    if (c != c) return 0xFFFFFFFFu;
    if (c == 0.0f) c = 0.0f;
    const uint32_t u = __float_as_uint(c);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_float(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// center, each operation rounded (no contraction into an fma)
__device__ __forceinline__ float center(float lo, float hi) {
    return __fadd_rn(__fmul_rn(0.5f, lo), __fmul_rn(0.5f, hi));
}
__device__ __forceinline__ uint32_t key_x(const float4 v) { return order_key(center(v.x, v.z)); }
__device__ __forceinline__ uint32_t key_y(const float4 v) { return order_key(center(v.y, v.w)); }

constexpr uint32_t kStrInvalid = 1u;   // build flag: a rectangle is invalid
constexpr uint32_t kStrSkewed = 2u;    // a straddling bucket is too large to rank

// Rectangles checked, and the range of their finite x-centers: bounds[0] =
// ~key of the smallest, bounds[1] = key of the largest (both zero at the start).
__global__ void __launch_bounds__(256)
str_validate(const float4 *__restrict__ r, uint64_t n, uint32_t *__restrict__ flag, uint32_t *__restrict__ bounds) {
    uint32_t bad = 0, lo = 0, hi = 0;
    const uint64_t step = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i0 < n; i0 += 4 * step) {
        float4 x[4];   // four loads in flight
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = r[min(i0 + u * step, n - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float4 v = x[u];
            const bool nan = (v.x != v.x) || (v.y != v.y) || (v.z != v.z) || (v.w != v.w);
            if (nan || !(v.x <= v.z) || !(v.y <= v.w)) bad = 1;
            const float c = center(v.x, v.z);
            if (fabsf(c) <= 3.0e38f) {
                const uint32_t k = order_key(c);
                lo = max(lo, ~k);
                hi = max(hi, k);
            }
        }
    }
    for (int d = 32; d >= 1; d >>= 1) {
        lo = max(lo, (uint32_t)__shfl_xor((int)lo, d));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, d));
    }
    if (bad) atomicOr(flag, kStrInvalid);
    __shared__ uint32_t b[2][4];
    if ((threadIdx.x & 63u) == 0) {
        b[0][threadIdx.x >> 6] = lo;
        b[1][threadIdx.x >> 6] = hi;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const uint32_t *x = b[threadIdx.x];
        atomicMax(&bounds[threadIdx.x], max(max(x[0], x[1]), max(x[2], x[3])));
    }
}

// ---------------------------------------------------------------------------
// large levels
// ---------------------------------------------------------------------------
// Bucket of an x-center on a linear grid of nb buckets over the bounds (never
// decreasing with the order key; a NaN center goes last).
struct XGrid {
    float lo, scale;
    __device__ __forceinline__ XGrid(const uint32_t *bounds, uint32_t nb) {
        const uint32_t kl = ~bounds[0], kh = bounds[1];
        lo = kh >= kl ? key_float(kl) : 0.f;
        scale = kh > kl ? (float)nb / (key_float(kh) - lo) : 0.f;
        if (!(scale < 3.0e38f)) scale = 0.f;   // a range too small or too large for the division
    }
    __device__ __forceinline__ uint32_t bucket(float c, uint32_t nb) const {
        if (c != c) return nb - 1;
        if (scale == 0.f) return 0;
        const float t = fminf(fmaxf((c - lo) * scale, 0.f), (float)(nb - 1));
        return (uint32_t)t;
    }
};

template <uint32_t NB>
__global__ void __launch_bounds__(1024)
str_x_hist(const float4 *__restrict__ it, uint32_t c, const uint32_t *__restrict__ bounds, uint32_t *__restrict__ hist) {
    __shared__ uint32_t h[NB];
    for (uint32_t i = threadIdx.x; i < NB; i += 1024) h[i] = 0;
    __syncthreads();
    const XGrid g(bounds, NB);
    for (uint32_t i = blockIdx.x * 1024 + threadIdx.x; i < c; i += gridDim.x * 1024) {
        const float4 v = it[i];
        atomicAdd(&h[g.bucket(center(v.x, v.z), NB)], 1u);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < NB; i += 1024)
        if (h[i]) atomicAdd(&hist[i], h[i]);
}

// A bucket that straddles slices: its first x-rank, its items, where they are
// collected and how many have been (a cache line each: updates of one line are
// serialized, and eight counters to a line made the collecting pass of 10M
// items take 430 us; 175 with the table below in LDS too).
struct alignas(128) Straddler {
    uint32_t rank0, count, at, taken;
};
constexpr uint32_t kStrRankMax = 8192;   // items of a bucket ranked in LDS
constexpr uint32_t kStradBit = 0x8000u;   // beside a slice or straddler below kStrMaxSlices
constexpr uint32_t kStrMaxSlices = 4096;

__device__ __forceinline__ uint32_t block_excl_scan_1024(uint32_t v, uint32_t *wsum, uint32_t *total) {
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t x = __shfl_up(inc, d);
        if ((int)lane >= d) inc += x;
    }
    __syncthreads();
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
    for (uint32_t i = 0; i < 16; ++i) {
        if (i < w) base += wsum[i];
        tot += wsum[i];
    }
    *total = tot;
    return base + inc - v;
}

// One block: per bucket its slice, or kStradBit | index into the straddlers.
template <uint32_t NB>
__global__ void __launch_bounds__(1024)
str_x_table(const uint32_t *__restrict__ hist, uint32_t slice, uint16_t *__restrict__ table,
            Straddler *__restrict__ strad, uint32_t *__restrict__ nstrad, uint32_t *__restrict__ flag) {
    constexpr uint32_t R = NB / 1024;
    __shared__ uint32_t wsum[16];
    uint32_t n[R], sum = 0, tot;
    if constexpr (R % 4 == 0) {
        const uint4 *h4 = reinterpret_cast<const uint4 *>(hist) + threadIdx.x * (R / 4);
#pragma unroll
        for (uint32_t r = 0; r < R; r += 4) {
            const uint4 v = h4[r / 4];
            n[r] = v.x;
            n[r + 1] = v.y;
            n[r + 2] = v.z;
            n[r + 3] = v.w;
        }
    } else {
#pragma unroll
        for (uint32_t r = 0; r < R; ++r) n[r] = hist[threadIdx.x * R + r];
    }
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) sum += n[r];
    const uint32_t rank0 = block_excl_scan_1024(sum, wsum, &tot);
    // slices of a bucket's first and last item; ranks only grow, so the slice
    // is stepped, not divided for
    const uint32_t slice0 = rank0 / slice;
    uint32_t ns = 0, items = 0, rank = rank0, end = (slice0 + 1) * slice;
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        if (rank + n[r] > end) {
            ns += 1;
            items += n[r];
        }
        rank += n[r];
        while (rank >= end) end += slice;
    }
    uint32_t total_s;
    uint32_t id = block_excl_scan_1024(ns, wsum, &total_s);
    uint32_t at = block_excl_scan_1024(items, wsum, &tot);
    uint32_t sl = slice0;
    rank = rank0;
    end = (slice0 + 1) * slice;
    uint16_t row[R];
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        row[r] = (uint16_t)sl;
        if (rank + n[r] > end) {
            row[r] = (uint16_t)(kStradBit | id);
            strad[id] = Straddler{rank, n[r], at, 0u};
            if (n[r] > kStrRankMax) atomicOr(flag, kStrSkewed);
            id += 1;
            at += n[r];
        }
        rank += n[r];
        while (rank >= end) {
            end += slice;
            sl += 1;
        }
    }
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) table[threadIdx.x * R + r] = row[r];
    if (threadIdx.x == 0) *nstrad = total_s;
}

// The table in LDS: looked up from memory, 64 items of a wave touch 64 lines.
template <uint32_t NB>
__global__ void __launch_bounds__(1024)
str_x_assign(const float4 *__restrict__ it, uint32_t c, const uint32_t *__restrict__ bounds,
             const uint16_t *__restrict__ table, Straddler *__restrict__ strad, uint64_t *__restrict__ collect,
             uint32_t *__restrict__ xs, const uint32_t *__restrict__ flag) {
    __shared__ uint32_t tb[NB / 2];
    if (*flag) return;
    for (uint32_t i = threadIdx.x; i < NB / 2; i += 1024) tb[i] = reinterpret_cast<const uint32_t *>(table)[i];
    __syncthreads();
    const XGrid g(bounds, NB);
    const uint32_t step = gridDim.x * 1024;
    for (uint32_t i0 = blockIdx.x * 1024 + threadIdx.x; i0 < c; i0 += 2 * step) {
        const float4 x[2] = {it[i0], it[min(i0 + step, c - 1)]};
        uint32_t t[2], at[2] = {0, 0};
        float m[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            m[u] = center(x[u].x, x[u].z);
            const uint32_t b = g.bucket(m[u], NB);
            t[u] = (tb[b >> 1] >> (16 * (b & 1u))) & 0xFFFFu;
            if (i0 + u * step < c && (t[u] & kStradBit)) {
                Straddler *s = &strad[t[u] & ~kStradBit];
                at[u] = s->at + atomicAdd(&s->taken, 1u);
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t i = i0 + u * step;
            if (i >= c) break;
            if (t[u] & kStradBit)
                collect[at[u]] = ((uint64_t)order_key(m[u]) << 32) | i;
            else
                xs[i] = t[u];
        }
    }
}

// One block per straddling bucket: every item's rank among the bucket's.
__global__ void __launch_bounds__(1024)
str_x_rank(const Straddler *__restrict__ strad, const uint32_t *__restrict__ nstrad,
           const uint64_t *__restrict__ collect, uint32_t slice, uint32_t *__restrict__ xs,
           const uint32_t *__restrict__ flag) {
    __shared__ uint64_t key[kStrRankMax];
    if (*flag) return;
    const uint32_t ns = *nstrad;
    for (uint32_t b = blockIdx.x; b < ns; b += gridDim.x) {
        const Straddler s = strad[b];
        const uint32_t n = min(s.count, kStrRankMax);
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < n; i += 1024) key[i] = collect[s.at + i];
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < n; i += 1024) {
            const uint64_t k = key[i];
            uint32_t r = s.rank0;
            for (uint32_t j = 0; j < n; ++j) r += key[j] < k ? 1u : 0u;
            xs[(uint32_t)k] = r / slice;
        }
    }
}

// Items to their slices as (y key, index) keys: a tile of 8192 is put in slice
// order in LDS, each slice's share reserved with one update of its cursor, and
// written out in runs.  The order inside a slice is arbitrary.
constexpr uint32_t kStrTile = 8192;

__global__ void __launch_bounds__(1024)
str_to_slices(const float4 *__restrict__ it, uint32_t c, const uint32_t *__restrict__ xs, uint32_t nslices,
              uint32_t slice, uint32_t *__restrict__ cursor, uint64_t *__restrict__ out,
              const uint32_t *__restrict__ flag) {
    __shared__ uint64_t stage[kStrTile];
    __shared__ uint32_t cnt[kStrMaxSlices], base[kStrMaxSlices];
    __shared__ uint16_t ssl[kStrTile];
    __shared__ uint32_t wsum[16];
    if (*flag) return;
    constexpr uint32_t R = kStrTile / 1024;
    const uint32_t t = threadIdx.x;
    const uint32_t i0 = blockIdx.x * kStrTile;
    const uint32_t n = min(c - i0, kStrTile);
    for (uint32_t i = t; i < kStrMaxSlices; i += 1024) cnt[i] = 0;
    __syncthreads();
    uint64_t key[R];
    uint32_t sl[R], rank[R];
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        const uint32_t i = r * 1024 + t;
        sl[r] = rank[r] = 0;
        key[r] = 0;
        if (i < n) {
            sl[r] = xs[i0 + i];
            key[r] = ((uint64_t)key_y(it[i0 + i]) << 32) | (i0 + i);
        }
    }
#pragma unroll
    for (uint32_t r = 0; r < R; ++r)
        if (r * 1024 + t < n) rank[r] = atomicAdd(&cnt[sl[r]], 1u);
    __syncthreads();
    uint32_t v[4], sum = 0, tot;
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r) sum += v[r] = cnt[4 * t + r];
    uint32_t ex = block_excl_scan_1024(sum, wsum, &tot);
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r) {
        const uint32_t s = 4 * t + r;
        cnt[s] = ex;   // place of the slice's first item in the tile
        if (v[r] && s < nslices) base[s] = s * slice + atomicAdd(&cursor[s], v[r]) - ex;
        ex += v[r];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < R; ++r)
        if (r * 1024 + t < n) {
            const uint32_t j = cnt[sl[r]] + rank[r];
            stage[j] = key[r];
            ssl[j] = (uint16_t)sl[r];
        }
    __syncthreads();
    for (uint32_t j = t; j < n; j += 1024) out[base[ssl[j]] + j] = stage[j];
}

// One block sorts one slice by (y key, index).  Its keys are bucketed on a
// linear grid of kSliceBuckets over the slice's finite y-centers (LDS counters,
// one scattered write of each key to tmp), and every key's place is its
// bucket's start plus the smaller keys of the bucket, whose y keys are also in
// LDS (of slices up to kSliceLds items): two reads and one scattered write
// where radix passes of 8 bits need seven of each (10M items: 727 -> 207
// us).  A slice with a bucket over
// kSliceBucketMax (y-centers far from uniform) takes the radix passes: the
// index bits first, a pass whose digit is the same in all keys skipped; stable,
// each wave on a contiguous part, ranks within a wave from digit ballots.
constexpr uint32_t kSliceBuckets = 8192, kSliceBucketMax = 1024, kSliceLds = 30720;

template <bool LDS>
__global__ void __launch_bounds__(1024)
str_sort_slices(uint64_t *__restrict__ keys, uint64_t *__restrict__ tmp, uint32_t c, uint32_t slice, int index_bits,
                uint32_t *__restrict__ order, const uint32_t *__restrict__ flag) {
    constexpr uint32_t W = 16, U = 8, NB = kSliceBuckets;
    __shared__ uint32_t lds[NB];
    __shared__ uint32_t ykey[LDS ? kSliceLds : 1];
    __shared__ uint32_t wsum[16];
    __shared__ uint32_t same, big, kmin, kmax;
    if (*flag) return;
    const uint32_t s0 = blockIdx.x * slice;
    const uint32_t n = min(c - s0, slice);
    uint64_t *src = keys + s0, *dst = tmp + s0;
    const uint32_t t = threadIdx.x, lane = t & 63u, w = t >> 6;
    // range of the finite y-centers
    if (t == 0) {
        kmin = 0xFFFFFFFFu;
        kmax = big = 0;
    }
    for (uint32_t i = t; i < NB; i += 1024) lds[i] = 0;
    __syncthreads();
    uint32_t lo = 0xFFFFFFFFu, hi = 0;
    for (uint32_t i = t; i < n; i += 1024) {
        const uint32_t k = (uint32_t)(src[i] >> 32);
        if (fabsf(key_float(k)) <= 3.0e38f) {
            lo = min(lo, k);
            hi = max(hi, k);
        }
    }
    for (int d = 32; d >= 1; d >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, d));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, d));
    }
    if (lane == 0) {
        atomicMin(&kmin, lo);
        atomicMax(&kmax, hi);
    }
    __syncthreads();
    const uint32_t bounds[2] = {~kmin, kmax};
    const XGrid g(bounds, NB);
    auto bucket = [&](uint64_t k) { return g.bucket(key_float((uint32_t)(k >> 32)), NB); };
    for (uint32_t i = t; i < n; i += 1024 * U) {
        uint64_t k[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) k[u] = i + 1024 * u < n ? src[i + 1024 * u] : 0ull;
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
            if (i + 1024 * u < n) atomicAdd(&lds[bucket(k[u])], 1u);
    }
    __syncthreads();
    {
        constexpr uint32_t R = NB / 1024;
        uint32_t v[R], sum = 0, tot, mx = 0;
#pragma unroll
        for (uint32_t r = 0; r < R; ++r) {
            v[r] = lds[t * R + r];
            mx = max(mx, v[r]);
            sum += v[r];
        }
        if (mx > kSliceBucketMax) big = 1;
        uint32_t ex = block_excl_scan_1024(sum, wsum, &tot);
        if (!big) {   // block-uniform (barriers lie between the write and here)
#pragma unroll
            for (uint32_t r = 0; r < R; ++r) {
                lds[t * R + r] = ex;
                ex += v[r];
            }
        }
    }
    __syncthreads();
    if (!big) {
        for (uint32_t i = t; i < n; i += 1024 * U) {
            uint64_t k[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) k[u] = i + 1024 * u < n ? src[i + 1024 * u] : 0ull;
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                if (i + 1024 * u < n) {
                    const uint32_t at = atomicAdd(&lds[bucket(k[u])], 1u);
                    dst[at] = k[u];
                    if (LDS) ykey[at] = (uint32_t)(k[u] >> 32);
                }
        }
        __syncthreads();   // lds[b]: end of bucket b
        for (uint32_t i = t; i < n; i += 1024) {
            const uint64_t k = dst[i];
            const uint32_t b = bucket(k), b0 = b ? lds[b - 1] : 0u, b1 = lds[b];
            uint32_t r = b0;
            if constexpr (LDS) {
                const uint32_t y = (uint32_t)(k >> 32);
                uint32_t equal = 0;
#pragma unroll 4
                for (uint32_t j = b0; j < b1; ++j) {
                    const uint32_t yj = ykey[j];
                    r += yj < y ? 1u : 0u;
                    equal += yj == y ? 1u : 0u;
                }
                if (equal > 1)   // ties by index
                    for (uint32_t j = b0; j < b1; ++j)
                        if (ykey[j] == y) r += (uint32_t)dst[j] < (uint32_t)k ? 1u : 0u;
            } else {
                for (uint32_t j = b0; j < b1; ++j) r += dst[j] < k ? 1u : 0u;
            }
            order[s0 + r] = (uint32_t)k;
        }
        return;
    }
    uint32_t *cnt = lds;   // [W][256]
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    const uint32_t per = ((n + W - 1) / W + 63) / 64 * 64;   // items per wave
    const uint32_t b0 = min(w * per, n), b1 = min(b0 + per, n);
    const int np = (index_bits + 7) / 8 + 4;
    for (int p = 0; p < np; ++p) {
        const int shift = p < np - 4 ? 8 * p : 32 + 8 * (p - (np - 4));
        for (uint32_t i = t; i < W * 256; i += 1024) cnt[i] = 0;
        if (t == 0) same = 0;
        __syncthreads();
        for (uint32_t i = b0 + lane; i < b1; i += 64 * U) {
            uint32_t d[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) d[u] = i + 64 * u < b1 ? (uint32_t)(src[i + 64 * u] >> shift) & 255u : 256u;
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                if (d[u] < 256u) atomicAdd(&cnt[w * 256 + d[u]], 1u);
        }
        __syncthreads();
        uint32_t sum = 0, tot;
        if (t < 256)
            for (uint32_t x = 0; x < W; ++x) {
                const uint32_t v = cnt[x * 256 + t];
                cnt[x * 256 + t] = sum;
                sum += v;
            }
        if (sum == n) same = 1;
        const uint32_t ex = block_excl_scan_1024(sum, wsum, &tot);
        if (same) {   // block-uniform (a barrier lies between the write and here)
            __syncthreads();
            continue;
        }
        if (t < 256)
            for (uint32_t x = 0; x < W; ++x) cnt[x * 256 + t] += ex;
        __syncthreads();
        for (uint32_t i = b0; i < b1; i += 64 * U) {
            uint64_t k[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t j = i + 64 * u + lane;
                k[u] = j < b1 ? src[j] : 0ull;
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                if (i + 64 * u >= b1) break;   // wave-uniform
                const bool ok = i + 64 * u + lane < b1;
                const uint32_t d = (uint32_t)(k[u] >> shift) & 255u;
                uint64_t peers = __ballot(ok);
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const uint64_t bb = __ballot((d >> b) & 1u);
                    peers &= ((d >> b) & 1u) ? bb : ~bb;
                }
                uint32_t at = 0;
                if (ok) at = cnt[w * 256 + d] + (uint32_t)__popcll(peers & lt);
                __builtin_amdgcn_wave_barrier();
                if (ok && (peers >> lane) == 1ull) cnt[w * 256 + d] += (uint32_t)__popcll(peers);
                __builtin_amdgcn_wave_barrier();
                if (ok) dst[at] = k[u];
            }
        }
        __syncthreads();
        uint64_t *x = src;
        src = dst;
        dst = x;
    }
    for (uint32_t i = t; i < n; i += 1024) order[s0 + i] = (uint32_t)src[i];
}

// ---------------------------------------------------------------------------
// any level: LSD radix sorts
// ---------------------------------------------------------------------------
// keys[i] = key(center_x or center_y of item i) << 32 | i
__global__ void str_center_keys(const float4 *__restrict__ it, uint32_t c, int axis, uint64_t *__restrict__ keys) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < c; i += gridDim.x * blockDim.x) {
        const float4 v = it[i];
        keys[i] = ((uint64_t)(axis ? key_y(v) : key_x(v)) << 32) | i;
    }
}

// xs[item] = the slice of its position in x order
__global__ void str_slices_of(const uint64_t *__restrict__ sorted, uint32_t c, uint32_t slice,
                              uint32_t *__restrict__ xs) {
    for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < c; p += gridDim.x * blockDim.x)
        xs[(uint32_t)sorted[p]] = p / slice;
}

// keys[q] = slice(item) << 32 | item, items taken in (y key, index) order
__global__ void str_slice_keys(const uint64_t *__restrict__ ys, const uint32_t *__restrict__ xs, uint32_t c,
                               uint64_t *__restrict__ keys) {
    for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < c; q += gridDim.x * blockDim.x) {
        const uint32_t i = (uint32_t)ys[q];
        keys[q] = ((uint64_t)xs[i] << 32) | i;
    }
}

__global__ void str_take_order(const uint64_t *__restrict__ keys, uint32_t c, uint32_t *__restrict__ order) {
    for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < c; q += gridDim.x * blockDim.x)
        order[q] = (uint32_t)keys[q];
}

// ---------------------------------------------------------------------------
// small levels: ranks by counting
// ---------------------------------------------------------------------------
// 64 items per block (one per lane), the keys they are compared with divided
// among the block's 16 waves.  Y = false: xs[i] = x-rank / slice.  Y = true:
// order[rank by (slice, y key, index)] = i.
constexpr uint32_t kStrSmall = 16384;

// Keys before the block's items count when not larger, keys after them when
// smaller (ties by index), so the loops are a compare and an add per key.
__device__ __forceinline__ uint32_t count_keys(const uint32_t *key, uint32_t j0, uint32_t j1, uint32_t k, bool ties) {
    uint32_t r = 0;
    if (ties) {
#pragma unroll 8
        for (uint32_t j = j0; j < j1; ++j) r += key[j] <= k ? 1u : 0u;
    } else {
#pragma unroll 8
        for (uint32_t j = j0; j < j1; ++j) r += key[j] < k ? 1u : 0u;
    }
    return r;
}
__device__ __forceinline__ uint32_t count_keys(const uint64_t *key, uint32_t j0, uint32_t j1, uint64_t k, bool ties) {
    uint32_t r = 0;
    if (ties) {
#pragma unroll 8
        for (uint32_t j = j0; j < j1; ++j) r += key[j] <= k ? 1u : 0u;
    } else {
#pragma unroll 8
        for (uint32_t j = j0; j < j1; ++j) r += key[j] < k ? 1u : 0u;
    }
    return r;
}

template <bool Y> struct RankKey { typedef uint32_t type; };
template <> struct RankKey<true> { typedef uint64_t type; };

template <bool Y>
__global__ void __launch_bounds__(1024)
str_count_ranks(const float4 *__restrict__ it, uint32_t c, uint32_t slice, uint32_t *__restrict__ xs,
                uint32_t *__restrict__ order) {
    typedef typename RankKey<Y>::type Key;
    constexpr uint32_t T = 4096;
    __shared__ Key key[T];
    __shared__ uint32_t part[16][64];
    auto key_of = [&](uint32_t i) -> Key {
        const float4 v = it[i];
        if constexpr (Y) return (uint64_t)xs[i] << 32 | key_y(v);
        else return key_x(v);
    };
    const uint32_t t = threadIdx.x, lane = t & 63u, w = t >> 6;
    const uint32_t i0 = blockIdx.x * 64, i = i0 + lane;
    const Key ki = i < c ? key_of(i) : Key(0);
    uint32_t r = 0;
    for (uint32_t t0 = 0; t0 < c; t0 += T) {
        const uint32_t n = min(c - t0, T);
        __syncthreads();
        for (uint32_t j = t; j < n; j += 1024) key[j] = key_of(t0 + j);
        __syncthreads();
        // a multiple of 64 keys per wave: the block's own items lie in one part
        const uint32_t per = (n + 16 * 64 - 1) / (16 * 64) * 64, j0 = min(w * per, n), j1 = min(j0 + per, n);
        const uint32_t own0 = min(max(i0, t0 + j0), t0 + j1) - t0, own1 = min(max(i0 + 64, t0 + j0), t0 + j1) - t0;
        r += count_keys(key, j0, own0, ki, true);
        for (uint32_t j = own0; j < own1; ++j) r += (key[j] < ki || (key[j] == ki && t0 + j < i)) ? 1u : 0u;
        r += count_keys(key, own1, j1, ki, false);
    }
    part[w][lane] = r;
    __syncthreads();
    if (w == 0 && i < c) {
        r = 0;
        for (uint32_t x = 0; x < 16; ++x) r += part[x][lane];
        if (Y) order[r] = i;
        else xs[i] = r / slice;
    }
}

// ---------------------------------------------------------------------------
// nodes of a level
// ---------------------------------------------------------------------------
// G lanes per node (lane e: packing position kF + e): optional low-x order
// (rank by (low x, packing position)), the items' rectangles in entry order
// (packed, if not NULL) and the node's MBR.  ident: the packing order is the
// identity and is written.
template <int G>
__global__ void __launch_bounds__(256)
str_nodes(const float4 *__restrict__ it, uint32_t *__restrict__ order, bool ident, uint32_t c, uint32_t F, uint32_t P,
          bool sort_lx, float4 *packed, float4 *__restrict__ mbr, const uint32_t *__restrict__ flag) {
    if (*flag) return;   // the order may be incomplete
    const uint32_t lane = threadIdx.x & 63u, e = lane & (G - 1), gbase = lane & ~(uint32_t)(G - 1);
    const uint32_t k = blockIdx.x * (256 / G) + threadIdx.x / G;
    const uint32_t r0 = k * F;
    const uint32_t cnt = k < P && c > r0 ? min(c - r0, F) : 0u;
    const bool in = e < cnt;
    uint32_t item = 0;
    float4 v = make_float4(INFINITY, INFINITY, -INFINITY, -INFINITY);
    if (in) {
        item = ident ? r0 + e : order[r0 + e];
        v = it[item];
    }
    uint32_t rank = e;
    if (sort_lx) {
        const uint32_t key = in ? order_key(v.x) : 0xFFFFFFFFu;
        rank = 0;
        for (uint32_t x = 0; x < F; ++x) {
            const uint32_t kx = (uint32_t)__shfl((int)key, (int)(gbase + x));
            rank += (x < cnt && (kx < key || (kx == key && x < e))) ? 1u : 0u;
        }
    }
    if (in) {
        if (ident || sort_lx) order[r0 + rank] = item;
        if (packed) packed[r0 + rank] = v;
    }
    float4 m = v;
    for (int d = G / 2; d >= 1; d >>= 1) {
        m.x = fminf(m.x, __shfl_xor(m.x, d));
        m.y = fminf(m.y, __shfl_xor(m.y, d));
        m.z = fmaxf(m.z, __shfl_xor(m.z, d));
        m.w = fmaxf(m.w, __shfl_xor(m.w, d));
    }
    if (e == 0 && k < P) mbr[k] = cnt ? m : make_float4(NAN, NAN, NAN, NAN);
}

// ---------------------------------------------------------------------------
// all levels
// ---------------------------------------------------------------------------
struct StrLevel {
    const float4 *items;   // rectangles (level 0) or the MBRs of the level below
    uint32_t *order;       // packing order
    float4 *mbr;           // node MBRs
    uint32_t *pos;         // place of every node inside its level
    uint32_t c, P, first;  // items, nodes, first node of the level in the tree
};
struct StrLevels {
    StrLevel l[32];
    uint32_t H, F;
};

// The levels from l0 up (at most 1024 items each), in one block: packing order,
// nodes, then the places of these levels' nodes and of level l0 - 1's.
__global__ void __launch_bounds__(1024)
str_top(StrLevels L, uint32_t l0, bool sort_lx, const uint32_t *__restrict__ slices, const uint32_t *__restrict__ flag) {
    __shared__ uint32_t kx[1024], ky[1024], sl[1024], ord[1024], ord2[1024], cnt[1024];
    __shared__ float4 r[1024];
    if (*flag) return;
    const uint32_t F = L.F, t = threadIdx.x;
    for (uint32_t l = l0; l < L.H; ++l) {
        const StrLevel v = L.l[l];
        const uint32_t c = v.c;
        __syncthreads();
        if (t < c) {
            r[t] = v.items[t];
            kx[t] = key_x(r[t]);
            ky[t] = key_y(r[t]);
            ord[t] = t;
        }
        __syncthreads();
        if (c > F) {
            // item t % cp against the keys of part t / cp
            uint32_t cp = 64;
            while (cp < c) cp <<= 1;
            const uint32_t parts = 1024 / cp, i = t & (cp - 1), part = t / cp;
            const uint32_t per = (c + parts - 1) / parts, j0 = min(part * per, c), j1 = min(j0 + per, c);
            uint32_t n = 0;
            cnt[t] = 0;
            __syncthreads();
            if (i < c) {
                const uint32_t k = kx[i];
#pragma unroll 8
                for (uint32_t j = j0; j < j1; ++j) n += (kx[j] < k || (kx[j] == k && j < i)) ? 1u : 0u;
                atomicAdd(&cnt[i], n);
            }
            __syncthreads();
            if (t < c) {
                sl[t] = cnt[t] / slices[l];
                cnt[t] = 0;
            }
            __syncthreads();
            if (i < c) {
                const uint32_t s = sl[i], y = ky[i];
                n = 0;
#pragma unroll 8
                for (uint32_t j = j0; j < j1; ++j)
                    n += (sl[j] < s || (sl[j] == s && (ky[j] < y || (ky[j] == y && j < i)))) ? 1u : 0u;
                atomicAdd(&cnt[i], n);
            }
            __syncthreads();
            if (t < c) ord[cnt[t]] = t;
            __syncthreads();
        }
        if (sort_lx && t < c) {
            const uint32_t a = t / F * F, b = min(a + F, c), key = order_key(r[ord[t]].x);
            uint32_t n = a;
            for (uint32_t j = a; j < b; ++j) {
                const uint32_t k = order_key(r[ord[j]].x);
                n += (k < key || (k == key && j < t)) ? 1u : 0u;
            }
            ord2[n] = ord[t];
        }
        __syncthreads();
        const uint32_t *o = sort_lx ? ord2 : ord;
        if (t < c) v.order[t] = o[t];
        if (t < v.P) {
            float4 m = make_float4(INFINITY, INFINITY, -INFINITY, -INFINITY);
            const uint32_t a = t * F, b = min(a + F, c);
            for (uint32_t j = a; j < b; ++j) {
                const float4 x = r[o[j]];
                m.x = fminf(m.x, x.x);
                m.y = fminf(m.y, x.y);
                m.z = fmaxf(m.z, x.z);
                m.w = fmaxf(m.w, x.w);
            }
            if (b <= a) m = make_float4(NAN, NAN, NAN, NAN);
            v.mbr[t] = m;
        }
    }
    if (t == 0) L.l[L.H - 1].pos[0] = 0;
    for (uint32_t l = L.H - 1; l >= l0 && l >= 1; --l) {
        __syncthreads();
        const StrLevel v = L.l[l];
        const uint32_t g_last = v.pos[v.P - 1], short_by = v.P * F - v.c;
        if (t < v.c) {
            const uint32_t g = v.pos[t / F];
            L.l[l - 1].pos[v.order[t]] = g * F - (g > g_last ? short_by : 0u) + t % F;
        }
    }
}

// Places of level l-1's nodes from the places of level l's: the children of
// the node at place g start at the entry counts of the nodes stored before it.
__global__ void str_child_pos(StrLevel v, uint32_t F, uint32_t *__restrict__ child_pos,
                              const uint32_t *__restrict__ flag) {
    if (*flag) return;
    const uint32_t g_last = v.pos[v.P - 1];
    const uint32_t short_by = v.P * F - v.c;   // missing entries of the last-created node
    for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < v.c; r += gridDim.x * blockDim.x) {
        const uint32_t k = r / F, e = r - k * F;
        const uint32_t g = v.pos[k];
        child_pos[v.order[r]] = g * F - (g > g_last ? short_by : 0u) + e;
    }
}

// First leaf place under place g of level l (g may be one past the last).
__device__ __forceinline__ uint32_t first_leaf_place(const StrLevels &L, uint32_t l, uint32_t g) {
    for (; l >= 1; --l) {
        const StrLevel &v = L.l[l];
        g = g * L.F - (g > v.pos[v.P - 1] ? v.P * L.F - v.c : 0u);
    }
    return g;
}

// Every node of every level in its final place, its entry count, its leaf
// range, and the leaves' ids one after another.  packed: level 0's rectangles
// in entry order.  host (pinned): {flag, place of the short leaf, root MBR}.
__global__ void __launch_bounds__(256)
str_write(StrLevels L, uint32_t layout, const float4 *__restrict__ packed, uint8_t *__restrict__ nodes,
          uint32_t *__restrict__ meta, uint2 *__restrict__ range, uint32_t *__restrict__ leaf_ids,
          const uint32_t *__restrict__ flag, uint32_t *__restrict__ host) {
    const uint32_t F = L.F;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        host[0] = *flag;
        if (!*flag) {
            host[1] = L.l[0].pos[L.l[0].P - 1];
            const float4 m = L.l[L.H - 1].mbr[0];
            host[2] = __float_as_uint(m.x);
            host[3] = __float_as_uint(m.y);
            host[4] = __float_as_uint(m.z);
            host[5] = __float_as_uint(m.w);
        }
    }
    if (*flag) return;
    uint64_t w = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t base = 0;
    for (uint32_t l = 0; l < L.H; ++l) {
        const StrLevel v = L.l[l];
        const uint64_t slots = (uint64_t)v.P * F;
        const uint32_t g_last = v.pos[v.P - 1], short_by = v.P * F - v.c;
        for (; w < base + slots; w += (uint64_t)gridDim.x * blockDim.x) {
            const uint32_t k = (uint32_t)((w - base) / F), e = (uint32_t)((w - base) - (uint64_t)k * F);
            const uint32_t r0 = k * F;
            const uint32_t cnt = v.c > r0 ? min(v.c - r0, F) : 0u;
            const uint32_t place = v.pos[k];
            float4 x = make_float4(NAN, NAN, NAN, NAN);
            uint32_t p = 0xFFFFFFFFu;
            if (e < cnt) {
                const uint32_t item = v.order[r0 + e];
                if (l == 0) {
                    x = packed[r0 + e];
                    p = item;
                    leaf_ids[(uint64_t)place * F - (place > g_last ? short_by : 0u) + e] = item;
                } else {
                    x = v.items[item];
                    p = L.l[l - 1].first + L.l[l - 1].pos[item];
                }
            }
            const uint32_t g = v.first + place;
            uint8_t *node = nodes + (uint64_t)g * (20u * F);
            float *f = reinterpret_cast<float *>(node);
            uint32_t *u = reinterpret_cast<uint32_t *>(node);
            if (layout == LAYOUT_SOA) {
                f[e] = x.x;
                f[F + e] = x.y;
                f[2 * F + e] = x.z;
                f[3 * F + e] = x.w;
                u[4 * F + e] = p;
            } else if (layout == LAYOUT_AOS) {
                f[5 * e + 0] = x.x;
                f[5 * e + 1] = x.y;
                f[5 * e + 2] = x.z;
                f[5 * e + 3] = x.w;
                u[5 * e + 4] = p;
            } else {
                f[2 * e] = x.x;
                f[2 * e + 1] = x.y;
                f[2 * F + 2 * e] = x.z;
                f[2 * F + 2 * e + 1] = x.w;
                u[4 * F + e] = p;
            }
            if (e == 0) {
                meta[g] = cnt | (l << 8);
                const uint32_t fl = L.l[0].first;
                range[g] = make_uint2(fl + first_leaf_place(L, l, place), fl + first_leaf_place(L, l, place + 1));
            }
        }
        base += slots;
    }
}

static uint32_t grid_for(uint64_t n) {
    uint64_t b = (n + 255) / 256;
    if (b == 0) b = 1;
    return (uint32_t)(b < 16384 ? b : 16384);
}

static uint64_t al(uint64_t b) { return (b + 255) & ~255ull; }

// Slices of S*F items of a level of c > F items with P nodes.
static uint64_t slice_len(uint64_t P, uint32_t F) {
    uint64_t S = (uint64_t)std::sqrt((double)P);
    while (S * S < P) ++S;
    while (S > 1 && (S - 1) * (S - 1) >= P) --S;
    return S * F;
}

template <uint32_t NB>
static void launch_x_slices(const StrLevel &v, uint32_t slice, const uint32_t *bounds, uint32_t *hist, uint16_t *table,
                            Straddler *strad, uint32_t *nstrad, uint64_t *collect, uint32_t *xs, uint32_t *flag,
                            hipStream_t s) {
    const uint32_t hb = std::min<uint32_t>((uint32_t)num_cus(), (v.c + 8191) / 8192);
    hipLaunchKernelGGL(str_x_hist<NB>, dim3(hb), dim3(1024), 0, s, v.items, v.c, bounds, hist);
    hipLaunchKernelGGL(str_x_table<NB>, dim3(1), dim3(1024), 0, s, hist, slice, table, strad, nstrad, flag);
    const uint32_t ab = std::min<uint32_t>((uint32_t)num_cus() * 2, (v.c + 1023) / 1024);
    hipLaunchKernelGGL(str_x_assign<NB>, dim3(ab), dim3(1024), 0, s, v.items, v.c, bounds, table, strad,
                       collect, xs, flag);
    hipLaunchKernelGGL(str_x_rank, dim3((uint32_t)num_cus() * 2), dim3(1024), 0, s, strad, nstrad, collect, slice, xs,
                       flag);
}

// Levels of the bucketed sort: its items fit the kernels' 32-bit places and its
// slices the tile kernel's counters.
static bool bucketed(uint64_t c, uint64_t nslices) { return c <= (1ull << 30) && nslices <= kStrMaxSlices; }

// The packing order of a level by LSD radix sorts.
static hipError_t lsd_order(const StrLevel &v, uint32_t slice, uint64_t nslices, uint64_t *keys, uint64_t *tmp,
                            uint32_t *xs, uint32_t *hist, uint64_t *hscan, uint64_t *stmp, hipStream_t s) {
    const int top32[4] = {32, 40, 48, 56};
    const uint32_t g = grid_for(v.c);
    bool in_tmp = false;
    // x order -> slice of every item
    hipLaunchKernelGGL(str_center_keys, dim3(g), dim3(256), 0, s, v.items, v.c, 0, keys);
    hipError_t e = launch_radix_sort_u64(keys, tmp, v.c, top32, 4, hist, hscan, stmp, &in_tmp, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(str_slices_of, dim3(g), dim3(256), 0, s, in_tmp ? tmp : keys, v.c, slice, xs);
    // (y key, index) order
    hipLaunchKernelGGL(str_center_keys, dim3(g), dim3(256), 0, s, v.items, v.c, 1, keys);
    e = launch_radix_sort_u64(keys, tmp, v.c, top32, 4, hist, hscan, stmp, &in_tmp, s);
    if (e != hipSuccess) return e;
    uint64_t *ys = in_tmp ? tmp : keys, *a = in_tmp ? keys : tmp;
    // stable by slice
    int sb = 0;
    while ((1ull << sb) < nslices) ++sb;
    hipLaunchKernelGGL(str_slice_keys, dim3(g), dim3(256), 0, s, ys, xs, v.c, a);
    e = launch_radix_sort_u64(a, ys, v.c, top32, (sb + 7) / 8, hist, hscan, stmp, &in_tmp, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(str_take_order, dim3(g), dim3(256), 0, s, in_tmp ? ys : a, v.c, v.order);
    return hipGetLastError();
}

struct StrWords {
    uint32_t w[32];
    explicit StrWords(const uint32_t *v) { std::memcpy(w, v, sizeof w); }
};
__global__ void str_set_words(uint32_t *dst, StrWords v) { dst[threadIdx.x] = v.w[threadIdx.x]; }

__global__ void str_gather(StrLevel v, float4 *__restrict__ packed, const uint32_t *__restrict__ flag) {
    if (*flag) return;
    for (uint32_t i = threadIdx.x; i < v.c; i += blockDim.x) packed[i] = v.items[v.order[i]];
}

// Device memory a build leaves in the workspace pool.
constexpr uint64_t kBuildKeep = 512ull << 20;

// lsd: sort every large level with LSD radix sorts.  Sets *redo (and builds
// nothing) when a level's x-centers are too skewed for the buckets.
static int build_str_levels(const float4 *d_rects, uint64_t n, uint32_t F, uint32_t layout, bool sort_lx, bool lsd,
                            hipStream_t s, rt_tree **out, bool *redo) {
    *redo = false;
    // level sizes, leaves first
    std::vector<uint64_t> items, nodes;
    for (uint64_t c = n;;) {
        items.push_back(c);
        const uint64_t P = c > F ? (c + F - 1) / F : 1;
        nodes.push_back(P);
        if (c <= F) break;
        c = P;
    }
    const uint32_t H = (uint32_t)items.size();
    std::vector<uint64_t> first(H);
    uint64_t total = 0;
    for (int l = (int)H - 1; l >= 0; --l) {
        first[l] = total;
        total += nodes[l];
    }
    if (H > 32 || total >= 0xFFFFFFFFull) return fail(RT_EINVAL, "too many nodes");
    uint32_t l0 = H - 1;   // first level built in one block
    while (l0 > 0 && items[l0 - 1] <= 1024) --l0;
    if (items[l0] > 1024) l0 = H;   // (never: the root level has at most F items)

    // workspace: counters (cleared together), per level the packing order, the
    // node MBRs and node places; sort buffers sized for the leaf level
    uint64_t ws = 0;
    auto take = [&](uint64_t bytes) {
        const uint64_t at = ws;
        ws += al(bytes);
        return at;
    };
    const uint64_t flag_off = take(4), bounds_off = take(8);
    std::vector<uint64_t> hist_off(H, 0), cur_off(H, 0), nbk(H, 0), slice(H, 1), nsl(H, 1);
    std::vector<bool> bucket(H, false);
    for (uint32_t l = 0; l < H; ++l) {
        const uint64_t c = items[l];
        if (c <= F) continue;
        slice[l] = slice_len(nodes[l], F);
        nsl[l] = (c + slice[l] - 1) / slice[l];
        if (l >= l0 || c <= kStrSmall || lsd || !bucketed(c, nsl[l])) continue;
        bucket[l] = true;
        nbk[l] = c <= (2u << 20) ? 2048 : (c <= (8u << 20) ? 8192 : 32768);
        hist_off[l] = take(4 * nbk[l]);
        cur_off[l] = take(4 * nsl[l]);
    }
    const uint64_t zero_bytes = ws;
    std::vector<uint64_t> ord_off(H), mbr_off(H), pos_off(H);
    for (uint32_t l = 0; l < H; ++l) {
        ord_off[l] = take(4 * std::max<uint64_t>(items[l], 1));
        mbr_off[l] = take(16 * nodes[l]);
        pos_off[l] = take(4 * nodes[l]);
    }
    const uint64_t cmax = n > 0 ? n : 1;
    const uint64_t slices_off = take(4 * 32), table_off = take(2 * 32768), nstrad_off = take(4);
    const uint64_t strad_off = take(sizeof(Straddler) * (kStrMaxSlices + 1));
    // two buffers of 8-byte keys, contiguous: once the leaf level is sorted
    // they hold its rectangles in entry order
    const uint64_t keys_off = take(16 * cmax);
    const uint64_t c1 = H > 1 ? items[1] : 0;
    const uint64_t keys1_off = take(16 * c1);   // the levels above must not touch those
    const uint64_t xs_off = take(4 * cmax);
    bool any_lsd = false;
    for (uint32_t l = 0; l < l0; ++l) any_lsd |= items[l] > kStrSmall && !bucket[l];
    const uint64_t he = any_lsd ? radix_hist_elems(cmax) : 0;
    const uint64_t rhist_off = take(4 * he), rscan_off = take(8 * (he + 1)), rtmp_off = take(8 * scan_tmp_elems(he + 1));

    void *mem = obj_alloc(KIND_TREE, sizeof(rt_tree));
    if (!mem) return fail(RT_ENOMEM, "host allocation failed");
    rt_tree *t = new (mem) rt_tree();
    (void)hipGetDevice(&t->device);
    t->fanout = F;
    t->layout = layout;
    t->sorted_lx = sort_lx ? 1u : 0u;
    t->height = H;
    t->n_nodes = (uint32_t)total;
    t->first_leaf = (uint32_t)first[0];
    t->node_bytes = 20u * F;
    t->n_objects = n;
    for (uint32_t l = 0; l < H; ++l) t->n_entries += items[l];
    for (uint32_t l = 0; l < H; ++l) t->level_start[l] = (uint32_t)first[l];
    const int dev = t->device;
    PoolWs *pw = nullptr;
    auto bail = [&](int rc) {
        (void)hipStreamSynchronize(s);
        pool_release(dev, pw, s, kBuildKeep);
        tree_release(t);
        std::free(reinterpret_cast<ObjHdr *>(t) - 1);
        return rc;
    };
    // one allocation: nodes, ranges, entry counts, leaf ids
    const uint64_t nodes_at = 0, range_at = al(total * t->node_bytes), meta_at = range_at + al(total * 8),
                   ids_at = meta_at + al(total * 4);
    hipError_t e = pool_acquire(dev, ws, 0, &pw, true);
    if (e != hipSuccess) return bail(hip_fail(e, "device build allocation"));
    e = block_alloc(dev, ids_at + al(n ? n * 4 : 16), &t->d_mem, &t->mem_bytes);
    if (e != hipSuccess) return bail(hip_fail(e, "device build allocation"));
    uint8_t *tb = static_cast<uint8_t *>(t->d_mem);
    t->d_nodes = tb + nodes_at;
    t->d_range = tb + range_at;
    t->d_meta = tb + meta_at;
    t->d_leaf_ids = tb + ids_at;
    uint8_t *wb = static_cast<uint8_t *>(pw->d);
    auto u32 = [&](uint64_t off) { return reinterpret_cast<uint32_t *>(wb + off); };
    auto u64 = [&](uint64_t off) { return reinterpret_cast<uint64_t *>(wb + off); };
    uint32_t *flag = u32(flag_off), *bounds = u32(bounds_off), *xs = u32(xs_off);
    float4 *packed = reinterpret_cast<float4 *>(wb + keys_off);
    StrLevels L;
    L.H = H;
    L.F = F;
    for (uint32_t l = 0; l < H; ++l) {
        StrLevel &v = L.l[l];
        v.items = l == 0 ? d_rects : L.l[l - 1].mbr;
        v.order = u32(ord_off[l]);
        v.mbr = reinterpret_cast<float4 *>(wb + mbr_off[l]);
        v.pos = u32(pos_off[l]);
        v.c = (uint32_t)items[l];
        v.P = (uint32_t)nodes[l];
        v.first = (uint32_t)first[l];
    }
    uint32_t *hw = reinterpret_cast<uint32_t *>(pw->host);   // 16 pinned words
    hw[0] = 0xFFFFFFFFu;
    uint32_t hslices[32] = {0};
    for (uint32_t l = 0; l < H; ++l) hslices[l] = (uint32_t)slice[l];

    e = launch_zero(wb, zero_bytes, s);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(str_set_words, dim3(1), dim3(32), 0, s, u32(slices_off), StrWords(hslices));
        if (n)
            hipLaunchKernelGGL(str_validate, dim3(std::min<uint32_t>(grid_for(n), (uint32_t)num_cus() * 8)), dim3(256),
                               0, s, d_rects, n, flag, bounds);
        e = hipGetLastError();
    }
    // bottom up: packing order and nodes of every level
    for (uint32_t l = 0; l < l0 && e == hipSuccess; ++l) {
        const StrLevel &v = L.l[l];
        const uint32_t sl = (uint32_t)slice[l];
        uint64_t *keys = u64(l == 0 ? keys_off : keys1_off), *tmp = keys + (l == 0 ? cmax : c1);
        if (v.c > F) {
            if (bucket[l]) {
                Straddler *strad = reinterpret_cast<Straddler *>(wb + strad_off);
                uint32_t *hist = u32(hist_off[l]), *ns = u32(nstrad_off);
                uint16_t *table = reinterpret_cast<uint16_t *>(u32(table_off));
#define RT_XS(NB_) launch_x_slices<NB_>(v, sl, bounds, hist, table, strad, ns, tmp, xs, flag, s)
                if (nbk[l] == 2048) RT_XS(2048);
                else if (nbk[l] == 8192) RT_XS(8192);
                else RT_XS(32768);
#undef RT_XS
                hipLaunchKernelGGL(str_to_slices, dim3((v.c + kStrTile - 1) / kStrTile), dim3(1024), 0, s, v.items,
                                   v.c, xs, (uint32_t)nsl[l], sl, u32(cur_off[l]), keys, flag);
                int ib = 0;
                while (ib < 32 && ((uint64_t)(v.c - 1) >> ib)) ++ib;
                if (sl <= kSliceLds)
                    hipLaunchKernelGGL(str_sort_slices<true>, dim3((uint32_t)nsl[l]), dim3(1024), 0, s, keys, tmp, v.c,
                                       sl, ib, v.order, flag);
                else
                    hipLaunchKernelGGL(str_sort_slices<false>, dim3((uint32_t)nsl[l]), dim3(1024), 0, s, keys, tmp,
                                       v.c, sl, ib, v.order, flag);
            } else if (v.c <= kStrSmall) {
                const dim3 g((v.c + 63) / 64), b(1024);
                hipLaunchKernelGGL(str_count_ranks<false>, g, b, 0, s, v.items, v.c, sl, xs, v.order);
                hipLaunchKernelGGL(str_count_ranks<true>, g, b, 0, s, v.items, v.c, sl, xs, v.order);
            } else {
                e = lsd_order(v, sl, nsl[l], keys, tmp, xs, u32(rhist_off), u64(rscan_off), u64(rtmp_off), s);
                if (e != hipSuccess) break;
            }
        }
        const bool ident = v.c <= F;
        float4 *pk = l == 0 ? packed : nullptr;
        const uint32_t G = group_width(F);
        const dim3 g((v.P + 256 / G - 1) / (256 / G)), b(256);
        if (G == 16)
            hipLaunchKernelGGL(str_nodes<16>, g, b, 0, s, v.items, v.order, ident, v.c, F, v.P, sort_lx, pk, v.mbr, flag);
        else if (G == 32)
            hipLaunchKernelGGL(str_nodes<32>, g, b, 0, s, v.items, v.order, ident, v.c, F, v.P, sort_lx, pk, v.mbr, flag);
        else
            hipLaunchKernelGGL(str_nodes<64>, g, b, 0, s, v.items, v.order, ident, v.c, F, v.P, sort_lx, pk, v.mbr, flag);
        e = hipGetLastError();
    }
    // the top levels, then the places of the nodes from there down, and the tree
    if (e == hipSuccess) {
        hipLaunchKernelGGL(str_top, dim3(1), dim3(1024), 0, s, L, l0, sort_lx, u32(slices_off), flag);
        if (l0 == 0)   // the leaf level's rectangles in entry order
            hipLaunchKernelGGL(str_gather, dim3(1), dim3(1024), 0, s, L.l[0], packed, flag);
        for (uint32_t l = l0 - 1; l0 > 0 && l >= 1; --l)
            hipLaunchKernelGGL(str_child_pos, dim3(grid_for(items[l])), dim3(256), 0, s, L.l[l], F, L.l[l - 1].pos,
                               flag);
        uint64_t slots = 0;
        for (uint32_t l = 0; l < H; ++l) slots += nodes[l] * F;
        hipLaunchKernelGGL(str_write, dim3(grid_for(slots)), dim3(256), 0, s, L, layout, packed,
                           static_cast<uint8_t *>(t->d_nodes), static_cast<uint32_t *>(t->d_meta),
                           static_cast<uint2 *>(t->d_range), static_cast<uint32_t *>(t->d_leaf_ids), flag, hw);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return bail(hip_fail(e, "device build"));
    if (hw[0] & kStrInvalid) return bail(fail(RT_EINVAL, "rects contain a NaN coordinate or low > high"));
    if (hw[0]) {
        *redo = !lsd;
        return bail(lsd ? fail(RT_EDEVICE, "build flags %u", hw[0]) : RT_OK);
    }
    // every leaf is full but the last-created one
    const uint32_t short_by = (uint32_t)(nodes[0] * F - n);
    t->partial_leaf = short_by ? t->first_leaf + hw[1] : 0xFFFFFFFFu;
    t->partial_cnt = F - short_by;
    std::memcpy(t->mbr, hw + 2, 16);
    pool_release(dev, pw, s, kBuildKeep);
    *out = t;
    return RT_OK;
}

int build_str_on_device(const float4 *d_rects, uint64_t n, uint32_t F, uint32_t layout, bool sort_lx,
                        hipStream_t s, rt_tree **out) {
    bool redo = false;
    const int rc = build_str_levels(d_rects, n, F, layout, sort_lx, false, s, out, &redo);
    return redo ? build_str_levels(d_rects, n, F, layout, sort_lx, true, s, out, &redo) : rc;
}

}  // namespace rtk

using namespace rtk;

extern "C" int rt_build_str_device(const float *d_rects, uint64_t n, uint32_t fanout, uint32_t layout, void *stream,
                                   rt_tree **out) {
    if (!out) return fail(RT_EINVAL, "out is NULL");
    *out = nullptr;
    try {
        if (fanout != 0 && (fanout < 2 || fanout > 64)) return fail(RT_EINVAL, "fanout %u not in 2..64", fanout);
        const bool sort_lx = (layout & RT_BUILD_SORT_LX) != 0;
        layout &= ~RT_BUILD_SORT_LX;
        if (layout != RT_LAYOUT_AOS && layout != RT_LAYOUT_SOA && layout != RT_LAYOUT_D2 && layout != RT_LAYOUT_AUTO)
            return fail(RT_EINVAL, "unknown layout %u", layout);
        if (n >= 0xFFFFFFFFull) return fail(RT_EINVAL, "n = %llu does not fit 32-bit ids", (unsigned long long)n);
        if (n && !d_rects) return fail(RT_EINVAL, "rects is NULL with n = %llu", (unsigned long long)n);
        if ((reinterpret_cast<uintptr_t>(d_rects) & 15) != 0) return fail(RT_EINVAL, "rects not 16-byte aligned");
        if (fanout == 0 || layout == RT_LAYOUT_AUTO)
            return build_tuned(reinterpret_cast<const float4 *>(d_rects), n, fanout, layout, sort_lx,
                               static_cast<hipStream_t>(stream), out);
        return build_str_on_device(reinterpret_cast<const float4 *>(d_rects), n, fanout, layout, sort_lx,
                                   static_cast<hipStream_t>(stream), out);
    } catch (const std::bad_alloc &) {
        return fail(RT_ENOMEM, "host allocation failed");
    } catch (...) {
        return fail(RT_EDEVICE, "unexpected failure");
    }
}
