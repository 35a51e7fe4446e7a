// Segmented sort of the CSR id lists (each query's ids ascending).
//
// Object ids are spread over [0, n), so a segment splits evenly when it is
// bucketed by the top bits of its ids.  The sort is therefore one MSD
// bucketing pass followed by independent sorts of small buckets:
//
//   classify   every segment with >= 2 ids goes to a size-class list
//              (appends aggregated per block);
//   class S    (<= 256 ids)     one wave per segment: the ids sit in
//              registers (up to 4 per lane) and a bitonic network runs over
//              them with __shfl_xor for cross-lane partners;
//   class M    (257 .. 32768, in four block shapes: 64 x 16, 128 x 32, 512 x 32
//              and 1024 x 32 threads x ids)  one block per segment: ids to
//              registers, a counting sort on the top b id bits (2^b ~
//              length/4 buckets, LDS counters), scatter into LDS, then rounds
//              that sort and merge neighbouring runs of 8 ids in registers
//              until every bucket is in order;
//   class L    (> 32768)        an MSD pass on the top 8 id bits into global
//              scratch, cut into parts of 16384 ids so that one segment
//              occupies many blocks (digit counts of a segment's parts added
//              up, every part digit-sorted in LDS and written as a run per
//              group of consecutive sub-buckets), then the groups (<= 4096 ids
//              each, or <= 32768 when a sub-bucket holds more) sorted back by
//              one block each;
//   fallback   a segment with a bucket too long for these rounds (ids far
//              from uniform) is sorted by a block bitonic network in
//              LDS (class M) or, for class L with a sub-bucket over 32768 ids,
//              by sorting 16384-id tiles that way and merging runs pairwise
//              through LDS-staged merge-path windows.
#include <algorithm>

#include "rt_internal.h"
#include "sort_space.h"

namespace rtk {

constexpr uint32_t kKeyPad = 0xFFFFFFFFu;   // never an object id (ids < 2^32 - 1)
constexpr uint32_t kTileMax = 16384;        // tile of the class-L fallback
constexpr uint32_t kNumCls = 6;             // S, M1, M2, M3, M4, L (by length)
constexpr uint32_t kLong = 5;
constexpr uint32_t kFallback = 6;           // fallback-L list
constexpr uint32_t kListCls = 7;

// Significant bits of the largest id below range (0 for range <= 1).
__device__ __forceinline__ int range_bits(uint32_t range) {
    return range > 1 ? 32 - __clz((int)(range - 1)) : 0;
}

// The id range of segment q: its own (seg_range, when given per segment) or
// the common one.
__device__ __forceinline__ uint32_t seg_id_range(const uint32_t *seg_range, uint32_t q, uint32_t id_range) {
    return seg_range ? seg_range[q] : id_range;
}

__device__ __forceinline__ constexpr uint32_t ceil_log2(uint32_t v) { return v > 1 ? 32 - __builtin_clz(v - 1) : 0; }

// The key of lane (lane ^ j), for the constant distances of a bitonic
// network: a DPP quad permutation for 1 and 2 (an ordinary vector move), the
// bit-mask swizzle for 4, 8 and 16 (within each 32-lane half, no address
// register), a lane permute for 32.  All 64 lanes must be active: DPP and
// swizzle reads of a lane outside the execution mask do not return its key.
__device__ __forceinline__ uint32_t xor_lane(uint32_t v, uint32_t j) {
    if (j == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);   // quad [1,0,3,2]
    if (j == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);   // quad [2,3,0,1]
    if (j == 4) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1F | (4 << 10));
    if (j == 8) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1F | (8 << 10));
    if (j == 16) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1F | (16 << 10));
    return (uint32_t)__shfl_xor((int)v, (int)j);
}

// Bitonic sort of the 64*R keys v[r] (element index r*64 + lane) ascending.
template <int R>
__device__ __forceinline__ void wave_bitonic(uint32_t (&v)[R]) {
    const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
    for (uint32_t k = 2; k <= 64u * R; k <<= 1) {
#pragma unroll
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            if (j >= 64) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int p = r ^ (int)(j / 64);
                    if (p > r) {
                        const bool up = (((uint32_t)r * 64 + lane) & k) == 0;
                        const uint32_t a = v[r], b = v[p];
                        const bool sw = up ? (a > b) : (a < b);
                        v[r] = sw ? b : a;
                        v[p] = sw ? a : b;
                    }
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const uint32_t o = xor_lane(v[r], j);
                    const bool up = (((uint32_t)r * 64 + lane) & k) == 0;
                    const bool lower = (lane & j) == 0;
                    v[r] = (lower == up) ? min(v[r], o) : max(v[r], o);
                }
            }
        }
    }
}

// Block bitonic sort of the first P (power of two) keys of an LDS array.
__device__ void block_bitonic(uint32_t *a, uint32_t P) {
    for (uint32_t k = 2; k <= P; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            for (uint32_t t = threadIdx.x; t < P / 2; t += blockDim.x) {
                const uint32_t i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
                const uint32_t l = i | j;
                const uint32_t x = a[i], y = a[l];
                const bool up = (i & k) == 0;
                if ((x > y) == up) {
                    a[i] = y;
                    a[l] = x;
                }
            }
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------
// class L work space
// ---------------------------------------------------------------------------
constexpr uint32_t kSubMax = 4096;      // longest group sorted by a 128-thread block
constexpr uint32_t kSubBigMax = 32768;  // longest group sorted by a 1024-thread block
constexpr uint32_t kSubCounts = 8;      // counters of the two group work lists (in the class counter block)
constexpr uint32_t kPartCount = 10;     // counter of the part list

// A part holds all that is needed to load its ids, so that a block reads one
// part ahead and never waits for a chain of dependent loads.  A run of at most
// 32768 ids: its place in ids in y and the low half of z, its length in the
// high half.
struct Run {
    uint64_t o;
    uint32_t n;
};
__device__ __forceinline__ Run run_of(uint4 it) {
    return {(uint64_t)(it.z & 0xFFFFu) << 32 | it.y, it.z >> 16};
}
__device__ __forceinline__ uint4 run_item(uint32_t x, uint64_t o, uint32_t n, uint32_t w) {
    return make_uint4(x, (uint32_t)o, (uint32_t)(o >> 32) | n << 16, w);
}

// Behind the cap ids of the scratch (sort_space.h).
struct LongWs {
    uint4 *parts;         // parts {place in the class-L list, run, digit shift}
    uint32_t *desc;       // kDesc words per class-L segment
    uint32_t *sub;        // groups (segment << 8 | group): those of the 128-thread sorts from the front,
    uint32_t *sub_end;    // those of the 1024-thread sorts from the end; at most 256 per segment
};

__device__ __forceinline__ uint32_t num_parts(uint64_t len) { return (uint32_t)((len + kPart - 1) / kPart); }

// Right shift that leaves the digit (the top 8 bits) of ids below range.
__device__ __forceinline__ uint32_t digit_shift(uint32_t range) {
    const int b = range_bits(range);
    return (uint32_t)(b < 8 ? 0 : b - 8);
}

// Part p of the segment of len ids at o, li-th of its class.
__device__ __forceinline__ uint4 part_item(uint32_t li, uint32_t p, uint64_t o, uint64_t len, uint32_t shift) {
    const uint64_t at = (uint64_t)p * kPart;
    return run_item(li, o + at, (uint32_t)min((uint64_t)kPart, len - at), shift);
}

// ---------------------------------------------------------------------------
// classify
// ---------------------------------------------------------------------------
// PER queries per thread: 16 for large batches (fewer list reservations), 2
// where 16 would leave most CUs idle (50k queries: 17.5 -> 6 us).
template <uint32_t PER>
__global__ void __launch_bounds__(256)
seg_classify(const uint64_t *__restrict__ offsets, uint64_t nq, uint64_t cap, uint32_t *__restrict__ lists,
             uint32_t *__restrict__ counts, LongWs lw, uint32_t id_range, const uint32_t *__restrict__ seg_range,
             const Ctrl *__restrict__ ctrl, uint64_t *__restrict__ status) {
    __shared__ uint32_t bcnt[kNumCls], gbase[kNumCls], bparts, pcur;
    if (status && blockIdx.x == 0 && threadIdx.x == 0) select_status(offsets, nq, cap, ctrl, status);
    if (offsets[nq] > cap) return;
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    if (threadIdx.x < kNumCls) bcnt[threadIdx.x] = 0;
    if (threadIdx.x == 0) bparts = 0;
    __syncthreads();
    const uint64_t q0 = (uint64_t)blockIdx.x * (256 * PER);
    int cls[PER];
    uint32_t pos[PER];
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        const uint64_t q = q0 + (uint64_t)k * 256 + threadIdx.x;
        int c = -1;
        if (q < nq) {
            const uint64_t len = offsets[q + 1] - offsets[q];
            if (len >= 2)
                c = len <= 256 ? 0 : len <= 1024 ? 1 : len <= 4096 ? 2 : len <= 16384 ? 3 : len <= kMidMax ? 4 : 5;
            if (c == (int)kLong) atomicAdd(&bparts, num_parts(len));
        }
        cls[k] = c;
        pos[k] = 0;
#pragma unroll
        for (int j = 0; j < (int)kNumCls; ++j) {
            const uint64_t m = __ballot(c == j);
            if (m == 0) continue;
            const uint32_t leader = (uint32_t)__builtin_ctzll(m);
            uint32_t at = 0;
            if (lane == leader) at = atomicAdd(&bcnt[j], (uint32_t)__popcll(m));
            at = __shfl(at, (int)leader);
            if (c == j) pos[k] = at + (uint32_t)__popcll(m & lt);
        }
    }
    __syncthreads();
    if (threadIdx.x < kNumCls)
        gbase[threadIdx.x] = bcnt[threadIdx.x] ? atomicAdd(&counts[threadIdx.x], bcnt[threadIdx.x]) : 0u;
    if (threadIdx.x == 0) pcur = bparts ? atomicAdd(&counts[kPartCount], bparts) : 0u;
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        const int c = cls[k];
        const uint64_t q = q0 + (uint64_t)k * 256 + threadIdx.x;
        if (c >= 0) lists[(uint64_t)c * nq + gbase[c] + pos[k]] = (uint32_t)q;
        if (c == (int)kLong) {
            const uint64_t o = offsets[q], len = offsets[q + 1] - o;
            const uint32_t li = gbase[kLong] + pos[k], np = num_parts(len);
            const uint32_t p0 = atomicAdd(&pcur, np), sh = digit_shift(seg_id_range(seg_range, (uint32_t)q, id_range));
            for (uint32_t d = 0; d < kLongDigits; ++d) lw.desc[(uint64_t)li * kDesc + d] = 0;
            for (uint32_t p = 0; p < np; ++p) lw.parts[p0 + p] = part_item(li, p, o, len, sh);
        }
    }
}

// ---------------------------------------------------------------------------
// class S: one wave per segment
// ---------------------------------------------------------------------------
// Sort the s <= 256 keys a wave holds (v[r] = key r*64 + lane, pad beyond
// s) into dst[0..s).
__device__ __forceinline__ void wave_sort_regs4(uint32_t (&v)[4], uint32_t *dst, uint32_t s) {
    const uint32_t lane = threadIdx.x & 63u;
    if (s < 2) {
        if (s == 1 && lane == 0) dst[0] = v[0];
        return;
    }
    if (s <= 16) {   // ranks by broadcasting each key
        uint32_t rk = 0;
        for (uint32_t j = 0; j < s; ++j) {
            const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)v[0], (int)j);
            rk += (x < v[0] || (x == v[0] && j < lane)) ? 1u : 0u;
        }
        if (lane < s) dst[rk] = v[0];
        return;
    }
    if (s <= 64) {
        uint32_t a[1] = {v[0]};
        wave_bitonic<1>(a);
        if (lane < s) dst[lane] = a[0];
    } else if (s <= 128) {
        uint32_t a[2] = {v[0], v[1]};
        wave_bitonic<2>(a);
#pragma unroll
        for (int r = 0; r < 2; ++r)
            if ((uint32_t)r * 64 + lane < s) dst[r * 64 + lane] = a[r];
    } else {
        wave_bitonic<4>(v);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if ((uint32_t)r * 64 + lane < s) dst[r * 64 + lane] = v[r];
    }
}

// One wave per segment; the wave's next segment is loaded into registers
// before the current one is sorted, so its load overlaps the sort.
__global__ void __launch_bounds__(256)
segsort_small(const uint64_t *__restrict__ offsets, uint32_t *__restrict__ ids, const uint32_t *__restrict__ list,
              const uint32_t *__restrict__ list_count) {
    const uint32_t m = *list_count;
    const uint32_t wpb = blockDim.x / 64;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t step = gridDim.x * wpb;
    uint32_t nv[4];
    uint64_t no = 0;
    uint32_t nc = 0;
    auto load = [&](uint32_t i) {
        const uint32_t q = list[i];
        no = offsets[q];
        nc = (uint32_t)(offsets[q + 1] - no);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t k = (uint32_t)r * 64 + lane;
            nv[r] = k < nc ? ids[no + k] : kKeyPad;
        }
    };
    uint32_t i = blockIdx.x * wpb + (threadIdx.x >> 6);
    if (i < m) load(i);
    for (; i < m; i += step) {
        uint32_t v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = nv[r];
        const uint64_t o = no;
        const uint32_t c = nc;
        if (i + step < m) load(i + step);   // segments are disjoint: never the ids written below
        wave_sort_regs4(v, ids + o, c);
    }
}

// ---------------------------------------------------------------------------
// classes M and L: counting sort on the top id bits, then in-bucket sorts
// ---------------------------------------------------------------------------
// With 2^b ~ length/4 buckets on the top b bits of the ids, a bucket holds a
// handful of ids.  One LDS counter per bucket first counts, is then turned
// into the bucket's start by an exclusive scan, and serves as the scatter
// cursor; after the scatter counter b holds the end of bucket b, so bucket b
// spans [end(b-1), end(b)).  Then only the order within buckets is open, so
// every id is within its bucket's length of its place, and a few rounds of
// sorting and merging neighbouring runs of 8 ids finish the sort
// (sort_near).  A bucket of more than kNearMax ids (ids far from uniform)
// sends the segment to a fallback.
constexpr uint32_t kNearMax = 256;   // 33 rounds; the bitonic fallback over 4096 ids: 78

// Inclusive sum scan over the wave and its running maximum (lane 63: the
// largest), as ordinary vector moves between lanes.  All lanes active.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_0(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t row_sum(uint32_t v) {   // within each row of 16 lanes
    v += dpp_or_0<0x111, 0xF>(v);
    v += dpp_or_0<0x112, 0xF>(v);
    v += dpp_or_0<0x114, 0xF>(v);
    return v + dpp_or_0<0x118, 0xF>(v);
}
__device__ __forceinline__ uint32_t row_max(uint32_t v) {
    v = max(v, dpp_or_0<0x111, 0xF>(v));
    v = max(v, dpp_or_0<0x112, 0xF>(v));
    v = max(v, dpp_or_0<0x114, 0xF>(v));
    return max(v, dpp_or_0<0x118, 0xF>(v));
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
    v = row_sum(v);
    v += dpp_or_0<0x142, 0xA>(v);   // last lane of a row to the next row
    return v + dpp_or_0<0x143, 0xC>(v);
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
    v = row_max(v);
    v = max(v, dpp_or_0<0x142, 0xA>(v));
    return max(v, dpp_or_0<0x143, 0xC>(v));
}
__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane);
}

// Exclusive scan in place of cnt[0 .. nbk) by T threads (nbk a multiple of
// 4); returns the largest count.  wsum: 2*T/64 words.
template <int T>
__device__ uint32_t block_scan_counters(uint32_t *cnt, uint32_t nbk, uint32_t *wsum) {
    constexpr uint32_t W = T / 64;
    static_assert(W <= 16, "one row of lanes holds the waves' sums");
    const uint32_t t = threadIdx.x, lane = t & 63u, w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
    uint4 *c4 = reinterpret_cast<uint4 *>(cnt);
    uint32_t carry = 0, mxall = 0;
    for (uint32_t b0 = 0; b0 < nbk; b0 += 4 * T) {
        const bool mine = b0 + 4 * t < nbk;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (mine) v = c4[b0 / 4 + t];
        const uint32_t sum = v.x + v.y + v.z + v.w;
        const uint32_t inc = wave_sum(sum), mx = wave_max(max(max(v.x, v.y), max(v.z, v.w)));
        if (lane == 63) {
            wsum[w] = inc;
            wsum[W + w] = mx;
        }
        __syncthreads();
        const bool in = (lane & 15u) < W;
        const uint32_t ws = row_sum(in ? wsum[lane & 15u] : 0u), wm = row_max(in ? wsum[W + (lane & 15u)] : 0u);
        uint32_t ex = carry + inc - sum + (w ? lane_value(ws, w - 1) : 0u);
        carry += lane_value(ws, 15);
        mxall = max(mxall, lane_value(wm, 15));
        if (mine) c4[b0 / 4 + t] = make_uint4(ex, ex + v.x, ex + v.x + v.y, ex + v.x + v.y + v.z);
        __syncthreads();
    }
    return mxall;
}

// Batcher's odd-even merge sort of N = 2^k inputs from merges of 2p on (all
// indices fixed at compile time): p = 1 sorts (63 comparators for 16 inputs),
// p = N/2 merges two sorted halves (25).
template <int N, int P0>
__device__ __forceinline__ void reg_oem(uint32_t (&v)[N]) {
#pragma unroll
    for (int p = P0; p < N; p <<= 1) {
#pragma unroll
        for (int k = p; k >= 1; k >>= 1) {
#pragma unroll
            for (int j = k % p; j + k < N; j += 2 * k) {
#pragma unroll
                for (int i = 0; i < k; ++i) {
                    if ((i + j) / (2 * p) == (i + j + k) / (2 * p)) {
                        const uint32_t x = v[i + j], y = v[i + j + k];
                        v[i + j] = x < y ? x : y;
                        v[i + j + k] = x < y ? y : x;
                    }
                }
            }
        }
    }
}

// Where id i of a staged array lies: within its 16 words, the 4-word units
// are exchanged so that lanes reading a whole run of 16 each, as 16-byte
// loads, use all banks (without it, two of eight units).
__device__ __forceinline__ uint32_t near_at(uint32_t i) { return i ^ ((i >> 3) & 12u); }

// The staged ids a (near_at order, pads in the 16 places behind the c ids),
// grouped into buckets of at most big ids that are in order among themselves:
// sorted by rounds over the runs of 8.  Round 0 sorts every aligned pair of
// runs, the odd rounds merge each run with odd place and its successor, the
// even ones the aligned pairs: an odd-even merge-split sort, which needs as
// many rounds as a bucket spans runs, at most (big - 2) / 8 + 2.  Per round
// and 64 ids two 16-byte accesses per 4 lanes and 8 (first) or 3 network
// instructions; a register network per bucket, padded to the longest bucket
// of a wave, took three reads and three writes per id instead.
template <int T>
__device__ __forceinline__ void sort_near(uint32_t *a, uint32_t c, uint32_t big) {
    const uint32_t rounds = big < 2 ? 0u : (big + 6) / 8 + 1;
    uint4 *a4 = reinterpret_cast<uint4 *>(a);
    for (uint32_t r = 0; r < rounds; ++r) {
        const uint32_t off = (r & 1u) * 2;
        for (uint32_t u0 = threadIdx.x * 4 + off; (u0 + off) * 4 < c; u0 += T * 4) {
            uint32_t v[16];
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                const uint32_t u = u0 + j;
                const uint4 x = a4[u ^ ((u >> 3) & 3u)];
                v[4 * j] = x.x, v[4 * j + 1] = x.y, v[4 * j + 2] = x.z, v[4 * j + 3] = x.w;
            }
            if (r == 0)
                reg_oem<16, 1>(v);
            else
                reg_oem<16, 8>(v);
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                const uint32_t u = u0 + j;
                a4[u ^ ((u >> 3) & 3u)] = make_uint4(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]);
            }
        }
        __syncthreads();
    }
}

// The n words at p as a buffer: what lies past them reads as 0 and is not
// written, without a comparison, a mask or a branch, so that many accesses of
// a ragged run are under way at once (a branch per row made the compiler wait
// for each load: 2.9 instead of 1.8 ms for the digit counts of 2.0G ids).
typedef __amdgpu_buffer_rsrc_t Buf;
__device__ __forceinline__ Buf buf_of(const uint32_t *p, uint32_t n) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p), 0, (int)(n * 4), 0x00027000);
}

// key[k] = src[k*T + thread] for the rows that begin below c (0 past the end).
// The scalar part of an offset stays below the buffer's size.
template <int T, int K>
__device__ __forceinline__ void load_keys(const uint32_t *src, uint32_t c, uint32_t (&key)[K]) {
    const Buf b = buf_of(src, c);
#pragma unroll
    for (int k = 0; k < K; k += 4) {
        if ((uint32_t)k * T < c) {
#pragma unroll
            for (int j = k; j < k + 4; ++j)
                key[j] = __builtin_amdgcn_raw_buffer_load_b32(b, (int)(((uint32_t)(j - k) * T + threadIdx.x) * 4),
                                                              k * T * 4, 0);
        }
    }
}

// first(k, in, i), then second(k, in, i) for the rows k of K that begin below
// c, four at a time without a branch, so that four memory operations are under
// way at once; i = k*T + thread is the place, in whether it lies below c.
// Rows past the end cost nothing: the work follows c rather than the tile.
template <int T, int K, typename F, typename G>
__device__ __forceinline__ void rows_by_four(uint32_t c, F &&first, G &&second) {
    static_assert(K % 4 == 0, "rows by fours");
#pragma unroll
    for (int k = 0; k < K; k += 4) {
        if ((uint32_t)(k + 4) * T <= c) {
#pragma unroll
            for (int j = k; j < k + 4; ++j) first(j, true, 0u);
#pragma unroll
            for (int j = k; j < k + 4; ++j) second(j, true, 0u);
        } else if ((uint32_t)k * T < c) {
#pragma unroll
            for (int j = k; j < k + 4; ++j) first(j, (uint32_t)j * T + threadIdx.x < c, (uint32_t)j * T + threadIdx.x);
#pragma unroll
            for (int j = k; j < k + 4; ++j) second(j, (uint32_t)j * T + threadIdx.x < c, (uint32_t)j * T + threadIdx.x);
        }
    }
}

// Sort c <= T*K ids, given in registers (key[k] holds id k*T + thread; any id
// beyond c), into dst with one block: counting sort into nbk = 2^b ~ c/4
// buckets of equal width over the id range (bucket of id x: (x - base) *
// nbk / range, as a 32-bit multiply-high; LDS counters), scatter into LDS,
// sort within the buckets, copy out.  The caller guarantees base <= id <
// base + range for every id.  A: target ids per bucket (nbk ~ c/A, at most
// T*K/A).  A bucket that is too long (ids far from uniform) switches the
// segment to a block bitonic network.  buf: T*K + kStagePad words, cnt: T*K/A
// words, both at 16-byte boundaries, wsum: 2*T/64 words of LDS.
constexpr uint32_t kStagePad = 16;
// next() is called as soon as the registers are free, to load the following
// ids while these are sorted.
template <int T, int K, int A, typename Next>
__device__ __forceinline__ void block_sort_keys(uint32_t (&key)[K], uint32_t *dst, uint32_t c, uint32_t range,
                                                uint32_t *buf, uint32_t *cnt, uint32_t *wsum, uint32_t base,
                                                Next &&next) {
    constexpr uint32_t N = T * K;
    constexpr uint32_t NB = N / A;   // most buckets
    const uint32_t t = threadIdx.x;
    uint32_t nb = ceil_log2((c + A - 1) / A);
    const uint32_t nbmax = ceil_log2(NB);
    nb = nb < 2 ? 2 : (nb > nbmax ? nbmax : nb);
    const uint32_t nbk = 1u << nb;
    // floor(y * mul / 2^32) never decreases with y, for any mul: nbk * 2^32 /
    // range to float precision does, and the min() takes what reaches nbk (a
    // 64-bit division here was a tenth of a short segment's instructions)
    const uint32_t mul =
        range > nbk ? (uint32_t)fminf((float)nbk * 4294967296.0f * __builtin_amdgcn_rcpf((float)range), 4294967040.0f)
                    : 0xFFFFFFFFu;
    auto bucket = [&](uint32_t x) { return min(__umulhi(x - base, mul), nbk - 1); };
    for (uint32_t b = 4 * t; b < nbk; b += 4 * T) *reinterpret_cast<uint4 *>(cnt + b) = make_uint4(0, 0, 0, 0);
    __syncthreads();
    // lanes past the end add nothing, in places of their own (in one place
    // their atomics would go one by one), and fill places past the end
    auto slot = [&](uint32_t x, bool in) { return in ? bucket(x) : t & (nbk - 1); };
    rows_by_four<T, K>(
        c, [&](int k, bool in, uint32_t) { atomicAdd(&cnt[slot(key[k], in)], in ? 1u : 0u); },
        [](int, bool, uint32_t) {});
    __syncthreads();
    const uint32_t big = block_scan_counters<T>(cnt, nbk, wsum);
    uint32_t at[4];
    rows_by_four<T, K>(
        c, [&](int k, bool in, uint32_t) { at[k & 3] = atomicAdd(&cnt[slot(key[k], in)], in ? 1u : 0u); },
        [&](int k, bool in, uint32_t i) {
            const uint32_t to = in ? at[k & 3] : i;
            buf[near_at(to)] = in ? key[k] : kKeyPad;
        });
    if (t < kStagePad) buf[near_at(c + t)] = kKeyPad;
    next();
    __syncthreads();
    if (big <= kNearMax) {
        sort_near<T>(buf, c, big);
        // near_at(i + T) = near_at(i) + T for multiples of 128
        auto staged = [&](uint32_t i) { return T % 128 == 0 ? buf[near_at(t) + (i - t)] : buf[near_at(i)]; };
        const Buf out = buf_of(dst, c);
        for (uint32_t r = 0; r * T < c; r += 4) {
            uint32_t x[4];
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) x[j] = staged((r + j) * T + t);
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j)
                __builtin_amdgcn_raw_buffer_store_b32(x[j], out, (int)((t + j * T) * 4), (int)(r * T * 4), 0);
        }
    } else {   // ids far from uniform: block bitonic over the whole segment
        uint32_t P = 1;
        while (P < c) P <<= 1;
        for (uint32_t i = c + t; i < P; i += T) buf[near_at(i)] = kKeyPad;
        __syncthreads();
        block_bitonic(buf, P);
        for (uint32_t i = t; i < c; i += T) dst[i] = buf[i];
    }
    __syncthreads();
}

// One block per segment of the class list.  The next segment's ids are loaded
// into registers once the current one's are staged, so their load overlaps
// the rest of the sort.  Few threads with many ids each: what a block does per
// segment is then shared by fewer waves, and one wave needs no barriers (257
// to 1024 ids: 64 x 16 0.25 ms, 128 x 8 0.38 ms; 1025 to 4096: 128 x 32 0.93
// ms, 256 x 16 0.97 ms; 10M rectangles / 1M windows, 0.11G and 0.43G ids: 3.7
// and 3.8 TB/s).  Shapes of 16384 ids and up are held to 4 waves per SIMD, so
// that two 512-thread blocks share a CU.
template <int T, int K>
constexpr int mid_waves_per_simd() {
    return T * K >= 16384 ? 4 : 1;
}

// The class-M segments list[0 .. m); buf, cnt, wsum as block_sort_keys'.
template <int T, int K, int A>
__device__ __forceinline__ void
sort_segments(const uint64_t *__restrict__ offsets, uint32_t *__restrict__ ids, const uint32_t *__restrict__ list,
              uint32_t m, uint32_t id_range, const uint32_t *__restrict__ seg_range, uint32_t *buf, uint32_t *cnt,
              uint32_t *wsum) {
    if (blockIdx.x >= m) return;
    // The list entry is read three segments ahead and the offsets two, so that
    // no load waits for another.
    const uint32_t g = gridDim.x;
    auto entry = [&](uint32_t li) { return list[min(li, m - 1)]; };
    uint32_t q = entry(blockIdx.x), key[K];
    uint64_t o = offsets[q], o1 = offsets[q + 1];
    uint32_t r = seg_id_range(seg_range, q, id_range);
    load_keys<T, K>(ids + o, (uint32_t)(o1 - o), key);
    q = entry(blockIdx.x + g);
    uint64_t no = offsets[q], no1 = offsets[q + 1];
    uint32_t nr = seg_id_range(seg_range, q, id_range);
    q = entry(blockIdx.x + 2 * g);
    for (uint32_t li = blockIdx.x; li < m; li += g) {
        const uint64_t co = o;
        const uint32_t cn = (uint32_t)(o1 - o), cr = r;
        block_sort_keys<T, K, A>(key, ids + co, cn, cr, buf, cnt, wsum, 0, [&] {
            // segments are disjoint: these reads never meet the writes of another
            o = no, o1 = no1, r = nr;
            if (li + g < m) load_keys<T, K>(ids + o, (uint32_t)(o1 - o), key);
            no = offsets[q], no1 = offsets[q + 1];
            nr = seg_id_range(seg_range, q, id_range);
            q = entry(li + 3 * g);
        });
    }
}

template <int T, int K, int A>
__global__ void __launch_bounds__(T, (mid_waves_per_simd<T, K>()))
segsort_mid(const uint64_t *__restrict__ offsets, uint32_t *__restrict__ ids, const uint32_t *__restrict__ list,
            const uint32_t *__restrict__ list_count, uint32_t id_range, const uint32_t *__restrict__ seg_range) {
    constexpr uint32_t N = T * K;
    // keys, then the bucket counters; the scan's per-wave sums use the head
    // of the keys, which hold nothing while the counters are scanned
    __shared__ __align__(16) uint32_t lds[N + kStagePad + N / A];
    sort_segments<T, K, A>(offsets, ids, list, *list_count, id_range, seg_range, lds, lds + N + kStagePad, lds);
}

// Class L: two levels.  First the segment is split by its top 8 id bits into
// 256 sub-buckets in global scratch, by parts of kPart ids: the digits of
// every part are counted and added to the segment's (segsort_wide), one block
// per segment cuts the sub-buckets into groups of G consecutive ones and turns
// the counts into the groups' write cursors (segsort_part_scan), and every part
// is counting-sorted by digit in LDS and written out as one run per group, whose
// place it reserves with an update of the group's cursor (segsort_part_split).
// Then the groups are sorted from scratch back into place by the whole grid, one
// block per group (segsort_sub): G is chosen so that a group
// holds at most 4096 ids, or at most 32768 (a 1024-thread block) when a
// sub-bucket holds more than 4096 (segments of about a million ids).  A
// segment with a sub-bucket over 32768 ids (ids far from uniform) is left as
// it is and goes to the fallback list.
//
// Parts keep all CUs at work whatever the number of segments: with one block
// per segment the split of 24 segments of 33K to 500K ids took 326 us (now
// 39 us) and that of 12K such segments, 2.0G ids, 8.2 ms (now 5.7 ms: counts
// 1.8, scan 0.1, split 3.8, at 4.3 to 4.6 TB/s).

// The parts of the XCD-contiguous share that workgroup wg of nwg works on
// (workgroups go round the 8 XCDs): parts of one segment write into the same
// lines of scratch, which meet in one XCD's L2 this way.
struct PartShare {
    uint32_t k, end, step;
};
__device__ __forceinline__ PartShare part_share(uint32_t n, uint32_t wg, uint32_t nwg) {
    if (nwg < 8 || (nwg & 7u)) return {wg, n, nwg};
    const uint32_t per = (n + 7) / 8, x = wg & 7u;
    const uint32_t lo = min(n, x * per), hi = min(n, lo + per);
    return {lo + (wg >> 3), hi, nwg >> 3};
}

// Segments of 16385 .. 32768 ids (class M), then the digit counts of the
// class-L parts: one launch for both, as most batches have few of either.
__global__ void __launch_bounds__(1024, 4)
segsort_wide(const uint64_t *__restrict__ offsets, uint32_t *__restrict__ ids, const uint32_t *__restrict__ lists,
             uint64_t nq, const uint32_t *__restrict__ counts, LongWs lw, uint32_t id_range,
             const uint32_t *__restrict__ seg_range) {
    constexpr uint32_t T = 1024, K = 32, A = 8, N = T * K, R = kPart / T;
    __shared__ __align__(16) uint32_t lds[N + kStagePad + N / A];
    const uint32_t m = counts[4], np = counts[kPartCount];
    sort_segments<T, K, A>(offsets, ids, lists + 4 * nq, m, id_range, seg_range, lds, lds + N + kStagePad, lds);
    const uint32_t t = threadIdx.x, g = gridDim.x;
    // the M segments went to the first blocks: the parts start behind them
    uint32_t k = (blockIdx.x + g - m % g) % g;
    if (k >= np) return;
    uint32_t *h = lds;   // two sets of counters in turn: one barrier less per part
    // two parts under way, the items one further ahead
    auto item = [&](uint32_t i) { return lw.parts[min(i, np - 1)]; };
    uint32_t ka[R], kb[R];
    uint4 ia = item(k), ib = item(k + g);
    load_keys<T, R>(ids + run_of(ia).o, run_of(ia).n, ka);
    auto count = [&](uint32_t (&key)[R], uint4 it) {
        if (t < kLongDigits) h[t] = 0;
        __syncthreads();
        const uint32_t sh = it.w;
        rows_by_four<T, R>(
            run_of(it).n, [&](int r, bool in, uint32_t) {
                atomicAdd(&h[in ? min(key[r] >> sh, kLongDigits - 1) : t % kLongDigits], in ? 1u : 0u);
            },
            [](int, bool, uint32_t) {});
        __syncthreads();
        // 256 counters per segment, added to by its parts: a row per part would
        // not fit the scratch
        if (t < kLongDigits && h[t]) atomicAdd(&lw.desc[(uint64_t)it.x * kDesc + t], h[t]);
        h = h == lds ? lds + kLongDigits : lds;
    };
    for (; k < np; k += g) {
        load_keys<T, R>(ids + run_of(ib).o, run_of(ib).n, kb);   // of the last part again at the end
        uint4 ic = item(k + 2 * g);
        count(ka, ia);
        ia = ic;
        if ((k += g) >= np) break;
        load_keys<T, R>(ids + run_of(ia).o, run_of(ia).n, ka);
        ic = item(k + 2 * g);
        count(kb, ib);
        ib = ic;
    }
}

// Exclusive scan of one value per thread of a 256-thread block; tot and mx:
// the sum and the largest value.  w4: 8 words of LDS.
__device__ __forceinline__ uint32_t scan_digits(uint32_t v, uint32_t *w4, uint32_t &tot, uint32_t &mx) {
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
    uint32_t inc = v;
    mx = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t x = __shfl_up(inc, d);
        if ((int)lane >= d) inc += x;
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, d));
    }
    if (lane == 63) w4[w] = inc;
    if (lane == 0) w4[4 + w] = mx;
    __syncthreads();
    uint32_t ex = inc - v;
    tot = mx = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
        if (i < w) ex += w4[i];
        tot += w4[i];
        mx = max(mx, w4[4 + i]);
    }
    return ex;
}

// One block per class-L segment, one thread per digit: the digits are put into
// groups, the counts become the groups' starts, and the groups are listed.
__global__ void __launch_bounds__(256)
segsort_part_scan(const uint64_t *__restrict__ offsets, const uint32_t *__restrict__ list,
                  const uint32_t *__restrict__ list_count, LongWs lw, uint32_t *__restrict__ sub_counts,
                  uint32_t *__restrict__ fb_list, uint32_t *__restrict__ fb_count, uint32_t id_range,
                  const uint32_t *__restrict__ seg_range) {
    __shared__ uint32_t w4[8], subbase, start[kLongDigits];
    static_assert(kLongDigits == 256, "one thread per digit");
    const uint32_t m = *list_count, t = threadIdx.x;
    for (uint32_t li = blockIdx.x; li < m; li += gridDim.x) {
        const uint32_t q = list[li];
        uint32_t *dsc = lw.desc + (uint64_t)li * kDesc;
        const uint64_t o = offsets[q];
        uint32_t tot, big;
        start[t] = scan_digits(dsc[t], w4, tot, big);
        // groups of G consecutive digits: G = (group limit) / (largest digit
        // count), so a group never exceeds the limit: kSubMax ids for the
        // 128-thread sort, or, when a digit holds more (segments of about a
        // million ids), kSubBigMax for the 1024-thread sort (its own list)
        const bool fallback = big > kSubBigMax, wide = big > kSubMax;
        const uint32_t G = fallback ? 0u : (wide ? kSubBigMax : kSubMax) / big;
        const uint32_t ngroups = G ? (kLongDigits + G - 1) / G : 0u;
        if (t == 0) {
            dsc[kDescGroup] = G;
            dsc[kDescOff] = (uint32_t)o;
            dsc[kDescOff + 1] = (uint32_t)(o >> 32);
            dsc[kDescRange] = seg_id_range(seg_range, q, id_range);
            if (fallback)
                fb_list[atomicAdd(fb_count, 1u)] = q;
            else
                subbase = atomicAdd(&sub_counts[wide ? 1 : 0], ngroups);
        }
        __syncthreads();
        if (t < ngroups) {
            dsc[t] = start[t * G];   // all counts have been read
            const uint32_t i = subbase + t;
            *(wide ? lw.sub_end - 1 - i : lw.sub + i) = li << 8 | t;
        }
        __syncthreads();
    }
}

// One block per part: its ids are counted and ranked by digit in LDS, staged in
// digit order and written as one run per group, whose place an atomic on the
// group's cursor reserves (a group's order within scratch does not matter, as
// it is sorted next).  Two blocks of 1024 threads per CU.
template <int T>
__global__ void __launch_bounds__(T, 8)
segsort_part_split(const uint32_t *__restrict__ ids, uint32_t *__restrict__ scratch,
                   const uint32_t *__restrict__ part_count, LongWs lw) {
    constexpr uint32_t R = kPart / T;
    __shared__ uint32_t stage[kPart];
    __shared__ uint32_t lcur[kLongDigits], gpos[kLongDigits];   // cursor in stage; scratch position minus stage position
    __shared__ uint32_t first[kLongDigits + 1], w4[4];          // digits' places in stage
    const uint32_t t = threadIdx.x, np = *part_count;
    const PartShare ps = part_share(np, blockIdx.x, gridDim.x);
    if (ps.k >= ps.end) return;
    uint4 nx = lw.parts[ps.k];
    for (uint32_t k = ps.k; k < ps.end; k += ps.step) {
        const uint4 it = nx;
        nx = lw.parts[min(k + ps.step, np - 1)];
        uint32_t *dsc = lw.desc + (uint64_t)it.x * kDesc;
        const uint32_t G = dsc[kDescGroup];
        if (G == 0) continue;   // left to the fallback
        const uint32_t len = run_of(it).n, sh = it.w;
        uint32_t key[R];
        load_keys<T, R>(ids + run_of(it).o, len, key);
        if (t < kLongDigits) lcur[t] = 0;
        __syncthreads();
        rows_by_four<T, R>(
            len,
            [&](int r, bool in, uint32_t) {
                atomicAdd(&lcur[in ? min(key[r] >> sh, kLongDigits - 1) : t % kLongDigits], in ? 1u : 0u);
            },
            [](int, bool, uint32_t) {});
        __syncthreads();
        uint32_t cnt = 0, inc = 0;
        if (t < kLongDigits) {
            cnt = lcur[t];
            inc = wave_sum(cnt);
            if ((t & 63u) == 63) w4[t >> 6] = inc;
        }
        __syncthreads();
        if (t < kLongDigits) {
            for (uint32_t i = 0; i < (t >> 6); ++i) inc += w4[i];
            first[t + 1] = inc;
            lcur[t] = inc - cnt;
            if (t == 0) first[0] = 0;
        }
        __syncthreads();
        const uint32_t d0 = t * G;
        if (d0 < kLongDigits) {
            const uint32_t d1 = min(d0 + G, kLongDigits), n = first[d1] - first[d0];
            const uint32_t at = n ? atomicAdd(&dsc[t], n) - first[d0] : 0u;
            for (uint32_t d = d0; d < d1; ++d) gpos[d] = at;
        }
        uint32_t to[4];
        rows_by_four<T, R>(
            len,
            [&](int r, bool in, uint32_t) {
                to[r & 3] = atomicAdd(&lcur[in ? min(key[r] >> sh, kLongDigits - 1) : t % kLongDigits], in ? 1u : 0u);
            },
            [&](int r, bool in, uint32_t i) { stage[in ? to[r & 3] : i] = key[r]; });
        __syncthreads();
        uint32_t *tmp = scratch + ((uint64_t)dsc[kDescOff + 1] << 32 | dsc[kDescOff]);
        for (uint32_t r = 0; r * T < len; r += 4) {
            uint32_t x[4];
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) x[j] = stage[(r + j) * T + t];
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) to[j] = gpos[min(x[j] >> sh, kLongDigits - 1)] + (r + j) * T + t;
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j)
                if ((r + j) * T + t < len) tmp[to[j]] = x[j];
        }
        __syncthreads();
    }
}

// Groups of sub-buckets (digits [gG, gG + G)): one block each, sorted from
// scratch into place; the ids of a group lie in [gG << sh, (gG + G) << sh).
// Two shapes: 128 x 32 for groups of at most kSubMax ids, 1024 x 32 for the
// groups of segments whose digits hold more.  item(k): the k-th of m > 0.  Items
// are read three groups ahead and descriptors two, so that no load waits for
// another.  After the split a group's cursor is its end.
template <int T, int K, int A, typename Item>
__device__ __forceinline__ void
sort_groups(uint32_t *__restrict__ ids, const uint32_t *__restrict__ scratch, const uint32_t *__restrict__ desc,
            uint32_t m, Item &&item, uint32_t *buf, uint32_t *cnt, uint32_t *wsum) {
    if (blockIdx.x >= m) return;
    const uint32_t g = gridDim.x;
    struct Raw {
        uint32_t it, s0, s1, G, lo, hi, rng;
    };
    auto look = [&](uint32_t it) {
        const uint32_t *dsc = desc + (uint64_t)(it >> 8) * kDesc;
        const uint32_t i = it & 255u;
        return Raw{it, i ? dsc[i - 1] : 0u, dsc[i], dsc[kDescGroup], dsc[kDescOff], dsc[kDescOff + 1], dsc[kDescRange]};
    };
    auto at = [&](uint32_t k) { return item(min(k, m - 1)); };
    uint32_t key[K];
    uint64_t o = 0;
    uint32_t n = 0, base = 0, range = 0;
    auto load = [&](const Raw &r) {
        // ids of digits [d0, d1): [d0 << sh, d1 << sh) within [0, rng)
        const uint32_t d0 = (r.it & 255u) * r.G, d1 = min(d0 + r.G, kLongDigits), sh = digit_shift(r.rng);
        const uint64_t end = min((uint64_t)d1 << sh, (uint64_t)r.rng);
        o = ((uint64_t)r.hi << 32 | r.lo) + r.s0;
        n = r.s1 - r.s0;
        base = d0 << sh;
        range = end > base ? (uint32_t)(end - base) : 0u;
        load_keys<T, K>(scratch + o, n, key);
    };
    load(look(at(blockIdx.x)));
    Raw nx = look(at(blockIdx.x + g));
    uint32_t it = at(blockIdx.x + 2 * g);
    for (uint32_t k = blockIdx.x; k < m; k += g) {
        const uint64_t co = o;
        const uint32_t cn = n, cb = base, cr = range;
        block_sort_keys<T, K, A>(key, ids + co, cn, cr, buf, cnt, wsum, cb, [&] {
            if (k + g < m) load(nx);
            nx = look(it);
            it = at(k + 3 * g);
        });
    }
}

__global__ void __launch_bounds__(128, 4)
segsort_sub(uint32_t *__restrict__ ids, const uint32_t *__restrict__ scratch, LongWs lw,
            const uint32_t *__restrict__ item_count) {
    constexpr int T = 128, K = 32, A = 4;
    __shared__ __align__(16) uint32_t lds[T * K + kStagePad + T * K / A];
    sort_groups<T, K, A>(ids, scratch, lw.desc, *item_count, [&](uint32_t k) { return lw.sub[k]; }, lds,
                         lds + T * K + kStagePad, lds);
}

// ---------------------------------------------------------------------------
// fallback for long segments with skewed ids: sorted tiles + pairwise merges
// ---------------------------------------------------------------------------
// Sort the 16384-id tiles of a segment in place (buf: kTileMax words of LDS).
__device__ void sort_tiles(uint32_t *seg, uint64_t c, uint32_t *buf) {
    for (uint64_t t0 = 0; t0 < c; t0 += kTileMax) {
        const uint32_t tc = (uint32_t)((c - t0) < kTileMax ? (c - t0) : kTileMax);
        uint32_t P = 1;
        while (P < tc) P <<= 1;
        for (uint32_t i = threadIdx.x; i < P; i += 1024) buf[i] = i < tc ? seg[t0 + i] : kKeyPad;
        __syncthreads();
        block_bitonic(buf, P);
        for (uint32_t i = threadIdx.x; i < tc; i += 1024) seg[t0 + i] = buf[i];
        __syncthreads();
    }
}

__device__ __forceinline__ uint32_t pidx(uint32_t i) { return i + (i >> 5); }

__device__ __forceinline__ uint32_t lds_merge_path(const uint32_t *lds, uint32_t a0, uint32_t la, uint32_t b0,
                                                   uint32_t lb, uint32_t d) {
    uint32_t lo = d > lb ? d - lb : 0;
    uint32_t hi = d < la ? d : la;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (lds[pidx(a0 + mid)] <= lds[pidx(b0 + d - mid - 1)])
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

__device__ __forceinline__ uint64_t glb_merge_path(const uint32_t *a, uint64_t la, const uint32_t *b, uint64_t lb,
                                                   uint64_t d) {
    uint64_t lo = d > lb ? d - lb : 0;
    uint64_t hi = d < la ? d : la;
    while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if (a[mid] <= b[d - mid - 1])
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Each listed segment: its 16384-id tiles sorted, then the runs merged
// pairwise until one is left; every merge proceeds in windows of 16384 outputs
// whose inputs are staged in LDS.
__device__ void sort_skewed(const uint64_t *__restrict__ offsets, uint32_t *__restrict__ ids,
                            uint32_t *__restrict__ scratch, const uint32_t *__restrict__ list, uint32_t m,
                            uint32_t *lds, uint64_t *split) {
    constexpr uint32_t T = 1024, K = 16, N = T * K;
    for (uint32_t li = blockIdx.x; li < m; li += gridDim.x) {
        const uint64_t q = list[li];
        const uint64_t o = offsets[q];
        const uint64_t c = offsets[q + 1] - o;
        uint32_t *src = ids + o, *dst = scratch + o;
        sort_tiles(src, c, lds);
        for (uint64_t w = kTileMax; w < c; w <<= 1) {
            for (uint64_t r0 = 0; r0 < c; r0 += 2 * w) {
                const uint64_t la = (c - r0) < w ? (c - r0) : w;
                const uint64_t rest = c - r0 - la;
                const uint64_t lb = rest < w ? rest : w;
                const uint32_t *A = src + r0, *B = src + r0 + la;
                uint32_t *out = dst + r0;
                for (uint64_t d0 = 0; d0 < la + lb; d0 += N) {
                    const uint64_t d1 = (d0 + N) < (la + lb) ? (d0 + N) : (la + lb);
                    if (threadIdx.x == 0) split[0] = glb_merge_path(A, la, B, lb, d0);
                    if (threadIdx.x == 1) split[1] = glb_merge_path(A, la, B, lb, d1);
                    __syncthreads();
                    const uint64_t ia0 = split[0], ia1 = split[1];
                    const uint32_t na = (uint32_t)(ia1 - ia0);
                    const uint32_t nb = (uint32_t)((d1 - d0) - na);
                    const uint64_t ib0 = d0 - ia0;
                    for (uint32_t i = threadIdx.x; i < na; i += T) lds[pidx(i)] = A[ia0 + i];
                    for (uint32_t i = threadIdx.x; i < nb; i += T) lds[pidx(na + i)] = B[ib0 + i];
                    __syncthreads();
                    uint32_t r[K];
                    const uint32_t dd = threadIdx.x * K;
                    const uint32_t tot = na + nb;
                    if (dd < tot) {
                        uint32_t ia = lds_merge_path(lds, 0, na, na, nb, dd);
                        uint32_t ib = dd - ia;
                        uint32_t a = ia < na ? lds[pidx(ia)] : kKeyPad;
                        uint32_t b = ib < nb ? lds[pidx(na + ib)] : kKeyPad;
#pragma unroll
                        for (uint32_t k = 0; k < K; ++k) {
                            const bool ta = ib >= nb || (ia < na && a <= b);
                            r[k] = ta ? a : b;
                            if (ta) {
                                ++ia;
                                a = ia < na ? lds[pidx(ia)] : kKeyPad;
                            } else {
                                ++ib;
                                b = ib < nb ? lds[pidx(na + ib)] : kKeyPad;
                            }
                        }
                    }
                    __syncthreads();
                    if (dd < tot) {
#pragma unroll
                        for (uint32_t k = 0; k < K; ++k)
                            if (dd + k < tot) lds[pidx(dd + k)] = r[k];
                    }
                    __syncthreads();
                    for (uint32_t i = threadIdx.x; i < tot; i += T) out[d0 + i] = lds[pidx(i)];
                    __syncthreads();
                }
            }
            uint32_t *t2 = src;
            src = dst;
            dst = t2;
        }
        if (src != ids + o) {
            for (uint64_t i = threadIdx.x; i < c; i += T) ids[o + i] = src[i];
        }
        __syncthreads();
    }
}

// The wide groups, then the fallback segments: one launch, as both are almost
// always empty (segments of about a million ids; skewed ids).
__global__ void __launch_bounds__(1024, 4)
segsort_rest(const uint64_t *__restrict__ offsets, uint32_t *__restrict__ ids, uint32_t *__restrict__ scratch,
             LongWs lw, const uint32_t *__restrict__ counts, const uint32_t *__restrict__ lists, uint64_t nq) {
    constexpr int T = 1024, K = 32, A = 8;
    __shared__ __align__(16) uint32_t lds[T * K + kStagePad + T * K / A];
    __shared__ uint64_t split[2];
    static_assert(T * K >= kTileMax + kTileMax / 32, "a padded merge window");
    sort_groups<T, K, A>(ids, scratch, lw.desc, counts[kSubCounts + 1], [&](uint32_t k) { return *(lw.sub_end - 1 - k); }, lds,
                         lds + T * K + kStagePad, lds);
    sort_skewed(offsets, ids, scratch, lists + kFallback * nq, counts[kFallback], lds, split);
}

// Batches of at most kFewMax segments: one block per segment sorts it if it
// has at most 4096 ids and lists it for the longer shapes otherwise, so that a
// small select needs no classification pass and one launch where its ids are
// few (each launch costs a small call about 3 us).
constexpr uint32_t kFewMax = 2048;
constexpr uint32_t kFewIds = 4096;

__global__ void __launch_bounds__(256, 6)
segsort_few(const uint64_t *__restrict__ offsets, uint32_t nq, uint64_t cap, uint32_t *__restrict__ ids,
            uint32_t *__restrict__ lists, uint32_t *__restrict__ counts, LongWs lw, uint32_t id_range,
            const uint32_t *__restrict__ seg_range, const Ctrl *__restrict__ ctrl, uint64_t *__restrict__ status) {
    constexpr uint32_t T = 256, K = 16, N = T * K;
    static_assert(N == kFewIds, "one tile per segment");
    __shared__ __align__(16) uint32_t lds[N + kStagePad + N / 4];
    const uint32_t q = blockIdx.x;
    if (status && q == 0 && threadIdx.x == 0) select_status(offsets, nq, cap, ctrl, status);
    const uint64_t o = offsets[q], len = offsets[q + 1] - o;
    if (len < 2 || offsets[nq] > cap) return;
    if (len > kFewIds) {
        const uint32_t np = len > kMidMax ? num_parts(len) : 0u;
        if (threadIdx.x == 0) {
            const uint32_t j = np ? kLong : 4u, li = atomicAdd(&counts[j], 1u);
            lists[(uint64_t)j * nq + li] = q;
            lds[0] = li;
            if (np) lds[1] = atomicAdd(&counts[kPartCount], np);
        }
        __syncthreads();
        const uint32_t sh = digit_shift(seg_id_range(seg_range, q, id_range));
        for (uint32_t d = threadIdx.x; np && d < kLongDigits; d += T) lw.desc[(uint64_t)lds[0] * kDesc + d] = 0;
        for (uint32_t p = threadIdx.x; p < np; p += T) lw.parts[lds[1] + p] = part_item(lds[0], p, o, len, sh);
        return;
    }
    const uint32_t c = (uint32_t)len;
    if (c <= 256) {
        if (threadIdx.x >= 64) return;   // no barrier below
        uint32_t v[4];
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t k = r * 64 + threadIdx.x;
            v[r] = k < c ? ids[o + k] : kKeyPad;
        }
        wave_sort_regs4(v, ids + o, c);
        return;
    }
    uint32_t key[K];
    load_keys<T, K>(ids + o, c, key);
    block_sort_keys<T, K, 4>(key, ids + o, c, seg_id_range(seg_range, q, id_range), lds, lds + N + kStagePad, lds,
                                 0, [] {});
}

uint64_t segsort_ws_elems(uint64_t nq) { return (uint64_t)kListCls * nq + kSortCounters; }

uint64_t segsort_scratch_elems(uint64_t cap) { return sort_scratch_words(cap); }

template <typename Kern>
static uint32_t resident_per_cu(Kern kern, int threads) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kern, threads, 0) != hipSuccess || n < 1) n = 1;
    return (uint32_t)n;
}

hipError_t launch_segsort(const uint64_t *offsets, uint64_t nq, uint32_t *ids, uint32_t *scratch, uint64_t cap,
                          uint32_t *ws, uint64_t id_range, const uint32_t *seg_range, bool zeroed, const Ctrl *ctrl,
                          uint64_t *status, hipStream_t s) {
    if (nq == 0) return hipSuccess;
    const uint32_t range = (uint32_t)(id_range < 0xFFFFFFFFull ? id_range : 0xFFFFFFFFull);
    uint32_t *counts = ws;                    // class counters
    uint32_t *lists = ws + kSortCounters;     // kListCls lists of up to nq query indices
    const uint32_t cus = (uint32_t)num_cus();
    // blocks per CU that fit at once (registers and LDS): each persistent
    // grid holds that many, so no block waits for another to finish its share
    static const uint32_t g_small = resident_per_cu(segsort_small, 256);
    static const uint32_t g_m1 = resident_per_cu(segsort_mid<64, 16, 4>, 64);
    static const uint32_t g_m2 = resident_per_cu(segsort_mid<128, 32, 4>, 128);
    static const uint32_t g_m3 = resident_per_cu(segsort_mid<512, 32, 8>, 512);
    static const uint32_t g_wide = resident_per_cu(segsort_wide, 1024);
    static const uint32_t g_split = resident_per_cu(segsort_part_split<1024>, 1024);
    static const uint32_t g_sub = resident_per_cu(segsort_sub, 128);
    static const uint32_t g_rest = resident_per_cu(segsort_rest, 1024);
    // no more blocks than the class can have work items: nq segments, or as
    // many longer than `longer` as fit the capacity (none: no launch)
    auto most = [&](uint32_t longer) { return std::min<uint64_t>(nq, cap / (longer + 1ull)); };
    auto grid = [&](uint32_t resident, uint64_t items) {
        return dim3((uint32_t)std::min<uint64_t>((uint64_t)cus * resident, items));
    };
    const LongSpace at = long_space(reinterpret_cast<uintptr_t>(scratch), cap);
    const LongWs lw{reinterpret_cast<uint4 *>(scratch + at.parts), scratch + at.desc, scratch + at.sub, scratch + at.end};
    hipError_t e = hipSuccess;
    if (!zeroed) e = launch_zero(counts, kSortCounters * 4, s);
    if (e != hipSuccess) return e;
    // every class on the caller's stream, shortest first (an extra stream
    // per call site would take one of the device's few hardware queues from
    // whatever else the process runs concurrently)
    if (nq <= kFewMax) {
        hipLaunchKernelGGL(segsort_few, dim3((uint32_t)nq), dim3(256), 0, s, offsets, (uint32_t)nq, cap, ids, lists,
                           counts, lw, range, seg_range, ctrl, status);
    } else {
        if (nq <= 262144)
            hipLaunchKernelGGL(seg_classify<2>, dim3((uint32_t)((nq + 511) / 512)), dim3(256), 0, s, offsets, nq, cap,
                               lists, counts, lw, range, seg_range, ctrl, status);
        else
            hipLaunchKernelGGL(seg_classify<16>, dim3((uint32_t)((nq + 4095) / 4096)), dim3(256), 0, s, offsets, nq,
                               cap, lists, counts, lw, range, seg_range, ctrl, status);
        if (most(1))
            hipLaunchKernelGGL(segsort_small, grid(g_small, (most(1) + 3) / 4), dim3(256), 0, s, offsets, ids, lists,
                               counts + 0);
        if (most(256))
            hipLaunchKernelGGL((segsort_mid<64, 16, 4>), grid(g_m1, most(256)), dim3(64), 0, s, offsets,
                               ids, lists + nq, counts + 1, range, seg_range);
        if (most(1024))
            hipLaunchKernelGGL((segsort_mid<128, 32, 4>), grid(g_m2, most(1024)), dim3(128), 0, s,
                               offsets, ids, lists + 2 * nq, counts + 2, range, seg_range);
        if (most(4096))
            hipLaunchKernelGGL((segsort_mid<512, 32, 8>), grid(g_m3, most(4096)), dim3(512), 0, s,
                               offsets, ids, lists + 3 * nq, counts + 3, range, seg_range);
    }
    const uint32_t wide_min = nq <= kFewMax ? kFewIds : 16384;
    const uint64_t nl = most(kMidMax), np = nl ? cap / kPart + nl : 0;   // class-L segments and parts at most
    if (most(wide_min))
        hipLaunchKernelGGL(segsort_wide, grid(g_wide, std::max(most(wide_min), np)), dim3(1024), 0, s, offsets, ids,
                           lists, nq, counts, lw, range, seg_range);
    if (nl) {
        hipLaunchKernelGGL(segsort_part_scan, grid(8, nl), dim3(256), 0, s, offsets, lists + kLong * nq,
                           counts + kLong, lw, counts + kSubCounts, lists + kFallback * nq, counts + kFallback, range,
                           seg_range);
        hipLaunchKernelGGL(segsort_part_split<1024>, grid(g_split, np), dim3(1024), 0, s, ids, scratch,
                           counts + kPartCount, lw);
        hipLaunchKernelGGL(segsort_sub, grid(g_sub, nl * kLongDigits), dim3(128), 0, s, ids, scratch, lw,
                           counts + kSubCounts);
        hipLaunchKernelGGL(segsort_rest, grid(g_rest, nl * kLongDigits), dim3(1024), 0, s, offsets, ids, scratch, lw,
                           counts, lists, nq);
    }
    return hipGetLastError();
}

}  // namespace rtk
