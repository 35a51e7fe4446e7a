// R-tree join kernels for gfx950: synchronized traversal of two trees.
//
// The paper's join (section 4) starts at both roots and follows every pair of
// intersecting children.  Its vectorized "one to many" form broadcasts one
// outer child MBR and compares it with all inner children at once (section
// 4.1, steps 1-3), then compress-stores the qualifying inner addresses and
// duplicates the outer address beside them (step 4).
//
// On the GPU the pairs of one tree level form a frontier that is processed
// level by level, one wave per node pair.  The wave covers the Fa x Fb tile of
// child pairs 64 at a time: lane l of round r tests outer child i and inner
// child j with r*64 + l = i*Fb + j, so each round compares (64/Fb) outer
// children against all inner children -- the one-to-many comparison, widened
// from one broadcast outer MBR to several.  Qualifying pairs are compacted
// with __ballot + popcount ranks into the next frontier (count pass, scan,
// fill pass) or, at the leaf level, written out as 64-bit (idA << 32 | idB)
// keys, which are then sorted (bucket sort at the end of this file) into the
// canonical pair order.
//
// Trees of unequal height: only the deeper side descends, with each of its
// children tested against the MBR of the whole shallower tree, until both
// sides are at the same level (this can only happen at the roots).
#include <algorithm>

#include "pair_sort.h"
#include "rt_internal.h"

namespace rtk {

constexpr uint32_t kSlotHits = 15;     // hit records kept per pair by the count pass
constexpr uint32_t kSlotStride = 16;   // uint16 per pair (32 bytes)

__device__ __forceinline__ void load_any(const TreeView &t, uint32_t node, uint32_t e, float &lx, float &ly,
                                         float &hx, float &hy) {
    const uint8_t *nb = t.nodes + (size_t)node * t.node_bytes;
    const uint32_t F = t.fanout;
    if (t.layout == LAYOUT_SOA) {
        const float *f = reinterpret_cast<const float *>(nb);
        lx = f[e];
        ly = f[F + e];
        hx = f[2 * F + e];
        hy = f[3 * F + e];
    } else if (t.layout == LAYOUT_AOS) {
        const float *f = reinterpret_cast<const float *>(nb) + 5 * e;
        lx = f[0];
        ly = f[1];
        hx = f[2];
        hy = f[3];
    } else {
        const float2 *lo = reinterpret_cast<const float2 *>(nb);
        const float2 a = lo[e], b = lo[F + e];
        lx = a.x;
        ly = a.y;
        hx = b.x;
        hy = b.y;
    }
}

__device__ __forceinline__ uint32_t ptr_any(const TreeView &t, uint32_t node, uint32_t e) {
    const uint32_t *u = reinterpret_cast<const uint32_t *>(t.nodes + (size_t)node * t.node_bytes);
    return t.layout == LAYOUT_AOS ? u[5 * e + 4] : u[4 * t.fanout + e];
}

// One wave per frontier pair; 4 pairs per block.  tests_acc (count pass
// only, NULL: not counted): per pair, the entry-pair predicates of a pair at
// equal levels (n_u * n_v real entries) are added to slot word 0, the real
// entries loaded (n_u + n_v, or the deeper node's n) to word 1 and the
// entry-versus-tree predicates of a descending pair to word 2.
template <int MODE, bool FILL>
__global__ void __launch_bounds__(256)
join_level_kernel(TreeView A, TreeView B, const uint2 *__restrict__ fr, uint32_t nfr,
                  const uint64_t *__restrict__ nfr_dev, uint32_t *__restrict__ counts,
                  const uint64_t *__restrict__ offsets, uint2 *__restrict__ next, uint64_t *__restrict__ keys,
                  uint64_t out_cap, Ctrl *__restrict__ ctrl, unsigned long long *__restrict__ tests_acc) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t p = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (nfr_dev && *nfr_dev < nfr) nfr = (uint32_t)*nfr_dev;
    if (p >= nfr) return;   // whole wave leaves together
    const uint2 pr = fr[p];
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    uint64_t pos = 0, end = 0;
    if (FILL) {
        pos = offsets[p];
        end = min(offsets[p + 1], out_cap);
    }
    uint32_t total = 0;

    if constexpr (MODE == JOIN_DESC_A || MODE == JOIN_DESC_B) {
        // Deeper side descends; each child is tested against the shallower
        // tree's MBR.  One round covers a node (F <= 64).
        const TreeView &D = (MODE == JOIN_DESC_A) ? A : B;
        const TreeView &S = (MODE == JOIN_DESC_A) ? B : A;
        const uint32_t node = (MODE == JOIN_DESC_A) ? pr.x : pr.y;
        bool hit = false, real = false;
        if (lane < D.fanout) {
            float lx, ly, hx, hy;
            load_any(D, node, lane, lx, ly, hx, hy);
            hit = (lx <= S.mbr[2]) && (S.mbr[0] <= hx) && (ly <= S.mbr[3]) && (S.mbr[1] <= hy);
            real = lx == lx;   // not a padding slot
        }
        const uint64_t m = __ballot(hit);
        total = (uint32_t)__popcll(m);
        if (!FILL && tests_acc) {
            const uint32_t nd = (uint32_t)__popcll(__ballot(real));
            if (lane == 0) {
                atomicAdd(&tests_acc[(p % kTestSlots) * 16 + 1], (unsigned long long)nd);
                atomicAdd(&tests_acc[(p % kTestSlots) * 16 + 2], (unsigned long long)nd);
            }
        }
        if (FILL && hit) {
            const uint64_t o = pos + (uint64_t)__popcll(m & below);
            const uint32_t c = ptr_any(D, node, lane);
            if (o < end)
                next[o] = (MODE == JOIN_DESC_A) ? make_uint2(c, pr.y) : make_uint2(pr.x, c);
            else if (o < out_cap)
                atomicOr(&ctrl->err, kErrBounds);
        }
    } else {
        const uint32_t Fa = A.fanout, Fb = B.fanout;
        const uint32_t tile = Fa * Fb;
        // lane's (i, j) for round 0 and the per-round advance
        uint32_t i = lane / Fb, j = lane % Fb;
        const uint32_t di = 64 / Fb, dj = 64 % Fb;
        uint32_t real_pairs = 0;
        for (uint32_t base = 0; base < tile; base += 64) {
            const bool in = base + lane < tile;
            bool hit = false, real = false;
            if (in) {
                float alx, aly, ahx, ahy, blx, bly, bhx, bhy;
                load_any(A, pr.x, i, alx, aly, ahx, ahy);
                load_any(B, pr.y, j, blx, bly, bhx, bhy);
                hit = (alx <= bhx) && (blx <= ahx) && (aly <= bhy) && (bly <= ahy);
                real = (alx == alx) && (blx == blx);   // neither is a padding slot
            }
            const uint64_t m = __ballot(hit);
            const uint32_t n = (uint32_t)__popcll(m);
            if (!FILL && tests_acc) real_pairs += (uint32_t)__popcll(__ballot(real));
            if (FILL && hit) {
                const uint64_t o = pos + total + (uint64_t)__popcll(m & below);
                const uint32_t ca = ptr_any(A, pr.x, i), cb = ptr_any(B, pr.y, j);
                if (o < end) {
                    if (MODE == JOIN_EMIT)
                        keys[o] = ((uint64_t)ca << 32) | cb;
                    else
                        next[o] = make_uint2(ca, cb);
                } else if (o < out_cap) {
                    atomicOr(&ctrl->err, kErrBounds);
                }
            }
            total += n;
            i += di;
            j += dj;
            if (j >= Fb) {
                j -= Fb;
                i += 1;
            }
        }
        if (!FILL && tests_acc) {
            float x, y, z, w;
            bool ra = false, rb = false;
            if (lane < Fa) {
                load_any(A, pr.x, lane, x, y, z, w);
                ra = x == x;
            }
            if (lane < Fb) {
                load_any(B, pr.y, lane, x, y, z, w);
                rb = x == x;
            }
            const uint32_t ne = (uint32_t)(__popcll(__ballot(ra)) + __popcll(__ballot(rb)));
            if (lane == 0) {
                atomicAdd(&tests_acc[(p % kTestSlots) * 16], (unsigned long long)real_pairs);
                atomicAdd(&tests_acc[(p % kTestSlots) * 16 + 1], (unsigned long long)ne);
            }
        }
    }
    if (!FILL && lane == 0) counts[p] = total;
}

// ---------------------------------------------------------------------------
// A level in one pass (replayed joins, whose buffers are sized already).
//
// The order of a frontier and of the keys is free (the keys are sorted at the
// end), so no offsets are needed: a block enumerates a few pairs per wave,
// collects the hits as (pair, i, j) codes in LDS, reserves as many places as
// there are with one atomic (one per wave would be 17 ns each, one after the
// other) and writes them, the child ids of all hits looked up at once.  If
// they outgrow the LDS list the block enumerates its pairs again and writes
// directly.  Places past out_cap are not written and set *over.
//
// Enumerating a pair: the entries of both nodes that do not reach into the
// other node's MBR have no hits; the rest are packed in LDS, the inner ones
// held one per lane (in as many copies as fit the wave), the outer ones read
// as broadcasts, 64 predicates a round.  Of 32 entries about 12 stay, three
// rounds in place of 16; the candidate lists by low x (below) cut about as
// many predicates but took some 60 lane permutes per pair, and bound the
// count pass by the LDS (2M x 2M rectangles, about 0.2M leaf pairs: count,
// scan and fill 253 us, here 89 us, bound by vector instructions, some 210 per
// pair).
// ---------------------------------------------------------------------------
constexpr uint32_t kOnceWaves = 16;
constexpr uint32_t kOncePairs = 8;     // pairs per wave at most
constexpr uint32_t kOnceBuf = 4096;    // hits a block collects

// Floats as integers of the same order (-0 below +0), and back.
__device__ __forceinline__ int ordered(float v) {
    const int i = __float_as_int(v);
    return i ^ ((i >> 31) & 0x7FFFFFFF);
}
__device__ __forceinline__ float unordered(int i) { return __int_as_float(i ^ ((i >> 31) & 0x7FFFFFFF)); }
// Smallest (SIGN < 0) or largest value of lanes 0..31 (in lane 31) and of
// 32..63, of all lanes with WAVE (in lane 63).  As integers, a step is one
// instruction; as floats each would canonicalize first.
template <int CTRL, int ROWS, int SIGN>
__device__ __forceinline__ int lanes_step(int v) {
    const int o = __builtin_amdgcn_update_dpp(SIGN < 0 ? 0x7FFFFFFF : -0x7FFFFFFF - 1, v, CTRL, ROWS, 0xF, false);
    return SIGN < 0 ? min(v, o) : max(v, o);
}
template <bool WAVE, int SIGN>
__device__ __forceinline__ int lanes_extreme(int v) {
    v = lanes_step<0x111, 0xF, SIGN>(v);
    v = lanes_step<0x112, 0xF, SIGN>(v);
    v = lanes_step<0x114, 0xF, SIGN>(v);
    v = lanes_step<0x118, 0xF, SIGN>(v);
    v = lanes_step<0x142, 0xA, SIGN>(v);
    if (WAVE) v = lanes_step<0x143, 0xC, SIGN>(v);
    return v;
}
__device__ __forceinline__ float lane_f(int v, int lane) { return unordered(__builtin_amdgcn_readlane(v, lane)); }

// PACK: both nodes have at most 32 entries, so lanes 0..31 take one and lanes
// 32..63 the other.
template <int MODE, bool PACK>
__global__ void __launch_bounds__(1024, 8)
join_once_kernel(TreeView A, TreeView B, const uint2 *__restrict__ fr, uint32_t nfr,
                 const uint64_t *__restrict__ nfr_dev, uint32_t per_wave, uint2 *__restrict__ next,
                 uint64_t *__restrict__ keys, uint64_t out_cap, unsigned long long *__restrict__ count,
                 uint32_t *__restrict__ over) {
    __shared__ float4 box[kOnceWaves][128];     // packed outer entries, then (from 64) inner ones
    __shared__ uint8_t at[kOnceWaves][128];     // their places in the nodes
    __shared__ uint32_t buf[kOnceBuf], bn;
    __shared__ unsigned long long gbase;
    if (nfr_dev && *nfr_dev < nfr) nfr = (uint32_t)*nfr_dev;
    const uint32_t t = threadIdx.x, lane = t & 63u, w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
    const uint32_t p0 = blockIdx.x * (kOnceWaves * per_wave);
    if (p0 >= nfr) return;   // the whole block
    const uint32_t pend = min(nfr - p0, kOnceWaves * per_wave);
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    const uint32_t Fa = A.fanout, Fb = B.fanout;
    auto put = [&](uint32_t code, uint64_t o) {
        if (o >= out_cap) return;
        const uint2 pr = fr[p0 + (code >> 12)];
        const uint32_t ca = ptr_any(A, pr.x, (code >> 6) & 63u), cb = ptr_any(B, pr.y, code & 63u);
        if (MODE == JOIN_EMIT)
            keys[o] = ((uint64_t)ca << 32) | cb;
        else
            next[o] = make_uint2(ca, cb);
    };
    struct Entry {
        float lx, ly, hx, hy;
    };
    // lane's entry of the pair: NaN past the node's entries, as unused slots
    Entry a, b;
    auto load = [&](uint32_t k) {
        const uint2 pr = fr[p0 + min(k, pend - 1)];
        a = b = {NAN, NAN, NAN, NAN};
        if constexpr (PACK) {
            const uint32_t e = lane & 31u;
            if (lane < 32) {
                if (e < Fa) load_any(A, pr.x, e, a.lx, a.ly, a.hx, a.hy);
            } else {
                if (e < Fb) load_any(B, pr.y, e, a.lx, a.ly, a.hx, a.hy);
            }
        } else {
            if (lane < Fa) load_any(A, pr.x, lane, a.lx, a.ly, a.hx, a.hy);
            if (lane < Fb) load_any(B, pr.y, lane, b.lx, b.ly, b.hx, b.hy);
        }
    };
    // all pairs of the wave; sink(code, hit, hits of the round)
    auto pairs = [&](auto &&sink) {
        load(w);
        for (uint32_t k = w; k < pend; k += kOnceWaves) {
            const Entry ca = a, cb = b;
            if (k + kOnceWaves < pend) load(k + kOnceWaves);
            uint32_t na, nb;
            if constexpr (PACK) {
                const bool real = ca.lx == ca.lx;
                const int lo = ordered(INFINITY), up = ordered(-INFINITY);   // of unused slots
                const int lx = lanes_extreme<false, -1>(real ? ordered(ca.lx) : lo);
                const int ly = lanes_extreme<false, -1>(real ? ordered(ca.ly) : lo);
                const int hx = lanes_extreme<false, 1>(real ? ordered(ca.hx) : up);
                const int hy = lanes_extreme<false, 1>(real ? ordered(ca.hy) : up);
                // the other half's MBR
                const bool hi = lane >= 32;
                const float olx = hi ? lane_f(lx, 31) : lane_f(lx, 63), oly = hi ? lane_f(ly, 31) : lane_f(ly, 63);
                const float ohx = hi ? lane_f(hx, 31) : lane_f(hx, 63), ohy = hi ? lane_f(hy, 31) : lane_f(hy, 63);
                const bool keep = ca.lx <= ohx && olx <= ca.hx && ca.ly <= ohy && oly <= ca.hy;
                const uint64_t m = __ballot(keep);
                na = (uint32_t)__popc((uint32_t)m);
                nb = (uint32_t)__popc((uint32_t)(m >> 32));
                if (keep) {
                    const uint32_t r = (uint32_t)__popcll(m & below);
                    const uint32_t to = hi ? 64 + r - na : r;
                    box[w][to] = make_float4(ca.lx, ca.ly, ca.hx, ca.hy);
                    at[w][to] = (uint8_t)(lane & 31u);
                }
            } else {
                const bool ra = ca.lx == ca.lx, rb = cb.lx == cb.lx;
                const int lo = ordered(INFINITY), up = ordered(-INFINITY);   // of unused slots
                const float alx = lane_f(lanes_extreme<true, -1>(ra ? ordered(ca.lx) : lo), 63);
                const float aly = lane_f(lanes_extreme<true, -1>(ra ? ordered(ca.ly) : lo), 63);
                const float ahx = lane_f(lanes_extreme<true, 1>(ra ? ordered(ca.hx) : up), 63);
                const float ahy = lane_f(lanes_extreme<true, 1>(ra ? ordered(ca.hy) : up), 63);
                const float blx = lane_f(lanes_extreme<true, -1>(rb ? ordered(cb.lx) : lo), 63);
                const float bly = lane_f(lanes_extreme<true, -1>(rb ? ordered(cb.ly) : lo), 63);
                const float bhx = lane_f(lanes_extreme<true, 1>(rb ? ordered(cb.hx) : up), 63);
                const float bhy = lane_f(lanes_extreme<true, 1>(rb ? ordered(cb.hy) : up), 63);
                const bool ka = ca.lx <= bhx && blx <= ca.hx && ca.ly <= bhy && bly <= ca.hy;
                const bool kb = cb.lx <= ahx && alx <= cb.hx && cb.ly <= ahy && aly <= cb.hy;
                const uint64_t ma = __ballot(ka), mb = __ballot(kb);
                na = (uint32_t)__popcll(ma);
                nb = (uint32_t)__popcll(mb);
                if (ka) {
                    const uint32_t to = (uint32_t)__popcll(ma & below);
                    box[w][to] = make_float4(ca.lx, ca.ly, ca.hx, ca.hy);
                    at[w][to] = (uint8_t)lane;
                }
                if (kb) {
                    const uint32_t to = 64 + (uint32_t)__popcll(mb & below);
                    box[w][to] = make_float4(cb.lx, cb.ly, cb.hx, cb.hy);
                    at[w][to] = (uint8_t)lane;
                }
            }
            __builtin_amdgcn_wave_barrier();
            if (na && nb) {   // wave-uniform
                // copies of the inner entries side by side: 64 >> sh outer ones a round
                const uint32_t sh = nb > 1 ? 32 - __builtin_clz(nb - 1) : 0;
                const uint32_t j = lane & ((1u << sh) - 1u), row = lane >> sh, rows = 64u >> sh;
                const float4 in = box[w][64 + min(j, nb - 1)];
                for (uint32_t r = 0; r < na; r += rows) {
                    const uint32_t i = r + row;
                    const float4 o = box[w][min(i, na - 1)];
                    const bool hit = j < nb && i < na && o.x <= in.z && in.x <= o.z && o.y <= in.w && in.y <= o.w;
                    const uint64_t m = __ballot(hit);
                    if (m) {
                        const uint32_t code = hit ? k << 12 | (uint32_t)at[w][i] << 6 | at[w][64 + j] : 0u;
                        uint32_t pos = 0;
                        if (lane == 0) pos = atomicAdd(&bn, (uint32_t)__popcll(m));
                        pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)pos) + (uint32_t)__popcll(m & below);
                        sink(code, hit, pos);
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    };
    if (t == 0) bn = 0;
    __syncthreads();
    pairs([&](uint32_t code, bool hit, uint32_t pos) {
        if (hit && pos < kOnceBuf) buf[pos] = code;
    });
    __syncthreads();
    const uint32_t n = bn;
    if (n == 0) return;
    if (t == 0) {
        gbase = atomicAdd(count, (unsigned long long)n);
        if (gbase + n > out_cap) atomicOr(over, 1u);
    }
    __syncthreads();
    const uint64_t base = gbase;
    if (n <= kOnceBuf) {
        for (uint32_t x = t; x < n; x += 1024) put(buf[x], base + x);
        return;
    }
    if (t == 0) bn = 0;
    __syncthreads();
    pairs([&](uint32_t code, bool hit, uint32_t pos) {
        if (hit) put(code, base + pos);
    });
}

hipError_t launch_join_once(const TreeView &a, const TreeView &b, const uint2 *fr, uint32_t nfr, const uint64_t *nd,
                            int mode, uint2 *next, uint64_t *keys, uint64_t cap, uint64_t *count, uint32_t *over,
                            hipStream_t s) {
    if (nfr == 0) return hipSuccess;
    // about three blocks per CU before a wave takes a second pair
    const uint32_t per = std::min(kOncePairs, nfr / (kOnceWaves * 3 * (uint32_t)num_cus()) + 1);
    const dim3 grid((nfr + kOnceWaves * per - 1) / (kOnceWaves * per)), block(kOnceWaves * 64);
    unsigned long long *c = reinterpret_cast<unsigned long long *>(count);
    const bool pack = a.fanout <= 32 && b.fanout <= 32;
#define RT_ONCE(M_, P_) \
    hipLaunchKernelGGL((join_once_kernel<M_, P_>), grid, block, 0, s, a, b, fr, nfr, nd, per, next, keys, cap, c, over)
    if (mode == JOIN_EMIT) {
        if (pack) RT_ONCE(JOIN_EMIT, true);
        else RT_ONCE(JOIN_EMIT, false);
    } else {
        if (pack) RT_ONCE(JOIN_BOTH, true);
        else RT_ONCE(JOIN_BOTH, false);
    }
#undef RT_ONCE
    return hipGetLastError();
}

// Clears what a replayed join counts into: the status, the level sizes and
// the overflow flag (nlv words), the bucket counts (if not NULL), and sets
// level 0 to the pair of roots.
__global__ void __launch_bounds__(256)
join_init_kernel(Ctrl *__restrict__ ctrl, uint64_t *__restrict__ lv, uint32_t nlv, uint2 *__restrict__ fr0,
                 uint32_t *__restrict__ cnt) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    for (uint32_t k = i; k < sizeof(Ctrl) / 4; k += gridDim.x * 256) reinterpret_cast<uint32_t *>(ctrl)[k] = 0;
    for (uint32_t k = i; k < nlv; k += gridDim.x * 256) lv[k] = 0;
    if (i == 0) *fr0 = make_uint2(0u, 0u);
    if (cnt && i < kPairBuckets) cnt[i] = 0;
}

hipError_t launch_join_init(Ctrl *ctrl, uint64_t *lv, uint32_t nlv, uint2 *fr0, uint32_t *cnt, hipStream_t s) {
    hipLaunchKernelGGL(join_init_kernel, dim3(kPairBuckets / 256), dim3(256), 0, s, ctrl, lv, nlv, fr0, cnt);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Node-pair expansion over candidate lists (section 4.1 pruning, section 4.2
// many-to-many).  One wave per frontier pair; lane i holds outer child i of
// node u (tree A) and lane j inner child j of node v (tree B) in registers,
// loaded once.  Each outer lane i gets a count f_i of inner candidates, the
// inner children 0..f_i-1:
//   no pruning          f_i = number of inner children
//   O3 (outer slicing)  f_i = 0 unless outer low x <= max inner high x; with
//                       children sorted by low x this keeps a prefix of the
//                       outer node (the first child that fails ends the scan)
//   O4 (one to many)    for each kept outer child, its high x is broadcast and
//                       compared with every inner low x in one ballot; f_i is
//                       the length of the leading run of qualifying children
//   O5 (many to many)   every outer lane searches the sorted inner low x on
//                       its own: gather at n/2, compare, and on a clear bit
//                       record the flip index and step down, else step up,
//                       log2(n)+1 rounds -- the same f_i as O4
// The candidates (i, j < f_i) are then enumerated 64 per round through an
// exclusive scan of f: lane t finds its i by a binary search over the scan
// and j = t - scan[i], fetches both MBRs from their lanes and applies the
// full overlap predicate.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float wave_max(float v) {
    for (int d = 32; d >= 1; d >>= 1) v = fmaxf(v, __shfl_xor(v, d));
    return v;
}

// exclusive prefix sum over the wave; *total receives the sum
__device__ __forceinline__ uint32_t wave_excl_scan(uint32_t v, uint32_t lane, uint32_t *total) {
    uint32_t inc = v;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t x = __shfl_up(inc, d);
        if (lane >= (uint32_t)d) inc += x;
    }
    *total = __shfl(inc, 63);
    return inc - v;
}

// slots (if not NULL): kSlotHits hit records (i << 8 | j) per pair, written
// by the count pass; the fill pass of a pair with at most that many hits
// takes its children from there instead of testing the candidates again.
// Every lane searches the values v (lane g holds entry g; entries 0..n-1 are
// sorted so that pred holds on a prefix) for the first entry where pred
// fails, n if none: the many-to-many search of section 4.2 (gather at n/2,
// compare, step by halves, log2(n)+1 rounds), each lane with its own pred.
template <class Pred>
__device__ __forceinline__ uint32_t first_failing(float v_lane, uint32_t n, Pred pred) {
    uint32_t npow = 1, lg = 0;
    while (npow < n) {
        npow <<= 1;
        ++lg;
    }
    int g = (int)(npow >> 1);
    uint32_t flip = npow;
    for (uint32_t it = 0; it <= lg; ++it) {
        const float v = __shfl(v_lane, g & 63);
        const bool in = g >= 0 && (uint32_t)g < npow;
        const bool bit = (uint32_t)g < n && pred(v);
        const int step = (it + 2 <= lg) ? (int)(npow >> (it + 2)) : 1;
        if (in) {
            if (bit) {
                g += step;
            } else {
                flip = (uint32_t)g;
                g -= step;
            }
        }
    }
    return flip;
}

template <int MODE, bool FILL, bool O3, int SHRINK, bool LB>
__global__ void __launch_bounds__(256)
join_cand_kernel(TreeView A, TreeView B, const uint2 *__restrict__ fr, uint32_t nfr,
                 const uint64_t *__restrict__ nfr_dev, uint32_t *__restrict__ counts,
                 const uint64_t *__restrict__ offsets, uint2 *__restrict__ next, uint64_t *__restrict__ keys,
                 uint64_t out_cap, uint16_t *__restrict__ slots, Ctrl *__restrict__ ctrl,
                 unsigned long long *__restrict__ tests_acc) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t p = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (nfr_dev && *nfr_dev < nfr) nfr = (uint32_t)*nfr_dev;
    if (p >= nfr) return;   // whole wave leaves together
    const uint2 pr = fr[p];
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    if (FILL && slots) {
        const uint64_t pos = offsets[p], end = min(offsets[p + 1], out_cap);
        const uint64_t n = offsets[p + 1] - pos;
        if (n <= kSlotHits) {   // wave-uniform
            if (lane < n) {
                const uint32_t h = slots[(uint64_t)p * kSlotStride + lane];
                const uint32_t ca = ptr_any(A, pr.x, h >> 8), cb = ptr_any(B, pr.y, h & 255u);
                const uint64_t o = pos + lane;
                if (o < end) {
                    if (MODE == JOIN_EMIT)
                        keys[o] = ((uint64_t)ca << 32) | cb;
                    else
                        next[o] = make_uint2(ca, cb);
                }
            }
            return;
        }
    }
    float alx = NAN, aly = NAN, ahx = NAN, ahy = NAN, blx = NAN, bly = NAN, bhx = NAN, bhy = NAN;
    if (lane < A.fanout) load_any(A, pr.x, lane, alx, aly, ahx, ahy);
    if (lane < B.fanout) load_any(B, pr.y, lane, blx, bly, bhx, bhy);
    // unused slots hold NaN and sit after the used ones
    const bool av = alx == alx, bv = blx == blx;
    const uint32_t nb = (uint32_t)__popcll(__ballot(bv));
    bool act = av;
    if (O3) {
        const float m = wave_max(bv ? bhx : -INFINITY);
        act = av && alx <= m;
    }
    uint32_t f = nb;
    if (SHRINK == 4) {
        f = 0;
        uint64_t todo = __ballot(act);
        while (todo) {
            const uint32_t i = (uint32_t)__builtin_ctzll(todo);
            todo &= todo - 1;
            const float h = __shfl(ahx, (int)i);
            const uint64_t q = __ballot(bv && blx <= h);
            const uint32_t stop = ~q ? (uint32_t)__builtin_ctzll(~q) : 64u;
            if (lane == i) f = stop;
        }
    } else if (SHRINK == 5) {
        f = first_failing(blx, nb, [&](float v) { return v <= ahx; });
    }
    // LB (lower bound, not in the paper): inner children are sorted by low
    // x and none is wider than wmax, so one whose low x lies below
    // olx - wmax ends left of the outer child and cannot qualify.  The bound
    // is lowered by a margin far above the rounding of its two subtractions,
    // so no qualifying pair is ever cut; candidates are j in [lo, f).
    uint32_t lo = 0;
    if (LB) {
        const float wmax = wave_max(bv ? bhx - blx : -INFINITY);
        const float thr = (alx - wmax) - (fabsf(alx) + wmax) * 0x1p-20f;
        lo = first_failing(blx, nb, [&](float v) { return v < thr; });
        lo = min(lo, f);
    }
    if (!act) f = lo = 0;
    uint32_t T = 0;
    const uint32_t pre = wave_excl_scan(f - lo, lane, &T);
    const int jbase = (int)lo - (int)pre;   // j = t + jbase of the outer child
    uint64_t pos = 0, end = 0;
    if (FILL) {
        pos = offsets[p];
        end = min(offsets[p + 1], out_cap);
    }
    uint32_t total = 0;
    for (uint32_t base = 0; base < T; base += 64) {
        const uint32_t t = base + lane;
        uint32_t i = 0;
        for (uint32_t sft = 32; sft >= 1; sft >>= 1) {
            const uint32_t c = __shfl(pre, (int)(i + sft));
            if (c <= t) i += sft;
        }
        const uint32_t j = min((uint32_t)((int)t + __shfl(jbase, (int)i)), 63u);
        const float olx = __shfl(alx, (int)i), oly = __shfl(aly, (int)i);
        const float ohx = __shfl(ahx, (int)i), ohy = __shfl(ahy, (int)i);
        const float ilx = __shfl(blx, (int)j), ily = __shfl(bly, (int)j);
        const float ihx = __shfl(bhx, (int)j), ihy = __shfl(bhy, (int)j);
        const bool hit = t < T && (olx <= ihx) && (ilx <= ohx) && (oly <= ihy) && (ily <= ohy);
        const uint64_t m = __ballot(hit);
        if (!FILL && slots && hit) {
            const uint32_t r = total + (uint32_t)__popcll(m & below);
            if (r < kSlotHits) slots[(uint64_t)p * kSlotStride + r] = (uint16_t)((i << 8) | j);
        }
        if (FILL && hit) {
            const uint64_t o = pos + total + (uint64_t)__popcll(m & below);
            const uint32_t ca = ptr_any(A, pr.x, i), cb = ptr_any(B, pr.y, j);
            if (o < end) {
                if (MODE == JOIN_EMIT)
                    keys[o] = ((uint64_t)ca << 32) | cb;
                else
                    next[o] = make_uint2(ca, cb);
            } else if (o < out_cap) {
                atomicOr(&ctrl->err, kErrBounds);
            }
        }
        total += (uint32_t)__popcll(m);
    }
    if (!FILL && lane == 0) {
        counts[p] = total;
        // spread over kTestSlots counters, one 128-byte line each
        if (tests_acc) atomicAdd(&tests_acc[(p % kTestSlots) * 16], (unsigned long long)T);
    }
}

template <int MODE, bool O3, int SHRINK, bool LB = false>
static hipError_t launch_cand(const TreeView &a, const TreeView &b, const uint2 *fr, uint32_t nfr,
                              const uint64_t *nfr_dev, bool fill, uint32_t *counts, const uint64_t *offsets,
                              uint2 *next, uint64_t *keys, uint64_t out_cap, uint16_t *slots, Ctrl *ctrl,
                              unsigned long long *tests_acc, hipStream_t s) {
    const uint32_t blocks = (nfr + 3) / 4;
    if (fill)
        hipLaunchKernelGGL((join_cand_kernel<MODE, true, O3, SHRINK, LB>), dim3(blocks), dim3(256), 0, s, a, b, fr, nfr,
                           nfr_dev, counts, offsets, next, keys, out_cap, slots, ctrl,
                           (unsigned long long *)nullptr);
    else
        hipLaunchKernelGGL((join_cand_kernel<MODE, false, O3, SHRINK, LB>), dim3(blocks), dim3(256), 0, s, a, b, fr,
                           nfr, nfr_dev, counts, offsets, next, keys, out_cap, slots, ctrl, tests_acc);
    return hipGetLastError();
}

template <int MODE>
static hipError_t launch_cand_flags(const TreeView &a, const TreeView &b, const uint2 *fr, uint32_t nfr,
                                    const uint64_t *nd, bool fill, uint32_t *counts, const uint64_t *offsets,
                                    uint2 *next, uint64_t *keys, uint64_t cap, uint16_t *sl, Ctrl *ctrl, int flags,
                                    unsigned long long *ta, hipStream_t s) {
    const bool o3 = flags & JOIN_O3;
    const int sh = (flags & JOIN_O5) ? 5 : ((flags & JOIN_O4) ? 4 : 0);
    if (flags & JOIN_LB) {   // only with O3 + O5 (checked by the caller)
        return launch_cand<MODE, true, 5, true>(a, b, fr, nfr, nd, fill, counts, offsets, next, keys, cap, sl, ctrl,
                                                ta, s);
    }
    if (o3) {
        if (sh == 5)
            return launch_cand<MODE, true, 5>(a, b, fr, nfr, nd, fill, counts, offsets, next, keys, cap, sl, ctrl, ta,
                                              s);
        if (sh == 4)
            return launch_cand<MODE, true, 4>(a, b, fr, nfr, nd, fill, counts, offsets, next, keys, cap, sl, ctrl, ta,
                                              s);
        return launch_cand<MODE, true, 0>(a, b, fr, nfr, nd, fill, counts, offsets, next, keys, cap, sl, ctrl, ta, s);
    }
    if (sh == 5)
        return launch_cand<MODE, false, 5>(a, b, fr, nfr, nd, fill, counts, offsets, next, keys, cap, sl, ctrl, ta, s);
    if (sh == 4)
        return launch_cand<MODE, false, 4>(a, b, fr, nfr, nd, fill, counts, offsets, next, keys, cap, sl, ctrl, ta, s);
    return launch_cand<MODE, false, 0>(a, b, fr, nfr, nd, fill, counts, offsets, next, keys, cap, sl, ctrl, ta, s);
}

template <int MODE>
static hipError_t launch_mode(const TreeView &a, const TreeView &b, const uint2 *fr, uint32_t nfr, const uint64_t *nd,
                              bool fill, uint32_t *counts, const uint64_t *offsets, uint2 *next, uint64_t *keys,
                              uint64_t cap, Ctrl *ctrl, unsigned long long *tests_acc, hipStream_t s) {
    const uint32_t blocks = (nfr + 3) / 4;
    if (fill)
        hipLaunchKernelGGL((join_level_kernel<MODE, true>), dim3(blocks), dim3(256), 0, s, a, b, fr, nfr, nd, counts,
                           offsets, next, keys, cap, ctrl, (unsigned long long *)nullptr);
    else
        hipLaunchKernelGGL((join_level_kernel<MODE, false>), dim3(blocks), dim3(256), 0, s, a, b, fr, nfr, nd,
                           counts, offsets, next, keys, cap, ctrl, tests_acc);
    return hipGetLastError();
}

hipError_t launch_join_level(const TreeView &a, const TreeView &b, const uint2 *frontier, uint32_t nfr,
                             const uint64_t *nd, int mode, bool fill, uint32_t *counts, const uint64_t *offsets,
                             uint2 *next, uint64_t *keys, uint64_t cap, uint16_t *slots, Ctrl *ctrl, int flags,
                             unsigned long long *tests_acc, hipStream_t s) {
    if (nfr == 0) return hipSuccess;
    if (!(flags & JOIN_TILE) && (mode == JOIN_BOTH || mode == JOIN_EMIT)) {
        if (mode == JOIN_BOTH)
            return launch_cand_flags<JOIN_BOTH>(a, b, frontier, nfr, nd, fill, counts, offsets, next, keys, cap,
                                                slots, ctrl, flags, tests_acc, s);
        return launch_cand_flags<JOIN_EMIT>(a, b, frontier, nfr, nd, fill, counts, offsets, next, keys, cap, slots,
                                            ctrl, flags, tests_acc, s);
    }
    switch (mode) {
    case JOIN_BOTH:
        return launch_mode<JOIN_BOTH>(a, b, frontier, nfr, nd, fill, counts, offsets, next, keys, cap, ctrl, tests_acc,
                                      s);
    case JOIN_EMIT:
        return launch_mode<JOIN_EMIT>(a, b, frontier, nfr, nd, fill, counts, offsets, next, keys, cap, ctrl, tests_acc,
                                      s);
    case JOIN_DESC_A:
        return launch_mode<JOIN_DESC_A>(a, b, frontier, nfr, nd, fill, counts, offsets, next, keys, cap, ctrl,
                                        tests_acc, s);
    default:
        return launch_mode<JOIN_DESC_B>(a, b, frontier, nfr, nd, fill, counts, offsets, next, keys, cap, ctrl,
                                        tests_acc, s);
    }
}

uint64_t join_slot_bytes(uint64_t nfr) { return nfr * kSlotStride * sizeof(uint16_t); }

__global__ void keys_to_pairs_kernel(const uint64_t *__restrict__ keys, uint64_t n, uint32_t *__restrict__ pairs) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t k = keys[i];
        pairs[2 * i] = (uint32_t)(k >> 32);
        pairs[2 * i + 1] = (uint32_t)k;
    }
}

__global__ void copy_err_kernel(const Ctrl *__restrict__ ctrl, uint32_t *__restrict__ dst) { *dst = ctrl->err; }

hipError_t launch_copy_err(const Ctrl *ctrl, uint32_t *dst, hipStream_t s) {
    hipLaunchKernelGGL(copy_err_kernel, dim3(1), dim3(1), 0, s, ctrl, dst);
    return hipGetLastError();
}

hipError_t launch_keys_to_pairs(const uint64_t *keys, uint64_t n, uint32_t *pairs, hipStream_t s) {
    if (n == 0) return hipSuccess;
    uint64_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(keys_to_pairs_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, keys, n, pairs);
    return hipGetLastError();
}

// ---- pair keys: bucket sort by the top digit --------------------------------
// Keys per block in the scatter, 4 per thread: both passes wait on memory, and
// a result of a million keys has no more tiles than the chip has CUs (with 256
// threads and 16 keys each they took 10 and 23 us, now 7 and 16).
constexpr uint32_t kPairTile = 4096, kPairThreads = 1024;

__global__ void __launch_bounds__(kPairThreads)
pair_bucket_hist(const uint64_t *__restrict__ keys, uint64_t n, const uint64_t *__restrict__ n_dev, int shift,
                 uint32_t *__restrict__ cnt) {
    __shared__ uint32_t h[kPairBuckets];
    if (n_dev) n = min(n, *n_dev);
    for (uint32_t i = threadIdx.x; i < kPairBuckets; i += blockDim.x) h[i] = 0;
    __syncthreads();
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        atomicAdd(&h[(uint32_t)(keys[i] >> shift)], 1u);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < kPairBuckets; i += blockDim.x)
        if (h[i]) atomicAdd(&cnt[i], h[i]);
}

// One block of 1024: exclusive scan of the counts into start[0 .. kPairBuckets]
// (start[kPairBuckets] = n) and zeroed cursors.
__global__ void __launch_bounds__(1024)
pair_bucket_scan(const uint32_t *__restrict__ cnt, uint32_t *__restrict__ start, uint32_t *__restrict__ cursor) {
    constexpr uint32_t W = 1024 / 64;
    __shared__ uint32_t wsum[W];
    const uint32_t t = threadIdx.x, lane = t & 63u, w = t >> 6;
    const uint32_t a = cnt[2 * t], b = cnt[2 * t + 1];
    uint32_t inc = a + b;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t x = __shfl_up(inc, d);
        if ((int)lane >= d) inc += x;
    }
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t base = 0;
    for (uint32_t i = 0; i < w; ++i) base += wsum[i];
    const uint32_t ex = base + inc - (a + b);
    start[2 * t] = ex;
    start[2 * t + 1] = ex + a;
    if (t == 1023) start[kPairBuckets] = ex + a + b;
    cursor[2 * t] = 0;
    cursor[2 * t + 1] = 0;
}

// A block takes a tile of keys: LDS ranks per bucket, one global reservation
// per bucket present in the tile, then every key goes to its bucket.  The
// order inside a bucket is arbitrary (the bucket is sorted next).
__global__ void __launch_bounds__(kPairThreads)
pair_bucket_scatter(const uint64_t *__restrict__ keys, uint64_t n, const uint64_t *__restrict__ n_dev, int shift,
                    const uint32_t *__restrict__ start, uint32_t *__restrict__ cursor, uint64_t *__restrict__ out) {
    constexpr uint32_t R = kPairTile / kPairThreads;
    __shared__ uint32_t c[kPairBuckets];
    if (n_dev) n = min(n, *n_dev);
    for (uint64_t t0 = (uint64_t)blockIdx.x * kPairTile; t0 < n; t0 += (uint64_t)gridDim.x * kPairTile) {
        for (uint32_t i = threadIdx.x; i < kPairBuckets; i += kPairThreads) c[i] = 0;
        __syncthreads();
        uint64_t k[R];
        uint32_t rk[R];
#pragma unroll
        for (uint32_t r = 0; r < R; ++r) {
            const uint64_t i = t0 + r * kPairThreads + threadIdx.x;
            k[r] = i < n ? keys[i] : 0ull;
            rk[r] = i < n ? atomicAdd(&c[(uint32_t)(k[r] >> shift)], 1u) : 0u;
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < kPairBuckets; i += kPairThreads)
            if (c[i]) c[i] = start[i] + atomicAdd(&cursor[i], c[i]);
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < R; ++r) {
            const uint64_t i = t0 + r * kPairThreads + threadIdx.x;
            if (i < n) out[c[(uint32_t)(k[r] >> shift)] + rk[r]] = k[r];
        }
        __syncthreads();
    }
}

// Bitonic sort of P (a power of two) keys in LDS by the block.
__device__ __forceinline__ void lds_bitonic_u64(uint64_t *buf, uint32_t P) {
    for (uint32_t k = 2; k <= P; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            for (uint32_t t = threadIdx.x; t < P / 2; t += blockDim.x) {
                const uint32_t i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
                const uint32_t l = i | j;
                const uint64_t x = buf[i], y = buf[l];
                const bool up = (i & k) == 0;
                if ((x > y) == up) {
                    buf[i] = y;
                    buf[l] = x;
                }
            }
            __syncthreads();
        }
    }
}

// Number of keys in v[0 .. n) below x (v sorted).
__device__ __forceinline__ uint32_t count_below(const uint64_t *v, uint32_t n, uint64_t x) {
    uint32_t lo = 0, hi = n;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (v[mid] < x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// One block per bucket: a counting sort in LDS on the next kPairSub bits of
// the keys, then every key counts the smaller ones of its sub-bucket (about
// one key each) and is written at its place.  Keys that crowd a sub-bucket
// (ids far from uniform) are sorted by a bitonic network instead, over the
// bucket padded to a power of two (keys are distinct; padding with all ones
// sorts last); for every bucket that network took 45 us where the counting
// takes 14 to 30 us (780K keys).  A bucket over the LDS cap is sorted that way in
// runs of the cap, which are then merged pairwise through tmp (the partition's
// input, free by now) at the bucket's own positions: every key finds its
// place as its index in its run plus the number of keys below it in the other
// run.  With `pairs` the results are (a, b) words there (which may be tmp:
// a block only touches its bucket's places), written if the count *n_dev fits
// `capacity` and bit 0 of *skip is clear, and *err_out receives the error
// word; else sorted keys, in place.
constexpr int kPairSub = 9;
typedef uint32_t Words __attribute__((ext_vector_type(2), aligned(4)));   // the caller's pairs: any word

__global__ void __launch_bounds__(256)
pair_bucket_sort(uint64_t *__restrict__ keys, uint64_t *tmp, const uint32_t *__restrict__ start, int shift,
                 PairsOut po) {
    constexpr uint32_t NS = 1u << kPairSub;
    __shared__ uint64_t buf[kPairBucketCap];
    __shared__ uint32_t sub[NS + 1], wsum[4], wmax[4];
    if (po.err_out && blockIdx.x == 0 && threadIdx.x == 0) *po.err_out = po.ctrl->err;
    if (po.pairs && (*po.n_dev > po.capacity || (*po.skip & 1u))) return;
    const uint32_t bk = blockIdx.x, t = threadIdx.x, lane = t & 63u, w = t >> 6;
    const uint32_t s0 = start[bk], c = start[bk + 1] - s0;
    if (c == 0 || (c == 1 && !po.pairs)) return;
    auto put = [&](uint32_t i, uint64_t x) {
        if (po.pairs)
            reinterpret_cast<Words *>(po.pairs)[s0 + i] = Words{(uint32_t)(x >> 32), (uint32_t)x};
        else
            keys[s0 + i] = x;
    };
    if (c <= kPairBucketCap) {
        const int sh = shift > kPairSub ? shift - kPairSub : 0;
        auto digit = [&](uint64_t x) { return (uint32_t)(x >> sh) & (NS - 1u); };
        for (uint32_t i = t; i < NS; i += 256) sub[i] = 0;
        __syncthreads();
        for (uint32_t i = t; i < c; i += 256) atomicAdd(&sub[digit(keys[s0 + i])], 1u);
        __syncthreads();
        const uint32_t x0 = sub[2 * t], x1 = sub[2 * t + 1];
        uint32_t inc = x0 + x1, mx = max(x0, x1);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(inc, d);
            if ((int)lane >= d) inc += y;
            mx = max(mx, (uint32_t)__shfl_xor((int)mx, d));
        }
        if (lane == 63) {
            wsum[w] = inc;
            wmax[w] = mx;
        }
        __syncthreads();
        uint32_t ex = inc - x0 - x1;
        for (uint32_t i = 0; i < w; ++i) ex += wsum[i];
        mx = max(max(wmax[0], wmax[1]), max(wmax[2], wmax[3]));
        sub[2 * t] = ex;
        sub[2 * t + 1] = ex + x0;
        __syncthreads();
        for (uint32_t i = t; i < c; i += 256) {
            const uint64_t x = keys[s0 + i];
            buf[atomicAdd(&sub[digit(x)], 1u)] = x;   // sub: now the ends
        }
        __syncthreads();
        if (mx <= 32) {
            for (uint32_t i = t; i < c; i += 256) {
                const uint64_t x = buf[i];
                const uint32_t d = digit(x), b = d ? sub[d - 1] : 0u, e = sub[d];
                uint32_t r = b;
                for (uint32_t k = b; k < e; ++k) r += buf[k] < x ? 1u : 0u;
                put(r, x);
            }
            return;
        }
        uint32_t P = 2;
        while (P < c) P <<= 1;
        for (uint32_t i = c + t; i < P; i += 256) buf[i] = ~0ull;
        __syncthreads();
        lds_bitonic_u64(buf, P);
        for (uint32_t i = t; i < c; i += 256) put(i, buf[i]);
        return;
    }
    for (uint32_t r0 = 0; r0 < c; r0 += kPairBucketCap) {
        const uint32_t rc = min(c - r0, kPairBucketCap);
        uint32_t P = 2;
        while (P < rc) P <<= 1;
        for (uint32_t i = t; i < P; i += 256) buf[i] = i < rc ? keys[s0 + r0 + i] : ~0ull;
        __syncthreads();
        lds_bitonic_u64(buf, P);
        for (uint32_t i = t; i < rc; i += 256) keys[s0 + r0 + i] = buf[i];
        __syncthreads();
    }
    uint64_t *src = keys + s0, *dst = tmp + s0;
    for (uint32_t wd = kPairBucketCap; wd < c; wd *= 2) {
        for (uint32_t i = t; i < c; i += 256) {
            const uint32_t a0 = i / (2 * wd) * (2 * wd);
            const uint32_t b0 = min(a0 + wd, c), b1 = min(a0 + 2 * wd, c);
            const uint64_t x = src[i];
            const uint32_t pos = i < b0 ? i + count_below(src + b0, b1 - b0, x)
                                        : (i - b0) + a0 + count_below(src + a0, b0 - a0, x);
            dst[pos] = x;
        }
        __syncthreads();
        uint64_t *t2 = src;
        src = dst;
        dst = t2;
    }
    if (po.pairs || src != keys + s0) {
        for (uint32_t i = t; i < c; i += 256) put(i, src[i]);
    }
}

hipError_t launch_pair_bucket_sort(uint64_t *keys, uint64_t n, int shift, uint64_t *out, uint32_t *ws,
                                   hipStream_t s, const PairsOut *po) {
    if (n == 0) return hipSuccess;
    uint32_t *cnt = ws, *start = ws + kPairBuckets, *cursor = ws + 2 * kPairBuckets + 4;
    const uint64_t *n_dev = po ? po->n_dev : nullptr;
    if (!po) {
        hipError_t e = launch_zero(cnt, 4 * kPairBuckets, s);
        if (e != hipSuccess) return e;
    }
    const uint64_t tiles = (n + kPairTile - 1) / kPairTile;
    const uint32_t cus = (uint32_t)num_cus();
    const uint32_t hb = (uint32_t)(tiles < (uint64_t)cus * 4 ? tiles : (uint64_t)cus * 4);
    hipLaunchKernelGGL(pair_bucket_hist, dim3(hb), dim3(kPairThreads), 0, s, keys, n, n_dev, shift, cnt);
    hipLaunchKernelGGL(pair_bucket_scan, dim3(1), dim3(1024), 0, s, cnt, start, cursor);
    const uint32_t sb = (uint32_t)(tiles < (uint64_t)cus * 8 ? tiles : (uint64_t)cus * 8);
    hipLaunchKernelGGL(pair_bucket_scatter, dim3(sb), dim3(kPairThreads), 0, s, keys, n, n_dev, shift, start, cursor, out);
    hipLaunchKernelGGL(pair_bucket_sort, dim3(kPairBuckets), dim3(256), 0, s, out, keys, start, shift,
                       po ? *po : PairsOut{});
    return hipGetLastError();
}

}  // namespace rtk
