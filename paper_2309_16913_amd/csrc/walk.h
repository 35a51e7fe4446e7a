// Group traversal of the count passes: several nodes of a lane group's stack
// visited per round.
//
// A walk that pops one node at a time waits one full memory latency per node
// (its next node is known only after the compare), so a window that reaches a
// few hundred nodes takes a few hundred latencies however idle the chip is.
// Here a round takes up to kWalkBatch leaves, or up to kWalkInner internal
// nodes while the stack leaves room (see walk_stack_bound), from the top of
// the stack and issues all their loads before the first compare.  What bounds
// the pass is vector instructions where many windows run (the loads take one
// scalar base and a 32-bit offset for that reason) and the chain of rounds
// where few do.  Recording count pass, one node per pop -> this walk: 1M
// windows on 10M rectangles (fanout 64) 2.72 -> 1.9 ms, 50k windows on 1.2M
// (fanout 32) 0.295 -> 0.17, 50k large windows on 50M with the split mapping
// (shared subtrees) 4.3 -> 1.7, 100 of those 0.30 -> 0.08.
#pragma once

#include "rt_internal.h"

namespace rtk {

template <int LAYOUT>
__device__ __forceinline__ void load_entry(const uint8_t *__restrict__ node, uint32_t F, uint32_t e,
                                           float &lx, float &ly, float &hx, float &hy) {
    if constexpr (LAYOUT == LAYOUT_SOA) {
        const float *f = reinterpret_cast<const float *>(node);
        lx = f[e];
        ly = f[F + e];
        hx = f[2 * F + e];
        hy = f[3 * F + e];
    } else if constexpr (LAYOUT == LAYOUT_AOS) {
        const float *f = reinterpret_cast<const float *>(node) + 5 * e;
        lx = f[0];
        ly = f[1];
        hx = f[2];
        hy = f[3];
    } else {
        const float2 *lo = reinterpret_cast<const float2 *>(node);
        const float2 a = lo[e];
        const float2 b = lo[F + e];
        lx = a.x;
        ly = a.y;
        hx = b.x;
        hy = b.y;
    }
}

template <int LAYOUT>
__device__ __forceinline__ uint32_t load_ptr(const uint8_t *__restrict__ node, uint32_t F, uint32_t e) {
    const uint32_t *u = reinterpret_cast<const uint32_t *>(node);
    if constexpr (LAYOUT == LAYOUT_AOS) return u[5 * e + 4];
    return u[4 * F + e];
}

// Byte offset of a node in the tree: 32 bits when the tree's nodes are below
// 4 GiB (WIDE = false), so that a load takes its address as one scalar base and
// one 32-bit register.
template <bool WIDE> struct NodeOffset { typedef uint32_t type; };
template <> struct NodeOffset<true> { typedef uint64_t type; };

// Entry e of the node at byte offset o.
template <int LAYOUT, class Off>
__device__ __forceinline__ void load_entry_at(const uint8_t *__restrict__ nodes, Off o, uint32_t F, uint32_t e,
                                              float &lx, float &ly, float &hx, float &hy) {
    if constexpr (LAYOUT == LAYOUT_SOA) {
        const Off b = o + 4u * e;
        const uint32_t c = 4u * F;
        lx = *reinterpret_cast<const float *>(nodes + b);
        ly = *reinterpret_cast<const float *>(nodes + (Off)(b + c));
        hx = *reinterpret_cast<const float *>(nodes + (Off)(b + 2u * c));
        hy = *reinterpret_cast<const float *>(nodes + (Off)(b + 3u * c));
    } else if constexpr (LAYOUT == LAYOUT_AOS) {
        const float *f = reinterpret_cast<const float *>(nodes + (Off)(o + 20u * e));
        lx = f[0];
        ly = f[1];
        hx = f[2];
        hy = f[3];
    } else {
        const Off b = o + 8u * e;
        const float2 x = *reinterpret_cast<const float2 *>(nodes + b);
        const float2 y = *reinterpret_cast<const float2 *>(nodes + (Off)(b + 8u * F));
        lx = x.x;
        ly = x.y;
        hx = y.x;
        hy = y.y;
    }
}

// Work of a persistent grid in kXcds lists (block b works on XCD b % kXcds,
// whose list it drains first, so that neighbouring units share that XCD's L2).
// The lists' counters are single addresses whose updates are serialized (about
// 17 ns each: with one update per unit, and eight more per group to find every
// list drained, they took 270 us of a pass over 50k windows).  So a group's
// first unit is fixed by its place in the grid; later ones come `chunk` at a
// time, the block's groups sharing what one of them took through an LDS word;
// and the block remembers which lists it found drained.  A grid whose units
// all are first units touches no counter.
struct ListShare {                 // one per block, in LDS
    unsigned long long span;       // units taken for the block: next << 32 | end
    uint32_t tried;                // lists home .. home + tried - 1 are drained
    __device__ __forceinline__ void init() {
        if (threadIdx.x == 0) {
            span = 0;
            tried = 0;
        }
        __syncthreads();
    }
};

struct ListGrab {
    uint32_t home, first, fixed;   // fixed: units of every list handed out by place
    bool started = false;

    // groups: lane groups per block, g: this group's index in its block; the
    // grid is a multiple of kXcds blocks
    __device__ __forceinline__ ListGrab(uint32_t groups, uint32_t g) {
        home = blockIdx.x % kXcds;
        first = (blockIdx.x / kXcds) * groups + g;
        fixed = (gridDim.x / kXcds) * groups;
    }

    // For a group's leader: the next units [*p0, *p0 + result), 0 at the end.
    // begin(x), len(x): the units of list x.
    template <class Begin, class Len>
    __device__ __forceinline__ uint32_t take(ListShare *sh, uint32_t (*taken)[32], uint32_t chunk, Begin begin,
                                             Len len, uint32_t *p0) {
        if (!started) {
            started = true;
            if (first < len(home)) {
                *p0 = begin(home) + first;
                return 1;
            }
        }
        if (chunk > 1) {
            const unsigned long long s = atomicAdd(&sh->span, 1ull << 32);
            if ((uint32_t)(s >> 32) < (uint32_t)s) {
                *p0 = (uint32_t)(s >> 32);
                return 1;
            }
        }
        uint32_t v = *(volatile uint32_t *)&sh->tried;
        for (; v < kXcds; ++v) {
            const uint32_t x = (home + v) % kXcds;
            const uint32_t n = len(x);
            if (n <= fixed) continue;
            const uint32_t k = atomicAdd(&taken[x][0], chunk);
            if (k >= n - fixed) continue;
            atomicMax(&sh->tried, v);
            const uint32_t p = begin(x) + fixed + k, c = min(chunk, n - fixed - k);
            *p0 = p;
            if (c > 1) {
                // share all but the first, unless another group's units are
                // still there (then they stay with this group)
                unsigned long long cur = *(volatile unsigned long long *)&sh->span;
                for (int i = 0; i < 4 && (uint32_t)(cur >> 32) >= (uint32_t)cur; ++i) {
                    const unsigned long long old = atomicCAS(&sh->span, cur, (unsigned long long)(p + 1) << 32 | (p + c));
                    if (old == cur) return 1;
                    cur = old;
                }
            }
            return c;
        }
        atomicMax(&sh->tried, v);
        return 0;
    }
};

// Where the record-keeping count passes write (rec NULL: no records).
struct RecArena {
    uint4 *rec;
    uint32_t *count;    // records per chunk
    uint32_t nchunks;
    uint32_t nfixed;    // chunks [0, nfixed) belong to groups by their place (ctrl->rec_chunks starts there)
};

// The state of one lane group (G lanes, lane e in the group, wave lane gbase
// + e).  SHARED: several units of one query run in different groups, so the
// query's counter is advanced with atomics and a record's position is known
// only then (settle); otherwise the group owns the query's counter.
template <int G, int LAYOUT, bool REC, bool SHARED, bool WIDE>
struct GroupWalk {
    typedef typename NodeOffset<WIDE>::type Off;
    static constexpr uint32_t U = kWalkBatch;
    uint32_t e, gbase;
    uint64_t below;
    uint32_t *stk;
    uint32_t stack_cap;
    uint32_t sp = 0;
    uint32_t pos = 0;         // ids counted for the unit (SHARED: since the last settle)
    // records collect in LDS and go out to the group's chunk of the arena up
    // to kRecBuf at a time: loads and stores share one in-order completion
    // counter, so a store issued before a node load delays the wait for it
    // (SHARED: to places reserved at the arena's end, a chunk's worth at a time
    // if the buffer fills up, and exactly as many as there are at the end.  Such
    // a launch has a group for every few items, and most groups write a handful
    // of records: with a chunk each, 1000 windows of up to 1e-2 of the space on
    // 10M rectangles took 8.7K chunks for 0.04M records, more than twice the
    // arena.  An update per 64 records instead of 256 is no way out: 0.40 ->
    // 1.66 ms for the large subtrees of 50k windows on 50M rectangles.)
    uint4 *rbuf;
    uint32_t nbuf = 0, rchunk = kNoNode, rcnt = 0, ustart = 0;
    uint32_t room = 0, limit = 0;   // SHARED: places reserved from rchunk on, and those there are
    uint32_t own = kNoNode;   // the chunk that is the group's by its place, until it is used
    RecArena ar;
    Ctrl *ctrl;

    __device__ __forceinline__ GroupWalk(uint32_t lane, uint32_t *stack, uint32_t cap, uint4 *records,
                                         const RecArena &arena, Ctrl *c)
        : e(lane & (G - 1)), gbase(lane & ~(uint32_t)(G - 1)), stk(stack), stack_cap(cap), rbuf(records), ar(arena),
          ctrl(c) {
        // the launches of items take no chunks: how many are taken is settled
        if (REC && SHARED) limit = tail_limit(c->rec_chunks, arena.nchunks);
        below = e == 0 ? 0ull : (~0ull >> (64 - e));
    }

    // SHARED: reserve the unit's pos ids in the query's counter and give its
    // buffered records their positions.
    __device__ __forceinline__ void settle(uint32_t *counts, uint32_t slot) {
        if constexpr (SHARED) {
            if (pos) {
                uint32_t b = 0;
                if (e == 0) b = atomicAdd(&counts[slot], pos);
                b = (uint32_t)__shfl((int)b, (int)gbase);
                __builtin_amdgcn_wave_barrier();
                for (uint32_t i = ustart + e; i < nbuf; i += G) rbuf[i].y += b;
                __builtin_amdgcn_wave_barrier();
                pos = 0;
            }
            ustart = nbuf;
        }
    }

    // SHARED: place of record i of the group's reservation.
    __device__ __forceinline__ uint4 *tail_place(uint32_t i) {
        return ar.rec + ((size_t)ar.nchunks * kRecChunk - 1 - rchunk - i);
    }

    // SHARED: room for the buffered records; what is left of the room before is
    // filled with records of nothing.
    __device__ __forceinline__ void reserve(bool last) {   // group-uniform
        if (rchunk == kRecDead || rcnt + nbuf <= room) return;
        for (uint32_t i = rcnt + e; i < room; i += G) put_rec(tail_place(i), 0u, 0u, 0u, 0u);
        const uint32_t n = last ? nbuf : kRecChunk;
        uint32_t at = 0;
        if (e == 0) {
            at = atomicAdd(&ctrl->rec_tail, n);
            if (at + n > limit) {
                atomicOr(&ctrl->rec_overflow, 1u);
                at = kRecDead;
            }
        }
        rchunk = (uint32_t)__shfl((int)at, (int)gbase);
        rcnt = 0;
        room = n;
    }

    __device__ __forceinline__ void flush(uint32_t *counts, uint32_t slot, bool last = false) {   // group-uniform
        if constexpr (REC && SHARED) {
            if (nbuf == 0) return;
            settle(counts, slot);
            reserve(last);
            __builtin_amdgcn_wave_barrier();
            if (rchunk != kRecDead) {
                for (uint32_t i = e; i < nbuf; i += G) {
                    const uint4 v = rbuf[i];
                    put_rec(tail_place(rcnt + i), v.x, v.y, v.z, v.w);
                }
                rcnt += nbuf;
            }
            nbuf = ustart = 0;
            __builtin_amdgcn_wave_barrier();
        } else if constexpr (REC) {
            if (nbuf == 0) return;
            __builtin_amdgcn_wave_barrier();
            if (rchunk != kRecDead && (rchunk == kNoNode || rcnt + nbuf > kRecChunk)) {
                if (rchunk != kNoNode && e == 0) ar.count[rchunk] = rcnt;
                uint32_t c = own;
                if (own == kNoNode) {   // group-uniform
                    if (e == 0) c = atomicAdd(&ctrl->rec_chunks, 1u);
                    c = (uint32_t)__shfl((int)c, (int)gbase);
                }
                own = kNoNode;
                if (c < ar.nchunks) {
                    rchunk = c;
                    rcnt = 0;
                } else {
                    if (e == 0) atomicOr(&ctrl->rec_overflow, 1u);
                    rchunk = kRecDead;
                }
            }
            if (rchunk < kRecDead) {
                for (uint32_t i = e; i < nbuf; i += G) {
                    const uint4 v = rbuf[i];
                    put_rec(ar.rec + (size_t)rchunk * kRecChunk + rcnt + i, v.x, v.y, v.z, v.w);
                }
                rcnt += nbuf;
            }
            nbuf = ustart = 0;
            __builtin_amdgcn_wave_barrier();
        }
    }

    __device__ __forceinline__ void finish(uint32_t *counts) {   // after the group's last unit
        if constexpr (REC && SHARED) {
            flush(counts, 0, true);
            if (rchunk != kRecDead)
                for (uint32_t i = rcnt + e; i < room; i += G) put_rec(tail_place(i), 0u, 0u, 0u, 0u);
        } else if constexpr (REC) {
            flush(counts, 0);
            if (e == 0 && rchunk < kRecDead) ar.count[rchunk] = rcnt;
            if (e == 0 && own != kNoNode) ar.count[own] = 0;
        }
    }

    // A value that is the same in all lanes of the group; for a whole wave the
    // compiler is told so (scalar registers, scalar branches).
    static __device__ __forceinline__ uint32_t uni(uint32_t v) {
        return G == 64 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)v) : v;
    }

    // One of N internal nodes that a round visits together.
    struct Children {
        uint64_t cm, pm;   // contained children, children to descend into
        uint32_t first, lo, hi;   // first child; lanes where a run of contained children begins: its leaf range
    };

    // Neighbouring contained children hold one run of leaves: their first one
    // stands for all of them.
    static __device__ __forceinline__ uint64_t run_starts(uint64_t cm) { return cm & ~(cm << 1); }

    __device__ __forceinline__ void push_children(const TreeView &t, uint32_t *counts, uint32_t slot, const Children &c) {
        if (c.cm) {   // group-uniform: contained subtrees
            const uint64_t starts = run_starts(c.cm);
            const bool mine = (starts >> e) & 1u;
            uint32_t sc = mine ? subtree_objects(t, make_uint2(c.lo, c.hi)) : 0u;
            if constexpr (REC) {
                // one record per run: its leaf range, at the position after
                // the runs before it
                uint32_t inc = sc;
                for (uint32_t d = 1; d < G; d <<= 1) {
                    const uint32_t x = (uint32_t)__shfl_up((int)inc, d, G);
                    if (e >= d) inc += x;
                }
                const uint32_t n = (uint32_t)__popcll(starts);
                if (nbuf + n > kRecBuf) flush(counts, slot);
                if (mine)
                    rbuf[nbuf + (uint32_t)__popcll(starts & below)] =
                        make_uint4(slot, pos + inc - sc, kRecRun | c.lo, c.hi);
                nbuf += n;
                pos += uni((uint32_t)__shfl((int)inc, (int)(gbase + G - 1)));
            } else {
                for (uint32_t d = 1; d < G; d <<= 1) sc += (uint32_t)__shfl_xor((int)sc, (int)d);
                pos += uni(sc);
            }
        }
        if ((c.pm >> e) & 1u) {
            const uint32_t at = sp + (uint32_t)__popcll(c.pm & below);
            if (at < stack_cap)
                stk[at] = c.first + e;   // children of a node are contiguous
            else
                atomicOr(&ctrl->err, kErrStack);
        }
        sp = min(sp + (uint32_t)__popcll(c.pm), stack_cap);
    }

    // Visits the k <= N internal nodes nd (those past k repeat the first one
    // and are dropped).  The leaf ranges of all contained children are loaded
    // at once: a round waits twice for memory, however many nodes it visits.
    template <uint32_t N>
    __device__ __forceinline__ void descend(const TreeView &t, const float4 q, uint32_t *counts, uint32_t slot,
                                            const uint32_t *nd, uint32_t k, uint64_t fmask, uint32_t en) {
        const uint32_t F = t.fanout;
        float lx[N], ly[N], hx[N], hy[N];
        Children c[N];
#pragma unroll
        for (uint32_t u = 0; u < N; ++u) {
            const Off o = (Off)nd[u] * t.node_bytes;
            c[u].first = *reinterpret_cast<const uint32_t *>(t.nodes + (Off)(o + 16u * (LAYOUT == LAYOUT_AOS ? 1u : F)));
            load_entry_at<LAYOUT, Off>(t.nodes, o, F, en, lx[u], ly[u], hx[u], hy[u]);
        }
        uint64_t any = 0;
#pragma unroll
        for (uint32_t u = 0; u < N; ++u) {
            const bool hit = (lx[u] <= q.z) && (q.x <= hx[u]) && (ly[u] <= q.w) && (q.y <= hy[u]);
            // an entry whose MBR lies inside the window: every object below it
            // qualifies, so its subtree is taken whole
            const bool cont = hit && (q.x <= lx[u]) && (hx[u] <= q.z) && (q.y <= ly[u]) && (hy[u] <= q.w);
            const uint64_t m = u < k ? (__ballot(hit) >> gbase) & fmask : 0ull;
            c[u].cm = u < k ? (__ballot(cont) >> gbase) & fmask : 0ull;
            c[u].pm = m & ~c[u].cm;
            c[u].first = uni(c[u].first);
            any |= c[u].cm;
        }
        if (any) {
#pragma unroll
            for (uint32_t u = 0; u < N; ++u) {
                const bool mine = (run_starts(c[u].cm) >> e) & 1u;
                const uint64_t after = ~(c[u].cm >> e);   // 0 if all 64 are contained
                const uint32_t last = after ? e + (uint32_t)__builtin_ctzll(after) - 1 : 63u;   // of the run begun here
                c[u].lo = t.range[c[u].first + (mine ? e : 0u)].x;
                c[u].hi = t.range[c[u].first + (mine ? last : 0u)].y;
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < N; ++u) push_children(t, counts, slot, c[u]);
    }

    // One round on the stack of the group's unit (window q, output slot
    // `slot`); returns the nodes visited (0 with an empty stack).  The loads
    // of a round are issued without a branch between them: past the k nodes
    // taken they repeat the first one, past the node's F entries the last one,
    // and the hit masks drop both.
    __device__ __forceinline__ uint32_t round(const TreeView &t, const float4 q, uint32_t *counts, uint32_t slot) {
        if (sp == 0) return 0;   // group-uniform
        const uint32_t F = t.fanout;
        const uint64_t fmask = F == 64 ? ~0ull : ((1ull << F) - 1ull);
        const uint32_t en = min(e, F - 1);
        uint32_t nd[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) nd[u] = uni(stk[sp > u ? sp - 1 - u : 0u]);
        if (nd[0] >= t.first_leaf) {
            uint32_t k = 1;
#pragma unroll
            for (uint32_t u = 1; u < U; ++u) {
                if (k == u && u < sp && nd[u] >= t.first_leaf) k = u + 1;
                nd[u] = k > u ? nd[u] : nd[0];
            }
            sp -= k;
            float lx[U], ly[U], hx[U], hy[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                load_entry_at<LAYOUT, Off>(t.nodes, (Off)nd[u] * t.node_bytes, F, en, lx[u], ly[u], hx[u], hy[u]);
            if constexpr (REC) {
                if (nbuf + (G == 64 ? 2 * U : U) > kRecBuf) flush(counts, slot);
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const bool hit = (lx[u] <= q.z) && (q.x <= hx[u]) && (ly[u] <= q.w) && (q.y <= hy[u]);
                uint64_t m = (__ballot(hit) >> gbase) & fmask;
                if (u >= k) m = 0;
                if constexpr (REC) {   // one record per 32 entries with hits
                    const uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
                    if (lo) {
                        if (e == 0) rbuf[nbuf] = make_uint4(slot, pos, nd[u], lo);
                        nbuf += 1;
                        pos += (uint32_t)__popc(lo);
                    }
                    if (G == 64 && hi) {
                        if (e == 0) rbuf[nbuf] = make_uint4(slot, pos, nd[u] | kRecHi, hi);
                        nbuf += 1;
                        pos += (uint32_t)__popc(hi);
                    }
                } else {
                    pos += (uint32_t)__popcll(m);
                }
            }
            return k;
        }
        // internal nodes: several at a time while the stack leaves room
        const bool room = sp + kWalkInner * (F - 1) <= F + walk_extra(F);
        uint32_t k = 1;
#pragma unroll
        for (uint32_t u = 1; u < kWalkInner; ++u) {
            if (k == u && u < sp && room && nd[u] < t.first_leaf) k = u + 1;
            nd[u] = k > u ? nd[u] : nd[0];
        }
        sp -= k;
        if (k > 2)
            descend<kWalkInner>(t, q, counts, slot, nd, k, fmask, en);
        else
            descend<2>(t, q, counts, slot, nd, k, fmask, en);
        return k;
    }
};

}  // namespace rtk
