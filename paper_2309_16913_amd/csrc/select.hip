// Range-select traversal kernels for gfx950.
//
// One query is handled by a group of G lanes (G = 16, 32 or 64, the smallest
// power of two >= F), so a wave64 runs 64/G queries side by side.  Lane e of a
// group owns entry e of the node being visited.  Per visited node:
//   1. the query window sits in registers, the same in all lanes of the group
//      (the paper broadcasts the query into vector registers once per query,
//      section 3 step 1);
//   2. each lane loads its entry's MBR -- for the SoA layout D1 the group's
//      loads of lx[], ly[], hx[], hy[] are four coalesced 4F-byte reads
//      (section 3 step 2);
//   3. the four fp32 comparisons give a per-lane hit; __ballot turns the hits
//      of the wave into a 64-bit mask and the group takes its G bits (the
//      SIMD compare-to-bitmask of section 3 step 3);
//   4. at an internal node the qualifying children are pushed onto the group's
//      stack in LDS at base + rank (rank = popcount of the mask below the
//      lane), the GPU form of the masked compress-store into the queue
//      (section 3 step 4, and the recursion-free traversal O1).  Nodes are
//      numbered breadth first with the children of a node contiguous, so a
//      child index is the node's first child + the entry slot; only that one
//      pointer is read per internal node.  At a leaf the
//      group counts its hits (count pass) or writes the object ids at the
//      query's output cursor + rank (fill pass).
// The stack is depth-first (a LIFO of node ids) so its size stays bounded by
// (h-1)(F-1)+1 entries instead of a whole tree level.  The count passes of whole
// queries take several nodes from it per round (walk.h), which needs some more.
//
// Usually the count pass records what it finds and the fill writes the ids from
// the records (replay_kernel); walks by one node at a time fill what was not
// recorded, count by output slot, and make the visit statistics.
//
// Work distribution: the grids are persistent; a group that empties its stack
// takes further queries from device counters (grab_chunk; ListGrab in walk.h,
// whose first ones go by the group's place).  Both passes walk the same tree
// with the same predicate, so the fill writes exactly the count pass's number of
// ids for every query.
#include "rt_internal.h"
#include "walk.h"

namespace rtk {

// Next query for a group leader.  The processing order is cut into eight
// slices; a block on XCD `home` drains slice `home` first (the queries of a
// slice are close in space, so they share tree nodes in that XCD's L2), then
// the following slices in turn.  `visited` counts the slices found empty.
// Returns nq when everything has been handed out.
__device__ __forceinline__ uint32_t grab_query(Ctrl *ctrl, uint32_t slot, uint32_t nq, const uint32_t *order,
                                               uint32_t home, uint32_t &visited, uint32_t *slice = nullptr,
                                               bool look_first = false) {
    while (visited < kXcds) {
        const uint32_t x = (home + visited) % kXcds;
        const uint32_t b0 = (uint32_t)(((uint64_t)x * nq) / kXcds);
        const uint32_t b1 = (uint32_t)(((uint64_t)(x + 1) * nq) / kXcds);
        // look_first (grids sized independently of the work, where most
        // groups of a small batch are idle): read another XCD's counter
        // before taking from it.  A drained slice's counter only grows, so a
        // read that shows it drained is final and the atomic, which thousands
        // of idle groups would otherwise queue on, is skipped.  Otherwise the
        // read would only add a round trip per steal.
        if (look_first && visited > 0 &&
            __hip_atomic_load(&ctrl->xwork[slot][x][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= b1 - b0) {
            visited += 1;
            continue;
        }
        const uint32_t k = atomicAdd(&ctrl->xwork[slot][x][0], 1u);
        if (k < b1 - b0) {
            if (slice) *slice = x;
            return order ? order[b0 + k] : b0 + k;
        }
        visited += 1;
    }
    return nq;
}

// Work unit of a pass: a query started at the root, or -- for a query split
// into subtrees -- one (query, subtree root) item.  `oslot` is the output
// slot (count pass: index into counts; fill pass: index into offsets).
struct Unit {
    uint32_t q, node, oslot;
};

// Next split item for a group leader (split items are the long ones and go
// first), or q = nq when every list is drained.
__device__ __forceinline__ Unit next_split_item(Ctrl *ctrl, uint32_t slot, uint32_t nq, const SelectPlan &plan,
                                                uint32_t home, uint32_t &hvisited) {
    while (hvisited < kXcds) {
        const uint32_t x = (home + hvisited) % kXcds;
        const uint32_t nh = ctrl->hlist[x][0];
        if (hvisited > 0 &&
            __hip_atomic_load(&ctrl->hwork[slot][x][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= nh) {
            hvisited += 1;
            continue;
        }
        const uint32_t k = atomicAdd(&ctrl->hwork[slot][x][0], 1u);
        if (k < nh) {
            const uint4 it = plan.heavy[(uint64_t)x * plan.hcap + k];
            return Unit{it.x, it.y, it.z};
        }
        hvisited += 1;
    }
    return Unit{nq, 0u, 0u};
}

// Whole queries are handed out K at a time: one atomic on the slice counter
// takes K consecutive positions of the processing order, and the group loads
// their query indices and windows in one round (lane i holds the i-th).  The
// slice counters are single addresses that every group of an XCD updates, and
// their atomics are serialized: with one query per atomic the count pass (a
// few nodes per query) waits on them.  The fill pass keeps K = 1: its queries
// take longer, and a group holding several of them widens the XCD's front in
// the processing order, which costs L2 hits.  Returns the number taken (0:
// all handed out) and the first position in *p0.
__device__ __forceinline__ uint32_t grab_chunk(uint32_t (*work)[32], uint32_t nq, uint32_t home, uint32_t &visited,
                                               bool look_first, uint32_t K, uint32_t *p0) {
    while (visited < kXcds) {
        const uint32_t x = (home + visited) % kXcds;
        const uint32_t b0 = (uint32_t)(((uint64_t)x * nq) / kXcds);
        const uint32_t b1 = (uint32_t)(((uint64_t)(x + 1) * nq) / kXcds);
        if (look_first && visited > 0 &&
            __hip_atomic_load(&work[x][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= b1 - b0) {
            visited += 1;
            continue;
        }
        const uint32_t k = atomicAdd(&work[x][0], K);
        if (k < b1 - b0) {
            *p0 = b0 + k;
            return min(K, b1 - b0 - k);
        }
        visited += 1;
    }
    return 0;
}

__device__ __forceinline__ uint64_t shfl_u64(uint64_t v, int src) {
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, src);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(v >> 32), src);
    return ((uint64_t)hi << 32) | lo;
}

// LA = 1: lookahead (section 3, optimization O2, as a load issued one node
// ahead).  A leaf pushes nothing, so after popping a leaf the next node to be
// visited is already on top of the stack; its entries are loaded right away,
// while the leaf is compared and written out, and the next iteration uses
// them without waiting for a fresh load.  After an internal node the next
// node is one of its children, decided only by the comparison, so nothing is
// loaded ahead there.
// EXT = 1, fill pass: contained runs of at least kBulkMin ids are appended
// to the plan's descriptor list for the bulk copy instead of being copied in
// the pass.
constexpr uint32_t kCountChunk = 2;
// Contained runs of at most this many leaves are copied from the leaves' own
// ptr arrays (layouts D1, D2: a leaf's ids are 4F contiguous bytes of its
// node, and those nodes are the ones neighbouring queries read), longer ones
// from the leaf-id array -- except with 64-entry nodes, where every run is
// copied from the leaves' nodes (measured at 10M rectangles / 1M windows:
// fill 3.65 ms from the nodes, 4.22 ms through the array; with 32-entry
// nodes 5.29 vs 4.85 ms).
constexpr uint32_t kNodeCopyLeaves = 4;

template <int G, int LAYOUT, int MODE, int LA, int EXT>
__global__ void __launch_bounds__(256)
select_kernel(TreeView t, const float4 *__restrict__ qs, uint32_t nq, uint32_t *__restrict__ counts,
              const uint64_t *__restrict__ offsets, uint32_t *__restrict__ ids, uint64_t cap,
              Ctrl *__restrict__ ctrl, uint32_t slot, uint32_t stack_cap, SelectPlan plan, uint32_t noffsets) {
    extern __shared__ uint32_t smem[];
    if constexpr (MODE == SEL_FILL) {
        if (offsets[noffsets] > cap) return;   // result does not fit: leave ids untouched
        // the replay wrote everything, or the shared fill does
        const bool rec = ctrl->rec_nchunks != 0, over = ctrl->rec_overflow != 0;
        if (plan.fill_guard == FILL_UNLESS_REPLAYED && rec && !over) return;
        if (plan.fill_guard == FILL_IF_NOT_RECORDED && rec) return;
    }
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t e = lane & (G - 1);
    const uint32_t gbase = lane & ~(uint32_t)(G - 1);
    uint32_t *stk = smem + (threadIdx.x / G) * stack_cap;
    const uint32_t F = t.fanout;
    const uint64_t gmask = (G == 64) ? ~0ull : ((1ull << G) - 1ull);
    const uint64_t below = (e == 0) ? 0ull : (~0ull >> (64 - e));

    // XCD-relative cursor over the eight slices of the processing order
    const uint32_t home = blockIdx.x % kXcds;
    uint32_t visited = 0;
    uint32_t hvisited = plan.heavy ? 0u : kXcds;
    // the group's chunk of whole queries: lane i < cn holds query cq, its
    // window cw and output slot cs (kNoNode: split); ci = next to start
    // (and, fill pass, its output range [cpos, cend))
    uint32_t cn = 0, ci = 0, cq = 0, cs = 0;
    float4 cw = make_float4(0.f, 0.f, 0.f, 0.f);
    uint64_t cpos = 0, cend = 0;
    uint32_t oslot = 0;
    bool have = false, done = false;
    uint32_t sp = 0;
    float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
    uint64_t pos = 0, end = 0;
    uint64_t vnodes = 0, ventries = 0, vcont = 0;
    // lookahead registers: the node loaded ahead and this lane's entry of it
    uint32_t pf_node = kNoNode, pf_ref = 0;
    float pf_lx = 0.f, pf_ly = 0.f, pf_hx = 0.f, pf_hy = 0.f;
    while (true) {
        if (!done && sp == 0) {
            if (have) {
                if constexpr (MODE == SEL_COUNT) {
                    if (e == 0) counts[oslot] = (uint32_t)pos;
                }
            }
            Unit u{nq, 0u, 0u};
            bool from_chunk = false;
            if (hvisited < kXcds) {
                if (e == 0) u = next_split_item(ctrl, slot, nq, plan, home, hvisited);
                u.q = __shfl(u.q, (int)gbase);
                u.node = __shfl(u.node, (int)gbase);
                u.oslot = __shfl(u.oslot, (int)gbase);
                hvisited = __shfl(hvisited, (int)gbase);
                if (u.q < nq) q = qs[u.q];
            }
            // whole queries from the group's chunk, skipping split ones
            while (u.q >= nq) {
                if (ci >= cn) {
                    uint32_t p0 = 0, c = 0;
                    if (e == 0)
                        c = grab_chunk(ctrl->xwork[slot], nq, home, visited, plan.heavy != nullptr,
                                       MODE == SEL_FILL ? 1u : kCountChunk, &p0);
                    c = __shfl(c, (int)gbase);
                    p0 = __shfl(p0, (int)gbase);
                    visited = __shfl(visited, (int)gbase);
                    if (c == 0) break;
                    cn = c;
                    ci = 0;
                    if (e < c) {
                        cq = plan.order ? plan.order[p0 + e] : p0 + e;
                        cw = qs[cq];
                        cs = cq;
                        if (plan.slot_first) {
                            const uint64_t s0 = plan.slot_first[cq];
                            cs = plan.slot_first[cq + 1] - s0 == 1 ? (uint32_t)s0 : kNoNode;
                        }
                        if constexpr (MODE == SEL_FILL) {
                            if (cs != kNoNode) {
                                cpos = offsets[cs];
                                cend = offsets[cs + 1];
                            }
                        }
                    }
                }
                const int src = (int)(gbase + ci);
                ci += 1;
                const uint32_t os = __shfl(cs, src);
                if (os == kNoNode) continue;   // split: its items cover it
                u = Unit{(uint32_t)__shfl(cq, src), 0u, os};
                q = make_float4(__shfl(cw.x, src), __shfl(cw.y, src), __shfl(cw.z, src), __shfl(cw.w, src));
                if constexpr (MODE == SEL_FILL) {
                    pos = shfl_u64(cpos, src);
                    end = shfl_u64(cend, src);
                }
                from_chunk = true;
            }
            if (u.q < nq) {
                if constexpr (MODE == SEL_FILL) {
                    if (!from_chunk) {   // a split item
                        pos = offsets[u.oslot];
                        end = offsets[u.oslot + 1];
                    }
                } else {
                    pos = 0;
                }
                oslot = u.oslot;
                have = true;
                stk[0] = u.node;
                sp = 1;
            } else {
                have = false;
                done = true;
            }
        }
        if (__all(done)) break;
        __builtin_amdgcn_wave_barrier();

        uint32_t node = 0;
        if (have) {
            sp -= 1;
            node = stk[sp];
        }
        const uint8_t *nb = t.nodes + (size_t)node * t.node_bytes;
        const bool leaf = node >= t.first_leaf;
        bool hit = false, valid = false;
        uint32_t ref = 0;   // first child (internal node) or this entry's object id (leaf, fill pass)
        float lx = 0.f, ly = 0.f, hx = 0.f, hy = 0.f;
        bool got = false;
        if constexpr (LA != 0) {
            got = have && pf_node == node;
            if (got) {
                lx = pf_lx;
                ly = pf_ly;
                hx = pf_hx;
                hy = pf_hy;
                ref = pf_ref;
            }
        }
        if (have && e < F && !got) {
            // the id / first-child load does not depend on the comparison, so it
            // is in flight together with the coordinate loads
            if (!leaf)
                ref = load_ptr<LAYOUT>(nb, F, 0);
            else if constexpr (MODE == SEL_FILL)
                ref = load_ptr<LAYOUT>(nb, F, e);
            load_entry<LAYOUT>(nb, F, e, lx, ly, hx, hy);
        }
        if constexpr (LA != 0) {
            pf_node = kNoNode;
            if (have && leaf && sp > 0) {
                const uint32_t nx = stk[sp - 1];
                pf_node = nx;
                if (e < F) {
                    const uint8_t *nb2 = t.nodes + (size_t)nx * t.node_bytes;
                    pf_ref = 0;
                    if (nx < t.first_leaf)
                        pf_ref = load_ptr<LAYOUT>(nb2, F, 0);
                    else if constexpr (MODE == SEL_FILL)
                        pf_ref = load_ptr<LAYOUT>(nb2, F, e);
                    load_entry<LAYOUT>(nb2, F, e, pf_lx, pf_ly, pf_hx, pf_hy);
                }
            }
        }
        bool cont = false;
        if (have && e < F) {
            hit = (lx <= q.z) && (q.x <= hx) && (ly <= q.w) && (q.y <= hy);
            if constexpr (MODE == SEL_STATS) valid = (lx == lx);
            // an internal entry whose MBR lies inside the window: every object
            // below it qualifies, so its subtree is taken whole
            cont = hit && !leaf && (q.x <= lx) && (hx <= q.z) && (q.y <= ly) && (hy <= q.w);
        }
        const uint64_t m = (__ballot(hit) >> gbase) & gmask;
        const uint64_t cm = (__ballot(cont) >> gbase) & gmask;
        const uint64_t pm = m & ~cm;   // children to descend into
        const uint32_t n = (uint32_t)__popcll(m);
        const uint32_t rank = (uint32_t)__popcll(m & below);
        if constexpr (MODE == SEL_STATS) {
            const uint64_t vm = (__ballot(valid) >> gbase) & gmask;
            if (have) {
                vnodes += 1;
                ventries += (uint64_t)__popcll(vm);
            }
        }
        if (have) {
            if (leaf) {
                if constexpr (MODE == SEL_FILL) {
                    if (hit) {
                        const uint64_t o = pos + rank;
                        // ids are written once and read back only by the
                        // sort: stores that bypass the caches leave L2 to the
                        // tree nodes (fill pass 4.4 -> 3.8 ms at 10M/1M)
                        if (o < end)
                            put_id(ids + o, ref);
                        else
                            atomicOr(&ctrl->err, kErrBounds);
                    }
                }
                pos += n;
            } else {
                // children of a node are contiguous: entry e points at first + e
                const uint32_t first = __shfl(ref, (int)gbase);
                if (cm) {   // group-uniform: contained subtrees
                    if constexpr (MODE == SEL_FILL) {
                        // copy the ids of the contained subtrees' leaves.
                        // Consecutive contained children have consecutive
                        // leaves, so each run of them is one leaf range and
                        // one contiguous run of the tree's leaf-id array.
                        uint64_t todo = cm;
                        bool bad = false;
                        while (todo) {
                            const uint32_t j0 = (uint32_t)__builtin_ctzll(todo);
                            const uint64_t sh = todo >> j0;
                            const uint32_t len = ~sh ? (uint32_t)__builtin_ctzll(~sh) : 64u - j0;
                            todo = (j0 + len >= 64) ? 0ull : (todo & (~0ull << (j0 + len)));
                            const uint32_t l0 = t.range[first + j0].x, l1 = t.range[first + j0 + len - 1].y;
                            if constexpr (EXT != 0) {
                                if (subtree_objects(t, make_uint2(l0, l1)) >= kBulkMin) {
                                    pos += defer_leaf_run(t, l0, l1, ids, pos, end, e, G, gbase, plan.bulk,
                                                          plan.bulk_cap, ctrl, &bad);
                                    continue;
                                }
                            }
                            if (LAYOUT != LAYOUT_AOS && (G == 64 || l1 - l0 <= kNodeCopyLeaves)) {
                                // lane e copies entry e of U leaves at a time
                                const bool hasp = t.partial_leaf >= l0 && t.partial_leaf < l1;
                                constexpr uint32_t U = 4;
                                for (uint32_t lb = l0; lb < l1; lb += U) {
                                    uint32_t v[U];
                                    uint64_t o[U];
#pragma unroll
                                    for (uint32_t u = 0; u < U; ++u) {
                                        const uint32_t lf = lb + u;
                                        o[u] = ~0ull;
                                        v[u] = 0;
                                        if (lf < l1 && e < F && !(hasp && lf == t.partial_leaf && e >= t.partial_cnt)) {
                                            o[u] = pos + (uint64_t)(lf - l0) * F + e -
                                                   ((hasp && lf > t.partial_leaf) ? F - t.partial_cnt : 0u);
                                            v[u] = load_ptr<LAYOUT>(t.nodes + (size_t)lf * t.node_bytes, F, e);
                                        }
                                    }
#pragma unroll
                                    for (uint32_t u = 0; u < U; ++u) {
                                        if (o[u] != ~0ull) {
                                            if (o[u] < end)
                                                __builtin_nontemporal_store(v[u], ids + o[u]);
                                            else
                                                atomicOr(&ctrl->err, kErrBounds);
                                        }
                                    }
                                }
                                pos += subtree_objects(t, make_uint2(l0, l1));
                            } else
                                pos += copy_leaf_run<EXT != 0 ? 2 : 4>(t, l0, l1, ids, pos, end, e, G, &bad);
                        }
                        if (bad && e == 0) atomicOr(&ctrl->err, kErrBounds);
                    } else {
                        uint32_t sc = cont ? subtree_objects(t, t.range[first + e]) : 0u;
                        for (uint32_t d = 1; d < G; d <<= 1) sc += (uint32_t)__shfl_xor((int)sc, (int)d);
                        pos += sc;
                        if constexpr (MODE == SEL_STATS) vcont += sc;
                    }
                }
                const uint32_t prank = (uint32_t)__popcll(pm & below);
                if (hit && !cont) {
                    if (sp + prank < stack_cap)
                        stk[sp + prank] = first + e;
                    else
                        atomicOr(&ctrl->err, kErrStack);
                }
                sp = min(sp + (uint32_t)__popcll(pm), stack_cap);
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    if constexpr (MODE == SEL_STATS) {
        if (e == 0 && (vnodes | ventries)) {
            atomicAdd((unsigned long long *)&ctrl->stats[0], (unsigned long long)vnodes);
            atomicAdd((unsigned long long *)&ctrl->stats[1], (unsigned long long)ventries);
            atomicAdd((unsigned long long *)&ctrl->stats[2], (unsigned long long)vcont);
        }
    }
}

// ---------------------------------------------------------------------------
// count pass on the batched walk (walk.h)
// ---------------------------------------------------------------------------
// SRC 0: units are whole queries, started at the root; the group owns the
// query's counter.  With DUMP, a group whose unit has visited `budget` nodes
// hands the rest of its stack to the items of `out` (per-XCD lists), so that
// the groups of the next launch share one large window's remaining subtrees.
// SRC 1: units are such items of `in` ({query, node}), whose results are
// added to the query's counter with atomics (the order of a query's records,
// and so of its unsorted ids, does not matter: the ids are sorted later).
struct WalkItems {
    uint2 *item;         // kXcds lists of cap items
    uint32_t cap;
    uint32_t (*n)[32];   // per list: items appended (may pass cap; the rest stayed with their group)
    uint32_t (*taken)[32];
};

template <int G, int LAYOUT, bool REC, int SRC, bool DUMP, bool WIDE>
__global__ void __launch_bounds__(256)
walk_kernel(TreeView t, const float4 *__restrict__ qs, uint32_t nq, const uint32_t *__restrict__ order,
            uint32_t *__restrict__ counts, Ctrl *__restrict__ ctrl, uint32_t chunk, uint32_t stack_cap, RecArena ar,
            uint32_t budget, WalkItems in, WalkItems out) {
    extern __shared__ uint32_t smem[];
    const uint32_t lane = threadIdx.x & 63u;
    uint4 *rbuf = reinterpret_cast<uint4 *>(smem + ((256 / G) * stack_cap + 3u) / 4u * 4u) + (threadIdx.x / G) * kRecBuf;
    GroupWalk<G, LAYOUT, REC, SRC != 0, WIDE> w(lane, smem + (threadIdx.x / G) * stack_cap, stack_cap, rbuf, ar, ctrl);
    const uint32_t e = w.e, gbase = w.gbase;
    __shared__ ListShare share;
    share.init();
    ListGrab grab(256 / G, threadIdx.x / G);
    if constexpr (REC && SRC == 0) {
        // With no more units than groups only the groups with a first unit
        // have a chunk: that unit's.
        const uint32_t groups = gridDim.x * (256 / G), x = grab.home;
        const uint32_t b = (uint32_t)(((uint64_t)x * nq) / kXcds), n = (uint32_t)(((uint64_t)(x + 1) * nq) / kXcds) - b;
        const uint32_t c = nq > groups ? blockIdx.x * (256 / G) + threadIdx.x / G
                                       : (grab.first < n ? b + grab.first : kNoNode);
        if (c < ar.nfixed) w.own = c;
    }
    // the group's chunk of units: lane i < cn holds the i-th unit's query cq,
    // window cw (and root node cd); ci = next to start
    uint32_t cn = 0, ci = 0, cq = 0, cd = 0;
    float4 cw = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 q = cw;
    uint32_t slot = 0, vis = 0;
    bool have = false, done = false;
    while (true) {
        if (!done && w.sp == 0) {
            if (have) {
                if constexpr (SRC == 0) {
                    if (e == 0) counts[slot] = w.pos;
                    w.pos = 0;
                } else {
                    w.settle(counts, slot);
                }
            }
            if (ci >= cn) {
                uint32_t p0 = 0, c = 0;
                if (e == 0) {
                    if constexpr (SRC == 0) {   // list x: the x-th eighth of the processing order
                        const auto begin = [&](uint32_t x) { return (uint32_t)(((uint64_t)x * nq) / kXcds); };
                        c = grab.take(&share, ctrl->xwork[0], chunk, begin,
                                      [&](uint32_t x) { return begin(x + 1) - begin(x); }, &p0);
                    } else {
                        c = grab.take(
                            &share, in.taken, chunk, [&](uint32_t x) { return x * in.cap; },
                            [&](uint32_t x) { return min(in.n[x][0], in.cap); }, &p0);
                    }
                }
                c = (uint32_t)__shfl((int)c, (int)gbase);
                p0 = (uint32_t)__shfl((int)p0, (int)gbase);
                cn = c;
                ci = 0;
                if (e < c) {
                    if constexpr (SRC == 0) {
                        cq = order ? order[p0 + e] : p0 + e;
                    } else {
                        const uint2 it = in.item[p0 + e];
                        cq = it.x;
                        cd = it.y;
                    }
                    cw = qs[cq];
                }
            }
            if (ci < cn) {
                const int src = (int)(gbase + ci);
                ci += 1;
                slot = (uint32_t)__shfl((int)cq, src);
                q = make_float4(__shfl(cw.x, src), __shfl(cw.y, src), __shfl(cw.z, src), __shfl(cw.w, src));
                w.stk[0] = SRC == 0 ? 0u : (uint32_t)__shfl((int)cd, src);
                w.sp = 1;
                vis = 0;
                have = true;
            } else {
                have = false;
                done = true;
            }
        }
        if (__all(done)) break;
        __builtin_amdgcn_wave_barrier();
        vis += w.round(t, q, counts, slot);
        __builtin_amdgcn_wave_barrier();
        if constexpr (DUMP) {
            if (vis >= budget && w.sp) {   // group-uniform
                uint32_t b = 0;
                if (e == 0) b = atomicAdd(&out.n[grab.home][0], w.sp);
                b = (uint32_t)__shfl((int)b, (int)gbase);
                const uint32_t n = b < out.cap ? min(w.sp, out.cap - b) : 0u;
                for (uint32_t i = e; i < n; i += G)
                    out.item[grab.home * out.cap + b + i] = make_uint2(slot, w.stk[w.sp - 1 - i]);
                w.sp -= n;
                if (w.sp) budget = 0xFFFFFFFFu;   // the list is full: the group walks on
            }
        }
    }
    w.finish(counts);
}

// ---------------------------------------------------------------------------
// walking fill of shared windows
// ---------------------------------------------------------------------------
// The fill of a select with the split mapping whose records did not fit their
// arena.  A window of n ids is cut into 1 + n / kShareIds shares, at most
// max_shares: each walks the levels above the parents of leaves on its own (a
// thousandth of the window's nodes) and takes those of the parents of leaves
// whose number falls to it.  A share's ids go wherever the window's range has
// room -- `left` holds the ids still to come, the count pass's counts at first
// -- as the sort puts them in order afterwards.  Bound by the latency of one
// node and one update of `left` per step, so a share is short: with 8192 ids
// and up to 64 shares 100 windows of up to 1e-2 of the space on 10M rectangles
// (fanout 32) took 1.22 ms, with 512 ids 0.55, with 256 ids and up to 256
// shares 0.47, now 0.40; one group per window 1.16.
constexpr uint32_t kShareIds = 64;
constexpr uint32_t kMaxShares = 512;
constexpr uint32_t kShareChunk = 16;   // units taken per counter update, one per lane

template <int G, int LAYOUT>
__global__ void __launch_bounds__(256)
shared_fill_kernel(TreeView t, const float4 *__restrict__ qs, uint32_t nq, const uint32_t *__restrict__ order,
                   uint32_t *__restrict__ left, const uint64_t *__restrict__ offsets, uint32_t *__restrict__ ids,
                   uint64_t cap, Ctrl *__restrict__ ctrl, uint32_t split_parent, uint32_t parents, uint32_t max_shares,
                   uint32_t stack_cap) {
    extern __shared__ uint32_t smem[];
    if (!ctrl->rec_nchunks || !ctrl->rec_overflow || offsets[nq] > cap) return;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t e = lane & (G - 1);
    const uint32_t gbase = lane & ~(uint32_t)(G - 1);
    uint32_t *stk = smem + (threadIdx.x / G) * stack_cap;
    const uint32_t F = t.fanout;
    const uint64_t gmask = (G == 64) ? ~0ull : ((1ull << (G & 63)) - 1ull);
    const uint64_t below = (e == 0) ? 0ull : (~0ull >> (64 - e));
    const uint32_t home = blockIdx.x % kXcds;
    uint32_t visited = 0;
    // the group's units: bit i of pend: lane i's (window cq, its share cs of cn) is still to do
    uint64_t pend = 0;
    uint32_t cq = 0, cs = 0, cn = 1;
    bool have = false, done = false;
    uint32_t sp = 0, qi = 0, share = 0, shares = 1;
    float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
    bool bad = false;
    // the place of n more ids of the window (group-uniform)
    auto place = [&](uint32_t n) {
        uint32_t rest = 0;
        if (e == 0) rest = atomicSub(&left[qi], n);
        rest = (uint32_t)__shfl((int)rest, (int)gbase);
        if (rest < n) bad = true;
        return offsets[qi] + (uint64_t)(rest - n);
    };
    while (true) {
        while (!done && sp == 0) {
            if (pend == 0) {
                // units of slice x of the order, share by share: the first
                // shares of all its windows, then the second ones, ...
                uint32_t x = 0, v = 0, c = 0;
                if (e == 0) {
                    for (; visited < kXcds; ++visited) {
                        x = (home + visited) % kXcds;
                        const uint32_t m = (uint32_t)(((uint64_t)(x + 1) * nq) / kXcds) - (uint32_t)(((uint64_t)x * nq) / kXcds);
                        v = atomicAdd(&ctrl->xwork[1][x][0], kShareChunk);
                        if (v < m * max_shares) {
                            c = min(kShareChunk, m * max_shares - v);
                            break;
                        }
                    }
                }
                x = (uint32_t)__shfl((int)x, (int)gbase);
                v = (uint32_t)__shfl((int)v, (int)gbase);
                c = (uint32_t)__shfl((int)c, (int)gbase);
                if (c == 0) {
                    have = false;
                    done = true;
                    break;
                }
                bool mine = false;
                if (e < c) {
                    const uint32_t b0 = (uint32_t)(((uint64_t)x * nq) / kXcds);
                    const uint32_t m = (uint32_t)(((uint64_t)(x + 1) * nq) / kXcds) - b0;
                    const uint32_t p = b0 + (v + e) % m;
                    cs = (v + e) / m;
                    cq = order ? order[p] : p;
                    const uint64_t n = offsets[cq + 1] - offsets[cq];
                    cn = (uint32_t)min((uint64_t)max_shares, 1 + n / kShareIds);
                    mine = n && cs < cn;
                }
                pend = (__ballot(mine) >> gbase) & gmask;
                continue;
            }
            const int src = (int)(gbase + (uint32_t)__builtin_ctzll(pend));
            pend &= pend - 1;
            qi = (uint32_t)__shfl((int)cq, src);
            share = (uint32_t)__shfl((int)cs, src);
            shares = (uint32_t)__shfl((int)cn, src);
            q = qs[qi];
            stk[0] = 0u;
            sp = 1;
            have = true;
        }
        if (__all(done)) break;
        __builtin_amdgcn_wave_barrier();
        uint32_t node = 0;
        if (have) {
            sp -= 1;
            node = stk[sp];
        }
        const uint8_t *nb = t.nodes + (size_t)node * t.node_bytes;
        const bool leaf = node >= t.first_leaf;
        bool hit = false, cont = false;
        uint32_t ref = 0;
        if (have && e < F) {
            ref = load_ptr<LAYOUT>(nb, F, leaf ? e : 0u);
            float lx, ly, hx, hy;
            load_entry<LAYOUT>(nb, F, e, lx, ly, hx, hy);
            hit = (lx <= q.z) && (q.x <= hx) && (ly <= q.w) && (q.y <= hy);
            // subtrees are taken whole from the parents of leaves down, so
            // that shares split everything above
            cont = hit && !leaf && node >= split_parent && (q.x <= lx) && (hx <= q.z) && (q.y <= ly) && (hy <= q.w);
        }
        const uint32_t first = (uint32_t)__shfl((int)ref, (int)gbase);
        if (hit && node >= split_parent && node < parents && (first + e) % shares != share) hit = cont = false;
        const uint64_t m = (__ballot(hit) >> gbase) & gmask;
        const uint64_t cm = (__ballot(cont) >> gbase) & gmask;
        const uint64_t pm = m & ~cm;
        if (have && leaf) {
            if (m) {   // group-uniform
                const uint64_t o = place((uint32_t)__popcll(m)) + (uint32_t)__popcll(m & below);
                if (hit && !bad) put_id(ids + o, ref);
            }
        } else if (have) {
            if (cm) {   // group-uniform: contained subtrees
                uint32_t n = cont ? subtree_objects(t, t.range[first + e]) : 0u;
                for (uint32_t d = 1; d < G; d <<= 1) n += (uint32_t)__shfl_xor((int)n, (int)d);
                uint64_t pos = place(n);
                const uint64_t end = pos + n;
                for (uint64_t todo = cm; todo && !bad;) {
                    // a run of neighbouring children is one run of ids
                    const uint32_t j0 = (uint32_t)__builtin_ctzll(todo);
                    const uint64_t sh = todo >> j0;
                    const uint32_t len = ~sh ? (uint32_t)__builtin_ctzll(~sh) : 64u - j0;
                    todo = (j0 + len >= 64) ? 0ull : (todo & (~0ull << (j0 + len)));
                    pos += copy_leaf_run<4>(t, t.range[first + j0].x, t.range[first + j0 + len - 1].y, ids, pos, end, e, G, &bad);
                }
            }
            if ((pm >> e) & 1u) {
                const uint32_t at = sp + (uint32_t)__popcll(pm & below);
                if (at < stack_cap)
                    stk[at] = first + e;
                else
                    atomicOr(&ctrl->err, kErrStack);
            }
            sp = min(sp + (uint32_t)__popcll(pm), stack_cap);
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (bad && e == 0) atomicOr(&ctrl->err, kErrBounds);
}

// Split pre-pass.  Walks only the internal levels above the parents of leaves
// (`split_parent` is the first node of the level above them) and finds the
// parents-of-leaves nodes a query reaches.  PHASE 0 counts them: a query reaching at least
// kmin of them (while the item budget lasts) gets one output slot per such
// node, others one slot.  PHASE 1 (after a scan of the slot counts) writes
// one work item {query, node, slot} per node of every split query.  Both
// phases walk identically, so the items match the counts.
template <int G, int LAYOUT, int PHASE>
__global__ void __launch_bounds__(256)
split_kernel(TreeView t, const float4 *__restrict__ qs, uint32_t nq, uint32_t split_parent, uint32_t kmin,
             uint32_t hcap, float min_area, uint32_t *__restrict__ nslots, const uint64_t *__restrict__ slot_first,
             uint4 *__restrict__ heavy, const uint32_t *__restrict__ order, Ctrl *__restrict__ ctrl,
             uint32_t stack_cap) {
    extern __shared__ uint32_t smem[];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t e = lane & (G - 1);
    const uint32_t gbase = lane & ~(uint32_t)(G - 1);
    uint32_t *stk = smem + (threadIdx.x / G) * stack_cap;
    const uint32_t F = t.fanout;
    const uint64_t gmask = (G == 64) ? ~0ull : ((1ull << G) - 1ull);
    const uint64_t below = (e == 0) ? 0ull : (~0ull >> (64 - e));
    uint32_t qi = 0, sp = 0, k = 0, base = 0, slot0 = 0, list = 0;
    bool have = false, done = false;
    float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
    const uint32_t home = blockIdx.x % kXcds;
    uint32_t visited = 0;
    while (true) {
        if (!done && sp == 0) {
            if (have && PHASE == 0 && e == 0) {
                uint32_t ns = 1;
                if (k >= kmin) {
                    const uint32_t old = atomicAdd(&ctrl->budget_used[list][0], k);
                    if (old + k <= hcap) ns = k;
                }
                nslots[qi] = ns;
            }
            have = false;
            uint32_t nxt = 0, b = 0, sl = 0;
            if (e == 0) {
                while (true) {
                    nxt = grab_query(ctrl, 2, nq, order, home, visited, &sl);
                    if (nxt >= nq) break;
                    const float4 w = qs[nxt];
                    if constexpr (PHASE == 0) {
                        // windows too small to reach kmin subtrees keep one slot
                        if (!((w.z - w.x) * (w.w - w.y) >= min_area)) {
                            nslots[nxt] = 1;
                            continue;
                        }
                        break;
                    } else {
                        const uint32_t ns = (uint32_t)(slot_first[nxt + 1] - slot_first[nxt]);
                        if (ns <= 1) continue;
                        b = (uint32_t)(sl * hcap) + atomicAdd(&ctrl->hlist[sl][0], ns);
                        break;
                    }
                }
            }
            nxt = __shfl(nxt, (int)gbase);
            b = __shfl(b, (int)gbase);
            sl = __shfl(sl, (int)gbase);
            if (nxt < nq) {
                qi = nxt;
                list = sl;
                have = true;
                q = qs[qi];
                stk[0] = 0u;
                sp = 1;
                k = 0;
                base = b;
                if constexpr (PHASE == 1) slot0 = (uint32_t)slot_first[qi];
            } else {
                done = true;
            }
        }
        if (__all(done)) break;
        __builtin_amdgcn_wave_barrier();
        uint32_t node = 0;
        if (have) {
            sp -= 1;
            node = stk[sp];
        }
        const uint8_t *nb = t.nodes + (size_t)node * t.node_bytes;
        bool hit = false;
        uint32_t ref = 0;
        if (have && e < F) {
            ref = load_ptr<LAYOUT>(nb, F, 0);
            float lx, ly, hx, hy;
            load_entry<LAYOUT>(nb, F, e, lx, ly, hx, hy);
            hit = (lx <= q.z) && (q.x <= hx) && (ly <= q.w) && (q.y <= hy);
        }
        const uint64_t m = (__ballot(hit) >> gbase) & gmask;
        const uint32_t n = (uint32_t)__popcll(m);
        const uint32_t rank = (uint32_t)__popcll(m & below);
        if (have) {
            // group-uniform test: only nodes above the parents-of-leaves level are
            // ever pushed, so a popped node at or past split_parent (the first
            // grandparent-of-leaves node) has parents of leaves as children
            if (node >= split_parent) {
                // the children are parents of leaves: they are the split nodes
                if constexpr (PHASE == 1) {
                    if (hit) heavy[base + k + rank] = make_uint4(qi, ref + e, slot0 + k + rank, 0u);
                }
                k += n;
            } else {
                if (hit) {
                    if (sp + rank < stack_cap)
                        stk[sp + rank] = ref + e;
                    else
                        atomicOr(&ctrl->err, kErrStack);
                }
                sp = min(sp + n, stack_cap);
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Bulk copy of deferred contained runs: one block per descriptor at a time,
// descriptors by stride (they are about the same size; a counter that every
// block updates took 24 us on its own);
// stores start at a 64-byte boundary of the destination (the first ids up
// to it are written by the first lanes), so every store instruction writes
// whole granules.
__global__ void __launch_bounds__(256)
bulk_copy_kernel(const uint32_t *__restrict__ leaf_ids, BulkList replayed, BulkList walked,
                 uint32_t *__restrict__ ids, const Ctrl *__restrict__ ctrl) {
    const BulkList list = ctrl->rec_nchunks && !ctrl->rec_overflow ? replayed : walked;
    const uint4 *__restrict__ bulk = list.d;
    const uint32_t nitems = min(ctrl->bulk_n, list.cap);
    const uint32_t t = threadIdx.x;
    for (uint32_t it = blockIdx.x; it < nitems; it += gridDim.x) {
        const uint4 d = bulk[it];
        const uint32_t *__restrict__ src = leaf_ids + d.x;
        uint32_t *__restrict__ dst = ids + (((uint64_t)d.z << 32) | d.y);
        const uint32_t len = d.w;
        const uint32_t head = min((16u - (uint32_t)((reinterpret_cast<uintptr_t>(dst) >> 2) & 15u)) & 15u, len);
        // four ids per lane: stores at 16-byte boundaries, loads at any word
        typedef uint32_t vec4 __attribute__((ext_vector_type(4)));
        typedef uint32_t vec4_any __attribute__((ext_vector_type(4), aligned(4)));
        constexpr uint32_t U = 8;
        static_assert(kBulkChunk <= U * 1024, "one round per descriptor");
        const uint32_t body = (len - head) / 4, tail = head + 4 * body;   // vectors; the first id behind them
        const vec4_any *__restrict__ src4 = reinterpret_cast<const vec4_any *>(src + head);
        vec4 *__restrict__ dst4 = reinterpret_cast<vec4 *>(dst + head);
        // ids of the unaligned ends, loaded with the rest: lanes below 16 the
        // head, the next four the tail
        const uint32_t ei = t < 16 ? t : tail + (t - 16);
        const bool edge = t < 16 ? t < head : t < 20 && ei < len;
        const uint32_t ev = edge ? src[ei] : 0u;
        vec4 v[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t i = u * 256 + t;
            if (u * 256 < body) v[u] = src4[min(i, body - 1)];
        }
        asm volatile("" ::: "memory");
        if (edge) put_id(dst + ei, ev);
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t i = u * 256 + t;
            if (i < body) __builtin_nontemporal_store(v[u], dst4 + i);
        }
    }
}

// A lane's 64-bit value as a scalar, and a run of n words as a buffer whose
// bounds drop what lies past it.
template <typename P>
__device__ __forceinline__ P *scalar64(P *p, int lane) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return reinterpret_cast<P *>((uint64_t)hi << 32 | lo);
}
typedef __amdgpu_buffer_rsrc_t RunBuf;
constexpr int kStoreNt = 2;   // non-temporal
constexpr uint32_t kRunMax = 1u << 28;   // ids in one buffer at most: its size in bytes stays a positive int
__device__ __forceinline__ RunBuf run_buf(const uint32_t *p, uint32_t n) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p), 0, (int)(min(n, kRunMax) * 4), 0x00027000);
}

// Replay of the recording count pass: persistent waves take quarters of record
// chunks, one record per lane.  A lane works out its record once (output
// address, source address in the leaf-id array, bounds check); the next
// quarter's records, then their offsets, are loaded meanwhile.  Leaf records
// go through a list in LDS, of which every half-wave takes every other one, RU
// at a time: lane l reads entry l of the record's 32 and stores it at its rank
// in the hit mask.  Ranges are copied by the whole wave.  Bound by memory
// (10M rectangles / 1M windows, 1.44G ids, fanout 64 SoA: 2.24 ms, 5.8 GB
// written and the leaf ids read through L2 and Infinity Cache); with addresses
// and bounds worked out by every lane, 40 vector instructions per 64 entries,
// and one range per half-wave at a time it took 2.65 ms, and 2.5 instead of
// 1.1 ms on 50M rectangles.
// BULK: ranges of at least kReplayBulkMin ids are deferred to the bulk copy,
// whose blocks share them (one half-wave copying a subtree of 32K ids alone
// takes 150 us); an instance of its own, since the branch costs registers.
template <bool BULK>
__global__ void __launch_bounds__(256, 8)   // the whole grid resident: the work is dealt by stride
replay_kernel(TreeView t, const uint64_t *__restrict__ offsets, uint32_t noffsets, uint32_t *__restrict__ ids,
              uint64_t cap, Ctrl *__restrict__ ctrl, uint4 *__restrict__ bulk, uint32_t bulk_cap) {
    constexpr uint32_t W = 4;   // waves per block
    // addresses are kept as pointers to global memory (through LDS
    // or a structure the compiler would lose that and use flat accesses)
    typedef const __attribute__((address_space(1))) uint32_t *Src;
    typedef __attribute__((address_space(1))) uint32_t *Dst;
    __shared__ Src lsrc[W][64];
    __shared__ Dst ldst[W][64];
    __shared__ uint32_t lmask[W][64];
    const uint32_t nchunks = ctrl->rec_nchunks;
    if (!nchunks || ctrl->rec_overflow || offsets[noffsets] > cap) return;
    typedef const __attribute__((address_space(1))) rec_vec *Rec;
    const Rec rec = (Rec)ctrl->rec_base;
    const Src rec_count = (Src)ctrl->rec_count;
    const uint32_t taken = min(ctrl->rec_chunks, nchunks), tail = ctrl->rec_tail;
    const uint32_t nunits = units_of(taken, tail);
    const uint64_t nrec = (uint64_t)nchunks * kRecChunk;
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6, half = lane >> 5, l = lane & 31u;
    const uint64_t below = lane ? ~0ull >> (64 - lane) : 0ull;
    const uint32_t lbit = 1u << l;
    // Unit u: records [64 * (u % 4), + 64) of chunk u / 4 (replay_units.h).  What is read ahead
    // (past the last unit: of the last one again) is looked at when its turn
    // comes; lanes without a record, all of them past the last unit, then take
    // an empty one.
    const uint32_t step = gridDim.x * W;
    rec_vec rv;
    uint32_t rcnt;
    auto load = [&](uint32_t u) {
        const uint32_t v = unit_loaded(u, nunits), c = v / kChunkUnits;
        rv = __builtin_nontemporal_load(rec + unit_place(v, lane, taken, nrec));
        rcnt = c < taken ? rec_count[c] : tail_count(c, taken, tail);
    };
    uint4 d;
    uint64_t o0, o1;
    bool in;
    auto arrive = [&](uint32_t u) {   // the loaded record, and its slot's offsets
        in = unit_has(u, nunits, lane, rcnt) && rv.w != 0;
        d = in ? make_uint4(rv.x, rv.y, rv.z, rv.w) : make_uint4(0u, 0u, t.first_leaf, 0u);
        o0 = offsets[d.x], o1 = offsets[d.x + 1];
    };
    // Hands a range to the bulk copy (the whole wave; scalars); false if its list is full.
    auto defer = [&](const uint32_t *src, uint32_t *dst, uint32_t n) {
        const uint32_t nd = (n + kBulkChunk - 1) / kBulkChunk;
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&ctrl->bulk_n, nd);
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        const bool fits = at < bulk_cap && nd <= bulk_cap - at;
        for (uint32_t k = lane; k < nd && at + k < bulk_cap; k += 64) {   // empty ones if not all fit
            const uint32_t off = k * kBulkChunk;
            const uint64_t to = (uint64_t)(dst - ids) + off;
            bulk[at + k] = make_uint4((uint32_t)(src - t.leaf_ids) + off, (uint32_t)to, (uint32_t)(to >> 32),
                                      fits ? min(kBulkChunk, n - off) : 0u);
        }
        return fits;
    };
    uint32_t unit = blockIdx.x * W + w;
    if (unit >= nunits) return;   // no block barriers below
    load(unit);
    arrive(unit);
    for (; unit < nunits; unit += step) {
        const bool run = in && (d.z & kRecRun);
        const uint64_t b = o0 + d.y;
        uint64_t n;
        const uint32_t *src;
        if (run) {
            const uint64_t s0 = leaf_start(t, d.z & ~kRecRun);
            n = leaf_start(t, d.w) - s0;
            src = t.leaf_ids + s0;
        } else {
            n = (uint32_t)__popc(d.w);
            src = t.leaf_ids + leaf_start(t, d.z & ~kRecHi) + ((d.z & kRecHi) ? 32u : 0u);
        }
        const bool bad = in && b + n > o1;
        if (bad) atomicOr(&ctrl->err, kErrBounds);
        const bool leaf = in && !run && !bad;
        const uint64_t lm = __ballot(leaf), rm = __ballot(run && !bad);
        const uint32_t nl = (uint32_t)__popcll(lm);
        // leaf records to the front, in order; the lanes without one fill the
        // places behind with records without hits
        {
            const uint32_t at = leaf ? (uint32_t)__popcll(lm & below) : nl + (uint32_t)__popcll(~lm & below);
            lsrc[w][at] = (Src)(leaf ? src : t.leaf_ids);
            ldst[w][at] = (Dst)(ids + b);
            lmask[w][at] = leaf ? d.w : 0u;
        }
        const uint32_t rn = (uint32_t)n;   // n ids of one tree: fewer than 2^32
        uint32_t *const dst = ids + b;
        __builtin_amdgcn_wave_barrier();
        load(unit + step);
        constexpr uint32_t RU = 8;   // leaf records in flight per half-wave
        // A leaf record's ids are a short run next to the runs of the records
        // beside it (the same wave, the same L2): cached stores let L2 merge
        // their partly written lines, where stores that bypass it write each
        // part to memory on its own (fill 2.83 -> 2.67 ms at 10M rectangles /
        // 1M windows).  Range copies write whole lines and keep the bypassing
        // stores.
        for (uint32_t r0 = 0; r0 < nl; r0 += 2 * RU) {
            uint32_t v[RU], m[RU];
#pragma unroll
            for (uint32_t u = 0; u < RU; ++u) {
                const uint32_t r = r0 + 2 * u + half;
                m[u] = lmask[w][r];
                // lanes without a hit read the first entry: no branch
                v[u] = lsrc[w][r][(m[u] & lbit) ? l : 0u];
            }
            asm volatile("" ::: "memory");   // keeps the loads above the conditional stores
#pragma unroll
            for (uint32_t u = 0; u < RU; ++u)
                if (m[u] & lbit) ldst[w][r0 + 2 * u + half][__popc(m[u] & (lbit - 1))] = v[u];
        }
        // Ranges: the whole wave copies one, four at a time; addresses and
        // lengths are scalars, the buffers' bounds take the ragged ends.
        constexpr uint32_t QU = 4, CU = 4;   // ranges in flight, loads of each
        for (uint64_t left = rm; left;) {
            RunBuf from[QU], to[QU];
            const uint32_t *rs[QU];
            uint32_t *rd[QU];
            uint32_t x[QU][CU], len[QU];
#pragma unroll
            for (uint32_t u = 0; u < QU; ++u) {
                const int at = left ? __builtin_ctzll(left) : 0;
                len[u] = left ? (uint32_t)__builtin_amdgcn_readlane((int)rn, at) : 0u;
                left &= left - 1;
                rs[u] = scalar64(src, at);
                rd[u] = scalar64(dst, at);
                if (BULK && len[u] >= kReplayBulkMin && defer(rs[u], rd[u], len[u])) len[u] = 0;
                from[u] = run_buf(rs[u], len[u]);
                to[u] = run_buf(rd[u], len[u]);
#pragma unroll
                for (uint32_t k = 0; k < CU; ++k)
                    x[u][k] = __builtin_amdgcn_raw_buffer_load_b32(from[u], (int)(lane * 4 + k * 256), 0, 0);
            }
#pragma unroll
            for (uint32_t u = 0; u < QU; ++u) {
#pragma unroll
                for (uint32_t k = 0; k < CU; ++k)
                    __builtin_amdgcn_raw_buffer_store_b32(x[u][k], to[u], (int)(lane * 4 + k * 256), 0, kStoreNt);
            }
#pragma unroll
            for (uint32_t u = 0; u < QU; ++u) {
                for (uint32_t i = 64 * CU; i < len[u]; i += 64 * CU) {
                    if (i % kRunMax == 0) {   // the next buffer of a very long run
                        from[u] = run_buf(rs[u] + i, len[u] - i);
                        to[u] = run_buf(rd[u] + i, len[u] - i);
                    }
                    const int o = (int)(i % kRunMax * 4);   // scalar part of the offset: below the buffer's size
#pragma unroll
                    for (uint32_t k = 0; k < CU; ++k)
                        x[u][k] = __builtin_amdgcn_raw_buffer_load_b32(from[u], (int)(lane * 4 + k * 256), o, 0);
#pragma unroll
                    for (uint32_t k = 0; k < CU; ++k)
                        __builtin_amdgcn_raw_buffer_store_b32(x[u][k], to[u], (int)(lane * 4 + k * 256), o, kStoreNt);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        arrive(unit + step);
    }
}

hipError_t launch_replay(const TreeView &t, const uint64_t *offsets, uint32_t noffsets, uint32_t *ids,
                         uint64_t cap, Ctrl *ctrl, uint4 *defer, uint32_t defer_cap, uint32_t max_chunks, hipStream_t s) {
    const uint32_t most = (uint32_t)num_cus() * 8;   // no more blocks than chunks can be taken
    const dim3 grid(max_chunks < most ? max_chunks : most), block(256);
    if (defer)
        hipLaunchKernelGGL(replay_kernel<true>, grid, block, 0, s, t, offsets, noffsets, ids, cap, ctrl, defer,
                           defer_cap);
    else
        hipLaunchKernelGGL(replay_kernel<false>, grid, block, 0, s, t, offsets, noffsets, ids, cap, ctrl,
                           (uint4 *)nullptr, 0u);
    return hipGetLastError();
}

hipError_t launch_bulk_copy(const uint32_t *leaf_ids, BulkList replayed, BulkList walked, uint32_t *ids, Ctrl *ctrl,
                            hipStream_t s) {
    hipLaunchKernelGGL(bulk_copy_kernel, dim3((uint32_t)num_cus() * 8), dim3(256), 0, s, leaf_ids, replayed, walked,
                       ids, ctrl);
    return hipGetLastError();
}

int num_cus() {
    static int cus = 0;
    if (!cus) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 256;
        hipDeviceProp_t p;
        if (hipGetDeviceProperties(&p, dev) != hipSuccess) return 256;
        cus = p.multiProcessorCount > 0 ? p.multiProcessorCount : 256;
    }
    return cus;
}

template <int G, int LAYOUT, int MODE>
static hipError_t launch_g(const TreeView &t, const float4 *q, uint32_t nq, uint32_t *counts,
                           const uint64_t *offsets, uint32_t *ids, uint64_t cap, Ctrl *ctrl,
                           uint32_t slot, const SelectPlan &plan, uint32_t noffsets, hipStream_t s) {
    const uint32_t stack_cap = stack_bound(t.height, t.fanout);
    const uint32_t groups_per_block = 256 / G;
    const size_t smem = (size_t)groups_per_block * stack_cap * sizeof(uint32_t);
    uint64_t want = ((uint64_t)nq + groups_per_block - 1) / groups_per_block;
    uint64_t persistent = (uint64_t)num_cus() * 8;
    uint32_t blocks = (uint32_t)(want < persistent ? want : persistent);
    if (plan.heavy) blocks = (uint32_t)persistent;   // split items add work beyond nq
    blocks = (blocks + kXcds - 1) / kXcds * kXcds;   // every XCD gets blocks
    // the fill pass with deferred contained runs is an instance of its own:
    // the deferral branch costs the in-pass copies registers and time
    const bool la = MODE != SEL_STATS && t.lookahead;
    constexpr int EXT = MODE == SEL_FILL ? 1 : 0;
    if (MODE == SEL_FILL && plan.bulk) {
        if (la)
            hipLaunchKernelGGL((select_kernel<G, LAYOUT, MODE, 1, EXT>), dim3(blocks), dim3(256), smem, s,
                               t, q, nq, counts, offsets, ids, cap, ctrl, slot, stack_cap, plan, noffsets);
        else
            hipLaunchKernelGGL((select_kernel<G, LAYOUT, MODE, 0, EXT>), dim3(blocks), dim3(256), smem, s,
                               t, q, nq, counts, offsets, ids, cap, ctrl, slot, stack_cap, plan, noffsets);
    } else if (la)
        hipLaunchKernelGGL((select_kernel<G, LAYOUT, MODE, 1, 0>), dim3(blocks), dim3(256), smem, s, t, q, nq,
                           counts, offsets, ids, cap, ctrl, slot, stack_cap, plan, noffsets);
    else
        hipLaunchKernelGGL((select_kernel<G, LAYOUT, MODE, 0, 0>), dim3(blocks), dim3(256), smem, s, t, q, nq,
                           counts, offsets, ids, cap, ctrl, slot, stack_cap, plan, noffsets);
    return hipGetLastError();
}

template <int G, int LAYOUT, int PHASE>
static hipError_t launch_split_g(const TreeView &t, const float4 *q, uint32_t nq, uint32_t split_first,
                                 uint32_t kmin, uint32_t budget, float min_area, uint32_t *nslots,
                                 const uint64_t *slot_first, uint4 *heavy, const uint32_t *order, Ctrl *ctrl,
                                 hipStream_t s) {
    const uint32_t stack_cap = stack_bound(t.height, t.fanout);
    const uint32_t groups_per_block = 256 / G;
    const size_t smem = (size_t)groups_per_block * stack_cap * sizeof(uint32_t);
    uint64_t want = ((uint64_t)nq + groups_per_block - 1) / groups_per_block;
    uint64_t persistent = (uint64_t)num_cus() * 8;
    uint32_t blocks = (uint32_t)(want < persistent ? want : persistent);
    blocks = (blocks + kXcds - 1) / kXcds * kXcds;
    hipLaunchKernelGGL((split_kernel<G, LAYOUT, PHASE>), dim3(blocks), dim3(256), smem, s, t, q, nq, split_first,
                       kmin, budget, min_area, nslots, slot_first, heavy, order, ctrl, stack_cap);
    return hipGetLastError();
}

template <int G, int LAYOUT>
static hipError_t launch_m(const TreeView &t, const float4 *q, uint32_t nq, int mode, uint32_t *counts,
                           const uint64_t *offsets, uint32_t *ids, uint64_t cap, Ctrl *ctrl,
                           uint32_t slot, const SelectPlan &plan, uint32_t noffsets, hipStream_t s) {
    switch (mode) {
    case SEL_COUNT:
        return launch_g<G, LAYOUT, SEL_COUNT>(t, q, nq, counts, offsets, ids, cap, ctrl, slot, plan, noffsets, s);
    case SEL_FILL:
        return launch_g<G, LAYOUT, SEL_FILL>(t, q, nq, counts, offsets, ids, cap, ctrl, slot, plan, noffsets, s);
    default:
        return launch_g<G, LAYOUT, SEL_STATS>(t, q, nq, counts, offsets, ids, cap, ctrl, slot, plan, noffsets, s);
    }
}

template <int G>
static hipError_t launch_l(const TreeView &t, const float4 *q, uint32_t nq, int mode, uint32_t *counts,
                           const uint64_t *offsets, uint32_t *ids, uint64_t cap, Ctrl *ctrl,
                           uint32_t slot, const SelectPlan &plan, uint32_t noffsets, hipStream_t s) {
    switch (t.layout) {
    case LAYOUT_AOS:
        return launch_m<G, LAYOUT_AOS>(t, q, nq, mode, counts, offsets, ids, cap, ctrl, slot, plan, noffsets, s);
    case LAYOUT_SOA:
        return launch_m<G, LAYOUT_SOA>(t, q, nq, mode, counts, offsets, ids, cap, ctrl, slot, plan, noffsets, s);
    default:
        return launch_m<G, LAYOUT_D2>(t, q, nq, mode, counts, offsets, ids, cap, ctrl, slot, plan, noffsets, s);
    }
}

hipError_t launch_select_pass(const TreeView &t, const float4 *q, uint32_t nq, int mode,
                              uint32_t *counts, const uint64_t *offsets, uint32_t *ids,
                              uint64_t cap, Ctrl *ctrl, uint32_t slot, const SelectPlan &plan,
                              uint32_t noffsets, hipStream_t s) {
    switch (group_width(t.fanout)) {
    case 16:
        return launch_l<16>(t, q, nq, mode, counts, offsets, ids, cap, ctrl, slot, plan, noffsets, s);
    case 32:
        return launch_l<32>(t, q, nq, mode, counts, offsets, ids, cap, ctrl, slot, plan, noffsets, s);
    default:
        return launch_l<64>(t, q, nq, mode, counts, offsets, ids, cap, ctrl, slot, plan, noffsets, s);
    }
}

// Blocks of gpb groups for nq windows.
static uint32_t walk_blocks(uint32_t nq, uint32_t gpb) {
    const uint32_t persistent = (uint32_t)num_cus() * 8;
    const uint64_t want = ((uint64_t)nq + gpb - 1) / gpb;
    const uint32_t blocks = (uint32_t)(want < persistent ? want : persistent);
    return (blocks + kXcds - 1) / kXcds * kXcds;   // every XCD gets blocks
}

uint32_t walk_fixed_chunks(uint32_t fanout, uint32_t nq, uint32_t nchunks) {
    const uint32_t gpb = 256 / group_width(fanout);
    const uint32_t n = std::min(nq, walk_blocks(nq, gpb) * gpb);
    return nchunks >= n && nchunks - n >= n / 16 ? n : 0u;
}

template <int G, int LAYOUT, bool WIDE>
static hipError_t launch_walk_w(const TreeView &t, const float4 *q, uint32_t nq, uint32_t *counts, Ctrl *ctrl,
                                const SelectPlan &plan, uint2 *items, uint32_t icap, hipStream_t s) {
    const uint32_t stack_cap = walk_stack_bound(t.height, t.fanout);
    const uint32_t gpb = 256 / G;
    size_t smem = (size_t)gpb * stack_cap * sizeof(uint32_t);
    if (plan.rec) smem = (smem + 15) / 16 * 16 + (size_t)gpb * kRecBuf * 16;   // the groups' record buffers
    const uint32_t persistent = (uint32_t)num_cus() * 8;
    const uint32_t blocks = walk_blocks(nq, gpb);
    // units per counter update: the more each group will take, the more
    const uint64_t groups = (uint64_t)blocks * gpb;
    const uint32_t chunk = nq >= 16 * groups ? 8u : nq >= 8 * groups ? 4u : nq >= 2 * groups ? 2u : 1u;
    const RecArena ar{plan.rec, plan.rec_count, plan.rec_nchunks, plan.rec_fixed};
    const WalkItems none{nullptr, 0, nullptr, nullptr};
    const dim3 block(256);
    if (!plan.rec) {
        hipLaunchKernelGGL((walk_kernel<G, LAYOUT, false, 0, false, WIDE>), dim3(blocks), block, smem, s, t, q, nq,
                           plan.order, counts, ctrl, chunk, stack_cap, ar, 0u, none, none);
        return hipGetLastError();
    }
    if (!items) {
        hipLaunchKernelGGL((walk_kernel<G, LAYOUT, true, 0, false, WIDE>), dim3(blocks), block, smem, s, t, q, nq,
                           plan.order, counts, ctrl, chunk, stack_cap, ar, 0u, none, none);
        return hipGetLastError();
    }
    // three launches: queries, what the large ones left, what the large
    // subtrees among those left
    const WalkItems a{items, icap, ctrl->hlist, ctrl->hwork[0]};
    const WalkItems b{items + (size_t)kXcds * icap, icap, ctrl->budget_used, ctrl->hwork[1]};
    hipLaunchKernelGGL((walk_kernel<G, LAYOUT, true, 0, true, WIDE>), dim3(blocks), block, smem, s, t, q, nq, plan.order,
                       counts, ctrl, chunk, stack_cap, ar, kWalkBudget0, none, a);
    hipLaunchKernelGGL((walk_kernel<G, LAYOUT, true, 1, true, WIDE>), dim3(persistent), block, smem, s, t, q, nq, plan.order,
                       counts, ctrl, 2u, stack_cap, ar, kWalkBudget1, a, b);
    hipLaunchKernelGGL((walk_kernel<G, LAYOUT, true, 1, false, WIDE>), dim3(persistent), block, smem, s, t, q, nq,
                       plan.order, counts, ctrl, 2u, stack_cap, ar, 0u, b, none);
    return hipGetLastError();
}

template <int G, int LAYOUT>
static hipError_t launch_walk_g(const TreeView &t, const float4 *q, uint32_t nq, uint32_t *counts, Ctrl *ctrl,
                                const SelectPlan &plan, uint2 *items, uint32_t icap, hipStream_t s) {
    // node offsets fit 32 bits below 4 GiB of nodes
    if ((uint64_t)t.n_nodes * t.node_bytes <= 0xFFFFFFFFull)
        return launch_walk_w<G, LAYOUT, false>(t, q, nq, counts, ctrl, plan, items, icap, s);
    return launch_walk_w<G, LAYOUT, true>(t, q, nq, counts, ctrl, plan, items, icap, s);
}

hipError_t launch_walk(const TreeView &t, const float4 *q, uint32_t nq, uint32_t *counts, Ctrl *ctrl,
                       const SelectPlan &plan, uint2 *items, uint32_t items_per_list, hipStream_t s) {
#define RT_WALK(G_, L_) launch_walk_g<G_, L_>(t, q, nq, counts, ctrl, plan, items, items_per_list, s)
    const uint32_t G = group_width(t.fanout);
    if (t.layout == LAYOUT_AOS) return G == 16 ? RT_WALK(16, LAYOUT_AOS) : G == 32 ? RT_WALK(32, LAYOUT_AOS) : RT_WALK(64, LAYOUT_AOS);
    if (t.layout == LAYOUT_SOA) return G == 16 ? RT_WALK(16, LAYOUT_SOA) : G == 32 ? RT_WALK(32, LAYOUT_SOA) : RT_WALK(64, LAYOUT_SOA);
    return G == 16 ? RT_WALK(16, LAYOUT_D2) : G == 32 ? RT_WALK(32, LAYOUT_D2) : RT_WALK(64, LAYOUT_D2);
#undef RT_WALK
}

template <int G, int LAYOUT>
static hipError_t launch_shared_fill_g(const TreeView &t, const float4 *q, uint32_t nq, const uint32_t *order,
                                       uint32_t *counts, const uint64_t *offsets, uint32_t *ids, uint64_t cap, Ctrl *ctrl,
                                       uint32_t split_parent, uint32_t parents, hipStream_t s) {
    const uint32_t stack_cap = stack_bound(t.height, t.fanout);
    const size_t smem = (size_t)(256 / G) * stack_cap * sizeof(uint32_t);
    // at most about 4M units, which are looked at 16 per counter update
    const uint32_t shares = std::min(kMaxShares, std::max((1u << 22) / nq, 1u));
    hipLaunchKernelGGL((shared_fill_kernel<G, LAYOUT>), dim3((uint32_t)num_cus() * 8), dim3(256), smem, s, t, q, nq, order,
                       counts, offsets, ids, cap, ctrl, split_parent, parents, shares, stack_cap);
    return hipGetLastError();
}

hipError_t launch_shared_fill(const TreeView &t, const float4 *q, uint32_t nq, const uint32_t *order, uint32_t *counts,
                              const uint64_t *offsets, uint32_t *ids, uint64_t cap, Ctrl *ctrl, uint32_t split_parent,
                              uint32_t parents, hipStream_t s) {
#define RT_SHARED(G_, L_) \
    launch_shared_fill_g<G_, L_>(t, q, nq, order, counts, offsets, ids, cap, ctrl, split_parent, parents, s)
    const uint32_t G = group_width(t.fanout);
    if (t.layout == LAYOUT_AOS) return G == 16 ? RT_SHARED(16, LAYOUT_AOS) : G == 32 ? RT_SHARED(32, LAYOUT_AOS) : RT_SHARED(64, LAYOUT_AOS);
    if (t.layout == LAYOUT_SOA) return G == 16 ? RT_SHARED(16, LAYOUT_SOA) : G == 32 ? RT_SHARED(32, LAYOUT_SOA) : RT_SHARED(64, LAYOUT_SOA);
    return G == 16 ? RT_SHARED(16, LAYOUT_D2) : G == 32 ? RT_SHARED(32, LAYOUT_D2) : RT_SHARED(64, LAYOUT_D2);
#undef RT_SHARED
}

template <int PHASE>
static hipError_t launch_split_phase(const TreeView &t, const float4 *q, uint32_t nq, uint32_t split_first,
                                     uint32_t kmin, uint32_t budget, float min_area, uint32_t *nslots,
                                     const uint64_t *slot_first, uint4 *heavy, const uint32_t *order, Ctrl *ctrl,
                                     hipStream_t s) {
#define RT_SPLIT(G_, L_) \
    launch_split_g<G_, L_, PHASE>(t, q, nq, split_first, kmin, budget, min_area, nslots, slot_first, heavy, order, \
                                  ctrl, s)
    const uint32_t G = group_width(t.fanout);
    if (t.layout == LAYOUT_AOS) return G == 16 ? RT_SPLIT(16, LAYOUT_AOS) : G == 32 ? RT_SPLIT(32, LAYOUT_AOS) : RT_SPLIT(64, LAYOUT_AOS);
    if (t.layout == LAYOUT_SOA) return G == 16 ? RT_SPLIT(16, LAYOUT_SOA) : G == 32 ? RT_SPLIT(32, LAYOUT_SOA) : RT_SPLIT(64, LAYOUT_SOA);
    return G == 16 ? RT_SPLIT(16, LAYOUT_D2) : G == 32 ? RT_SPLIT(32, LAYOUT_D2) : RT_SPLIT(64, LAYOUT_D2);
#undef RT_SPLIT
}

hipError_t launch_split(const TreeView &t, const float4 *q, uint32_t nq, int phase, uint32_t split_parent,
                        uint32_t kmin, uint32_t hcap, float min_area, uint32_t *nslots, const uint64_t *slot_first,
                        uint4 *heavy, const uint32_t *order, Ctrl *ctrl, hipStream_t s) {
    return phase == 0 ? launch_split_phase<0>(t, q, nq, split_parent, kmin, hcap, min_area, nslots, slot_first,
                                              heavy, order, ctrl, s)
                      : launch_split_phase<1>(t, q, nq, split_parent, kmin, hcap, min_area, nslots, slot_first,
                                              heavy, order, ctrl, s);
}

// offsets[q] = slot_offsets[slot_first[q]] for q <= nq (the CSR of whole
// queries from the CSR of output slots)
__global__ void gather_offsets(const uint64_t *__restrict__ slot_first, const uint64_t *__restrict__ slot_off,
                               uint32_t nq, uint64_t *__restrict__ offsets) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i <= nq; i += gridDim.x * blockDim.x)
        offsets[i] = slot_off[slot_first[i]];
}

hipError_t launch_gather_offsets(const uint64_t *slot_first, const uint64_t *slot_off, uint32_t nq,
                                 uint64_t *offsets, hipStream_t s) {
    uint32_t blocks = (nq + 256) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(gather_offsets, dim3(blocks), dim3(256), 0, s, slot_first, slot_off, nq, offsets);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// query order for locality
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t spread16(uint32_t v) {
    v &= 0xFFFFu;
    v = (v | (v << 8)) & 0x00FF00FFu;
    v = (v | (v << 4)) & 0x0F0F0F0Fu;
    v = (v | (v << 2)) & 0x33333333u;
    v = (v | (v << 1)) & 0x55555555u;
    return v;
}

// Cell of a window center on a 64 x 64 grid over the tree's MBR, cells in
// Morton (Z) order.  Only the processing order depends on it; no result does.
__device__ __forceinline__ uint32_t order_cell(const float4 w, float lx, float ly, float sx, float sy) {
    float cx = (0.5f * w.x + 0.5f * w.z - lx) * sx;
    float cy = (0.5f * w.y + 0.5f * w.w - ly) * sy;
    cx = fminf(fmaxf(cx, 0.f), 63.f);   // NaN -> 0
    cy = fminf(fmaxf(cy, 0.f), 63.f);
    return spread16((uint32_t)cx) | (spread16((uint32_t)cy) << 1);
}

// Bucket sort of the queries by cell, three launches: queries per cell (LDS
// counters per block, one global update per cell a block has), a one-block
// scan, and the scatter (LDS ranks, each block reserving its share of a cell).
constexpr uint32_t kOrderT = 1024;

template <bool SCATTER>
__global__ void __launch_bounds__(kOrderT)
order_cells(const float4 *__restrict__ q, uint32_t nq, uint32_t per, float lx, float ly, float sx, float sy,
            uint32_t *__restrict__ cells, uint32_t *__restrict__ order) {
    __shared__ uint32_t c[kOrderCells];
    constexpr uint32_t R = 8;   // per <= R queries per thread
    for (uint32_t i = threadIdx.x; i < kOrderCells; i += kOrderT) c[i] = 0;
    __syncthreads();
    const uint32_t i0 = blockIdx.x * kOrderT * per + threadIdx.x;
    uint32_t cell[R], rank[R];
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        const uint32_t i = i0 + r * kOrderT;
        if (r < per && i < nq) {
            cell[r] = order_cell(q[i], lx, ly, sx, sy);
            rank[r] = atomicAdd(&c[cell[r]], 1u);
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < kOrderCells; i += kOrderT)
        if (c[i]) {
            const uint32_t at = atomicAdd(&cells[i], c[i]);
            if (SCATTER) c[i] = at;
        }
    if constexpr (SCATTER) {
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < R; ++r) {
            const uint32_t i = i0 + r * kOrderT;
            if (r < per && i < nq) order[c[cell[r]] + rank[r]] = i;
        }
    }
}

__global__ void __launch_bounds__(1024) order_scan(uint32_t *__restrict__ cells) {
    __shared__ uint32_t wsum[16];
    const uint32_t t = threadIdx.x, lane = t & 63u, w = t >> 6;
    uint32_t v[4], sum = 0;
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r) sum += v[r] = cells[4 * t + r];
    uint32_t inc = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t x = __shfl_up(inc, d);
        if ((int)lane >= d) inc += x;
    }
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t ex = inc - sum;
    for (uint32_t i = 0; i < w; ++i) ex += wsum[i];
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r) {
        cells[4 * t + r] = ex;
        ex += v[r];
    }
}

// 4 * kOrderCells + 4 * nq bytes are used, of batches that are ordered at all.
// The size is that of an earlier layout (two key buffers and the tables of
// 11-bit radix passes, more than that from kOrderMinQueries on), which keeps
// the sizes that a fixed scratch accepts.
uint64_t order_ws_bytes(uint64_t nq) {
    const auto al = [](uint64_t b) { return (b + 255) & ~255ull; };
    const uint64_t he = radix_hist_elems(nq, 11);
    return al(8 * nq) * 2 + al(4 * he) + al(8 * (he + 1)) + al(8 * scan_tmp_elems(he + 1));
}

hipError_t launch_query_order(const float4 *q, uint32_t nq, const float *mbr, void *ws, const uint32_t **order,
                              hipStream_t s) {
    uint32_t *cells = static_cast<uint32_t *>(ws);
    uint32_t *out = cells + kOrderCells;
    float lx = mbr[0], ly = mbr[1], w = mbr[2] - mbr[0], h = mbr[3] - mbr[1];
    const bool ok = (w > 0.f) && (h > 0.f) && (w < 3.0e38f) && (h < 3.0e38f);
    const float sx = ok ? 64.f / w : 0.f, sy = ok ? 64.f / h : 0.f;
    if (!ok) lx = ly = 0.f;
    // few queries: one per thread, so that there are blocks to run; many:
    // eight, so that a block updates each cell's counter once for more of them
    const uint32_t per = nq <= 131072 ? 1u : 8u;
    const dim3 grid((nq + kOrderT * per - 1) / (kOrderT * per)), block(kOrderT);
    hipLaunchKernelGGL(order_cells<false>, grid, block, 0, s, q, nq, per, lx, ly, sx, sy, cells, (uint32_t *)nullptr);
    hipLaunchKernelGGL(order_scan, dim3(1), dim3(1024), 0, s, cells);
    hipLaunchKernelGGL(order_cells<true>, grid, block, 0, s, q, nq, per, lx, ly, sx, sy, cells, out);
    *order = out;
    return hipGetLastError();
}

const uint32_t *query_order_result(const void *ws, uint64_t nq) {
    (void)nq;
    return static_cast<const uint32_t *>(ws) + kOrderCells;
}

}  // namespace rtk
