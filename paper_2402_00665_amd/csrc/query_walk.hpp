// Single-tree range queries: packets of queries walk the tree together; the
// rest of a heavy packet is cut into tasks for other waves; the fill copies
// or walks again.
#pragma once
#pragma clang fp contract(off)

#include "query_common.hpp"
#include "task_pool.hpp"

namespace lbvh {
namespace {

// the lanes where b holds (__ballot goes through a vector register)
__device__ __forceinline__ uint64_t ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }

__device__ __forceinline__ uint64_t shfl64(uint64_t v, int src)
{
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, src);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(v >> 32), src);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ int64_t readlane64(int64_t v, int lane)
{
    return ((int64_t)__builtin_amdgcn_readlane((int)(v >> 32), lane) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
}

__device__ __forceinline__ int wave_max(int v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = max(v, __shfl_xor(v, off));
    return v;
}

__device__ __forceinline__ float4 readlane4(float4 v, int lane)
{
    auto get = [&](float x) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane)); };
    return make_float4(get(v.x), get(v.y), get(v.z), get(v.w));
}

// ---------------------------------------------------------------- records

// A packet that left the rest of its walk to others: its queries that have
// a rest (each one's first leaf is in `resume`), its number, its first task
// and how many.
struct HeavyPacket {
    uint64_t queries;
    int32_t packet, first, tasks;
    int32_t nodes;        // of the rest, in leaf order, as the walk left them (0: no room for them)
    uint32_t first_node;  // the first of them
    int32_t unused;
};

// A node and the queries of the packet that walk it: passed its box, and of
// these the ones that contain it.
struct Task {
    int32_t l, r, g;      // leaf range, split
    int32_t packet;
    uint64_t in, all;
};

struct QueryCtrl {   // the count call's control words, zeroed at its start
    uint32_t done;       // one in kSample of the waves whose light walks are finished
    uint32_t scan_tile;  // the scan's tile counter
    uint32_t nodes;      // nodes that heavy packets left, and
    uint32_t heavy;      // heavy packets: one add moves both
    unsigned long long tasks;   // tasks asked for
    uint32_t error;      // at kQueryErrorByte
    int32_t ordered;     // the queries were walked in the order `perm`
    uint32_t tasks_end;  // where the pool of tasks ends when more were asked for than it holds
    uint32_t own;        // some packet's tasks lie in places of its own
    uint32_t sort_tile[2];
    uint32_t steps;      // of the waves that `done` counts, in units of kStepUnit
};
static_assert(offsetof(QueryCtrl, error) == kQueryErrorByte, "error word");
static_assert(offsetof(QueryCtrl, nodes) % 8 == 0 && offsetof(QueryCtrl, heavy) == offsetof(QueryCtrl, nodes) + 4,
              "one 64-bit word");

// ------------------------------------------------------------ packet walk
//
// One wave walks a packet of up to 64 queries (neighbours, where the queries
// are walked in Morton order) down the tree together, left to right: the
// current node is the wave's, one step loads both its children by scalar
// loads, and each lane tests its own query against both.  The right child
// waits on the wave's stack with the mask of the queries that passed it.
// At a node of at most kLeaves leaves the wave changes sides: each lane holds
// four of its leaf boxes, the queries that passed are read from LDS one after
// another, and a ballot gives the hits of each in leaf order (the tests are
// monotone under box inclusion, so the passing leaves of the range are exactly
// what Alg. 1 reports below the node, in its order).  A node whose box a query
// contains reports its leaf range from leaf_perm.  Ropes serve here only as
// the ends of the leaf ranges.
//
// What it is bound by, and what was measured (2^20 spheres of 16 neighbours
// over 2^23 points; 2^20 segments with 216 hits on 2^24 clustered boxes):
//   * one walk per lane, with leaves tested four at a time: 2.4 and 27 ms; each
//     lane fetches its own nodes, 12 and 178 GB in all, at the memory's rate;
//   * packets that follow the ropes and test 64 leaves at a time: 0.87 and
//     13.9 ms, 2.3 and 50 GB, bound half by the vector instructions of the
//     leaf tests and half by the latency of one node after another;
//   * this form: 0.65 and 7.3 ms.  256 leaves at a time cost more tests than
//     64 and save three of four round trips; 128 and 512 were slower (1.10 and
//     1.19 against 1.03 ms for the whole call on the spheres).
// A step takes about 0.7 us when the machine is nearly idle, so a walk's length
// sets the time of a small call, and packets of one query are used until the
// queries fill the machine.
constexpr int kLeaves = 256;
constexpr int kLookEvery = 32;   // steps between looks at the other waves
// one wave in so many counts itself done: adds to one word take turns, about
// 8 ns each (10^4 waves that all did: 77 us on a walk of 56)
constexpr uint32_t kSample = 16;
constexpr int kStepUnit = 4;        // the sum of steps counts in these
// ... and while it runs dry a packet is only worth cutting when it has taken
// this many times the mean walk's steps, or kLongCall (2^20 spheres of 8 hits
// 939 us without, 892 at 2, 878 at 3, 897 at 4; 2^20 segments, whose mean is
// long, 16.0 ms without, 17.9 at 3 with no kLongCall)
constexpr int kLongFor = 3, kLongCall = 512;
constexpr int kLongWalk = 1 << 16;  // steps after which a packet leaves its rest in any case
constexpr int kLongRange = 4096;    // leaves of a contained range that a light walk leaves to others
constexpr int kDrainWaves = 1024;   // walking waves at which the machine runs dry: one a SIMD (512 and 2048: slower)
constexpr int kWalkBlock = 64;
constexpr int kPacketDepth = 96;    // paths have at most 93 levels (see kRayDepth)

template <class Q>
struct PacketLds {
    int4 range[kPacketDepth];       // waiting nodes: first leaf, last leaf, split, unused
    int4 masks[kPacketDepth];       // ... queries that passed, of these the ones that contain it
    alignas(16) char queries[64 * sizeof(Q)];
};

__device__ __forceinline__ void load_uniform(const float4 *nodes, int v, float4 &a, float4 &b)
{
    typedef float Quad __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(4))) Quad *Const;
    Const p = (Const)(uintptr_t)(nodes + 2 * (int64_t)v);
    const Quad x = p[0], y = p[1];
    a = make_float4(x.x, x.y, x.z, x.w);
    b = make_float4(y.x, y.y, y.z, y.w);
}

// Where a packet walk stopped: the current node, if `in` is not zero, and so
// many waiting nodes on the stack.
struct PacketStop {
    int l, r, g, waiting;
    uint64_t in, all;
};

// What a packet walk covers.
struct PacketRun {
    int l, r, g;              // the node it starts at: leaf range, split (l -1: the root)
    uint64_t in, all;         // its queries there
    int from;                 // this lane's query: first leaf that counts
    const QueryCtrl *ctrl;    // light walks: counts the waves that finished (else null),
    uint32_t waves;           // ... of so many
    int patience;             // steps before it may leave the rest to others
};

// FILL false: counts the hits of each lane's query and keeps the first
// `limit` of them from out[at] on; a heavy packet returns the queries that
// have a rest in `left` and each lane's first leaf of it in `rest`.  FILL
// true: writes the first `limit` hits.
// (No node of at most kLeaves leaves holds a query's first leaf other than as
// its own first: it is the first leaf of a node that waited on a stack, whose
// parent has more leaves.)
template <class Q, class T, bool FILL>
__device__ __forceinline__ int packet_walk(const Tree &tr, const PacketRun &run, const Q &q, bool mine,
                                           PacketLds<Q> &lds, int32_t *__restrict__ out, int64_t out_at,
                                           int limit, uint64_t &left, int &rest, int *took, PacketStop *stop_at)
{
    const int lane = threadIdx.x & 63;
    const int leaf0 = tr.leaf0();
    const T *shared = reinterpret_cast<const T *>(lds.queries);
    const T t(q);
    if (mine) reinterpret_cast<T *>(lds.queries)[lane] = t;
    wave_sync();
    const bool capped = !FILL && tr.budget > 0;
    int budget = (int)tr.walk_budget();   // 2n, at most 2^31 - 4, or the knob's
    int cnt = 0, steps = 0, sp = 0, next_look = run.patience;
    bool off = !mine;      // this lane's query has stopped
    left = 0;
    rest = 0;
    // the current node: range, split, queries that passed it and contain it
    int l = run.l, r = run.r, g = run.g;
    uint64_t in = run.in, all = run.all;
    auto split_of = [&](float4 a) { return tr.index(__float_as_int(a.w)); };
    auto contained = [&](uint64_t some, int len, float4 a, float4 b) -> uint64_t {
        return some != 0 && len > kLeaves ? ballot(q.contains(a, b)) & some : 0ull;
    };
    if (l < 0) {
        float4 a, b;
        load_uniform(tr.nodes, 0, a, b);
        l = 0;
        r = tr.n - 1;
        g = split_of(a);
        in = ballot(mine && t.test(a, b));
        all = contained(in, tr.n, a, b);
    }
    // Stop in front of the current node.  A query's rest begins at the first
    // waiting node that has it: before that, a node that contains it may
    // already have been reported beyond the current one.
    auto leave = [&]() {
        wave_sync();
        left = in;
        rest = l;
        for (int k = sp - 1; k >= 0; --k) {
            const int4 mk = lds.masks[k];
            const uint64_t mm = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(mk.y) << 32) |
                                (uint32_t)__builtin_amdgcn_readfirstlane(mk.x);
            if (((mm & ~left) >> lane) & 1) rest = lds.range[k].x;
            left |= mm;
        }
        left &= ballot(!off);
        if (stop_at) *stop_at = PacketStop{l, r, g, sp, in, all};
    };
    // hits of query s, one bit per lane, whose leaf's primitive is prim
    auto report = [&](int s, uint64_t hits, int32_t prim) {
        if (hits) {
            const int c = __builtin_amdgcn_readlane(cnt, s);
            const int lim = FILL ? __builtin_amdgcn_readlane(limit, s) : limit;
            if (c < lim) {
                int32_t *o = out + (readlane64(out_at, s) + c);
                const int at = (int)lanes_below(hits);
                if (((hits >> lane) & 1) && at < lim - c) o[at] = prim;
            }
            cnt = lane == s ? c + __popcll(hits) : cnt;
        }
    };
    while (true) {
        if (in != 0) {
            // (the nodes of a tree are met once each, at most kPacketDepth of
            // them waiting: this ends a walk on nodes that are no tree; looked
            // at behind the loads of the children, 2^20 spheres took 902
            // instead of 888 us)
            if ((--budget | (kPacketDepth - 1 - sp)) < 0) {
                if (lane == 0) tr.budget_spent();
                break;
            }
            ++steps;
            if (r - l < kLeaves) {
                float4 lo[kLeaves / 64], hi[kLeaves / 64];
#pragma unroll
                for (int w = 0; w < kLeaves / 64; ++w)
                    if (w == 0 || 64 * w <= r - l)
                        tr.load_leaf_box(leaf0 + (l + 64 * w + lane < r ? l + 64 * w + lane : r), lo[w], hi[w]);
                steps += __popcll(in) >> 2;   // (a step's time, in about 4 queries' tests)
                for (uint64_t todo = in; todo; todo &= todo - 1) {
                    const int s = __ffsll((unsigned long long)todo) - 1;
                    const T x = shared[s];
#pragma unroll
                    for (int w = 0; w < kLeaves / 64; ++w)
                        if (w == 0 || 64 * w <= r - l)
                            report(s, ballot(x.leaf(lo[w], hi[w]) && l + 64 * w + lane <= r), __float_as_int(lo[w].w));
                }
                if (FILL) off = off || cnt >= limit;
                in = 0;
            } else {
                if (all) {
                    if (run.ctrl && !capped && r - l >= kLongRange) {
                        leave();
                        break;
                    }
                    steps += __popcll(all) * (1 + ((r - l) >> 7));   // (the fill copies the range)
                    for (uint64_t todo = all; todo; todo &= todo - 1) {
                        const int s = __ffsll((unsigned long long)todo) - 1;
                        const int c = __builtin_amdgcn_readlane(cnt, s);
                        const int lim = FILL ? __builtin_amdgcn_readlane(limit, s) : limit;
                        const int first = max(l, __builtin_amdgcn_readlane(run.from, s));
                        const int n = min(r - first + 1, lim - c);
                        int32_t *o = out + (readlane64(out_at, s) + c);
                        for (int k = lane; k < n; k += 64) o[k] = tr.perm[first + k];
                    }
                    if ((all >> lane) & 1) {
                        cnt += r - max(l, run.from) + 1;
                        off = off || (FILL && cnt >= limit);
                    }
                    in &= ~all;
                }
                if (in != 0) {
                    // both children
                    const bool lleaf = g == l, rleaf = g + 1 == r;
                    float4 la, lb, ra, rb;
                    load_uniform(tr.nodes, lleaf ? leaf0 + g : g, la, lb);
                    load_uniform(tr.nodes, rleaf ? leaf0 + r : g + 1, ra, rb);
                    // (tests on every lane: a branch around one would wait for
                    // the first child before it asks for the second)
                    const bool pl = t.test(la, lb) & (g >= run.from);
                    const bool pr = t.test(ra, rb) & (r >= run.from);
                    const uint64_t ml = ballot(pl) & in, mr = ballot(pr) & in;
                    if (mr) {
                        const uint64_t ar = contained(mr, r - g, ra, rb);
                        if (lane == 0) {
                            lds.range[sp] = make_int4(g + 1, r, split_of(ra), 0);
                            lds.masks[sp] = make_int4((int)(uint32_t)mr, (int)(mr >> 32), (int)(uint32_t)ar,
                                                      (int)(ar >> 32));
                        }
                        ++sp;
                    }
                    all = contained(ml, g - l + 1, la, lb);
                    in = ml;
                    r = g;
                    g = split_of(la);
                    if (in) continue;
                }
            }
        }
        if (sp == 0) break;
        // time to leave the rest of the queries that have one to other waves?
        if (run.ctrl && !capped && steps >= next_look) {
            next_look = steps + kLookEvery;
            bool stop = run.waves <= (uint32_t)kDrainWaves || steps >= kLongWalk;
            if (!stop) {
                const uint32_t done = __hip_atomic_load(&run.ctrl->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const uint32_t sum = __hip_atomic_load(&run.ctrl->steps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                stop = (int)(run.waves - kSample * done) <= kDrainWaves &&
                       (steps >= kLongCall || (uint64_t)steps * done >= (uint64_t)kLongFor * kStepUnit * sum);
            }
            if (stop) {
                in = 0;
                leave();
                break;
            }
        }
        wave_sync();
        --sp;
        const int4 rg = lds.range[sp], mk = lds.masks[sp];
        l = __builtin_amdgcn_readfirstlane(rg.x);
        r = __builtin_amdgcn_readfirstlane(rg.y);
        g = __builtin_amdgcn_readfirstlane(rg.z);
        const uint64_t on = ballot(!off);
        in = on & (((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(mk.y) << 32) |
                   (uint32_t)__builtin_amdgcn_readfirstlane(mk.x));
        all = on & (((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(mk.w) << 32) |
                    (uint32_t)__builtin_amdgcn_readfirstlane(mk.z));
        wave_sync();
    }
    wave_sync();   // the packet's LDS is free again
    if (took) *took = steps;
    return cnt;
}

// `whole`: the lanes of the packet or task, of which those with `mine` walk.
// All of them decide which form of the test is used, so that the count and
// the fill, which has fewer queries to walk, use the same one.
template <class Q, bool FILL>
__device__ __forceinline__ int packet(const Tree &tr, const PacketRun &run, const Q &q, bool whole, bool mine,
                                      PacketLds<Q> &lds, int32_t *__restrict__ out, int64_t at, int limit,
                                      uint64_t &left, int &rest, int *took = nullptr, PacketStop *stop_at = nullptr)
{
    if (ballot(whole && !q.plain()) == 0) {
        if (tr.points) return packet_walk<Q, typename Q::PlainPoint, FILL>(tr, run, q, mine, lds, out, at, limit, left, rest, took, stop_at);
        return packet_walk<Q, typename Q::Plain, FILL>(tr, run, q, mine, lds, out, at, limit, left, rest, took, stop_at);
    }
    return packet_walk<Q, Q, FILL>(tr, run, q, mine, lds, out, at, limit, left, rest, took, stop_at);
}

// ------------------------------------------------------------ light walks
//
// Every query walks from the root in a packet.  The first kHitCache hits of
// a query are kept for the fill call.  A packet is heavy once it has taken
// `patience` steps, and far more than others, while the machine runs dry, or
// kLongWalk, or when it meets a node of more than kLongRange leaves that one of
// its queries contains: then it stops in front of its next node, and the rest,
// the leaves from that node's first one on, is cut into tasks, from that node
// and those that wait on its stack (kept where `rows` and `places` will be).  The machine runs dry when no
// more than kDrainWaves of the launch's waves are still walking: until then
// other waves fill the gaps of a long walk, and cutting it up would only
// cost.  Where a walk stops depends on timing, the hits and their order do
// not: a query's hits are those of its light walk followed by those of its
// packet's tasks in leaf order.

// The packet that block b of `blocks` takes.  Blocks go round the 8 XCDs one
// by one; each XCD gets runs of kPacketRun neighbouring packets, which read
// many of the same nodes, so that its L2 holds them.
constexpr unsigned kPacketRun = 64;
__device__ __forceinline__ unsigned packet_of(unsigned b, unsigned blocks)
{
    const unsigned whole = blocks / (8 * kPacketRun) * (8 * kPacketRun);
    if (b >= whole) return b;
    const unsigned xcd = b % 8, k = b / 8;
    return (k / kPacketRun * 8 + xcd) * kPacketRun + k % kPacketRun;
}

// the query of a lane of packet `p` (-1: none)
__device__ __forceinline__ int packet_query(int64_t p, int packet_size, int m, const int32_t *perm)
{
    const int lane = threadIdx.x & 63;
    const int64_t t = p * packet_size + lane;
    int j = -1;
    if (lane < packet_size && t < m) j = perm ? perm[t] : (int)t;
    return (uint32_t)j < (uint32_t)m ? j : -1;   // always, unless the order's sort failed
}

template <class Q>
__global__ __launch_bounds__(kWalkBlock) void k_walk(Tree tr, const float *__restrict__ queries, int m,
                                                     int packet_size, int patience,
                                                     const int32_t *__restrict__ perm,
                                                     QueryCtrl *ctrl, int32_t *__restrict__ light,
                                                     int32_t *__restrict__ counts,
                                                     int32_t *__restrict__ cache,
                                                     int32_t *__restrict__ resume,
                                                     HeavyPacket *__restrict__ heavy, Task *__restrict__ nodes,
                                                     uint32_t max_nodes)
{
    __shared__ PacketLds<Q> lds;
    const int lane = threadIdx.x;
    const unsigned p = packet_of(blockIdx.x, gridDim.x);
    const int j = packet_query(p, packet_size, m, perm);
    const bool mine = j >= 0;
    Q q{};
    if (mine) q.load(queries, j);
    PacketRun run{};
    run.l = -1;
    run.ctrl = ctrl;
    run.waves = gridDim.x;
    run.patience = patience;
    uint64_t left;
    int rest, steps;
    PacketStop stop;
    const int cnt = packet<Q, false>(tr, run, q, mine, mine, lds, cache, (int64_t)(mine ? j : 0) * kHitCache,
                                     kHitCache, left, rest, &steps, &stop);
    if (mine) {
        light[j] = cnt;
        counts[j] = cnt;
        if ((left >> lane) & 1) resume[j] = rest;
    }
    if (left) {
        // the nodes of its rest, in leaf order, for the cut to start from
        // (fewer than 2^25 packets of at most 97 nodes: no carry)
        const int here = stop.in != 0;
        unsigned long long was = 0;
        if (lane == 0)
            was = atomicAdd(reinterpret_cast<unsigned long long *>(&ctrl->nodes),
                            (1ull << 32) | (uint32_t)(here + stop.waiting));
        const uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)was);
        const bool room = at <= max_nodes && (uint32_t)(here + stop.waiting) <= max_nodes - at;
        if (room) {
            if (here && lane == 0) nodes[at] = Task{stop.l, stop.r, stop.g, (int)p, stop.in, stop.all};
            for (int k = lane; k < stop.waiting; k += 64) {
                const int4 rg = lds.range[stop.waiting - 1 - k], mk = lds.masks[stop.waiting - 1 - k];
                nodes[at + here + k] = Task{rg.x, rg.y, rg.z, (int)p, ((uint64_t)(uint32_t)mk.y << 32) | (uint32_t)mk.x,
                                            ((uint64_t)(uint32_t)mk.w << 32) | (uint32_t)mk.z};
            }
        }
        if (lane == 0) {
            HeavyPacket h{};
            h.queries = left;
            h.packet = (int)p;
            h.nodes = room ? here + stop.waiting : 0;
            h.first_node = at;
            heavy[was >> 32] = h;
        }
    }
    if (lane == 0) {
        if (blockIdx.x / 8 % kSample == 0 && gridDim.x > (unsigned)kDrainWaves) {
            atomicAdd(&ctrl->steps, (uint32_t)(steps < 4096 ? steps : 4096) / kStepUnit);
            atomicAdd(&ctrl->done, 1u);
        }
    }
}

// ------------------------------------------------------------------- tasks
//
// One block cuts the rest of one heavy packet into tasks, level by level: an
// ordered list of nodes (range, split, queries that passed its box and that
// contain it), first those that the packet's walk left waiting, in which the
// nodes of more than `width` leaves are replaced by their children, as far as
// any query passes them.  Once they are not few, a level cuts those that are not
// much shorter than the longest: the parts of the short ones would fill the
// list and leave it whole.  A list longer than a quarter of `most` makes the
// width four times larger, one longer than half of it is left as it is.  The
// list is then the packet's tasks in leaf order.  Where the pool of tasks has
// no room for them (reserve_places), the packet is cut again from the root,
// into at most kOwnTasks tasks that have places of their own.
//
// Bound by the chain of levels, each at least a load's latency, of the packet
// with the longest one.  A lane holds a node and loads its children, so that a
// level loads once; a wave then takes its nodes to cut in turn, each lane
// testing its query.  While they are few, one wave works alone, without
// barriers (alone up to 2 or 4 cut nodes 31 and 26 us, up to 8 or 16 21).  On
// 150000 boxes of side 0.002 over 10^6 clustered boxes, and on 2^20 over 2^24:
// 21 and 82 us; from the root, each wave loading four nodes at a time, 58 and
// 126; so from the waiting nodes, 43 and 153.  Cutting all nodes at each level
// took 63 us for the latter, but left ranges of millions of leaves whole where
// the list filled up: 100 spheres of side 0.1 on 2^24 boxes 1334 us (now 253).
constexpr int kCutBlock = 512;  // (256 threads with lists of 512: 1.9 ms on the box queries, not 0.8)
constexpr int kCutWaves = kCutBlock / 64;
constexpr int kCutList = 1024;   // list entries, and so the most tasks of a packet
constexpr int kCutAlone = 32;    // nodes up to which one wave works alone,
constexpr int kCutFew = 8;       // ... while so many of them are cut
// a level cuts the nodes of at least this share of the longest one's length
// (2000 boxes of side 0.1 on 2^24: 0.49 ms, a quarter 2.98, an eighth 5.64)
constexpr int kCutFirst = 2;
static_assert(kCutList == 2 * kCutBlock, "a thread for each node of a list that is cut");

struct TaskCounter {
    QueryCtrl *ctrl;
    __device__ uint64_t add(uint32_t cnt) { return atomicAdd(&ctrl->tasks, (unsigned long long)cnt); }
    __device__ void close(uint32_t end) { ctrl->tasks_end = end; }
};

struct CutNode {
    int l, r, g;
    uint64_t in, all;
};

struct CutList {
    int l[kCutList], r[kCutList], g[kCutList];
    uint64_t in[kCutList], all[kCutList];
    __device__ void put(int at, const CutNode &x)
    {
        l[at] = x.l;
        r[at] = x.r;
        g[at] = x.g;
        in[at] = x.in;
        all[at] = x.all;
    }
    __device__ CutNode get(int at) const { return CutNode{l[at], r[at], g[at], in[at], all[at]}; }
};

// Cuts the nodes of the lanes in `cuts`: x becomes the left child and y the
// right one, with the queries of the wave that pass them.
template <class Q>
__device__ __forceinline__ void cut_nodes(const Tree &tr, const Q &q, int from, uint64_t cuts, CutNode &x, CutNode &y)
{
    const int lane = threadIdx.x & 63;
    const int leaf0 = tr.leaf0();
    const bool mine = (cuts >> lane) & 1;
    float4 la{}, lb{}, ra{}, rb{};
    if (mine) {
        tr.load(x.g == x.l ? leaf0 + x.g : x.g, la, lb);
        tr.load(x.g + 1 == x.r ? leaf0 + x.r : x.g + 1, ra, rb);
    }
    const CutNode node = x;
    if (mine) {
        x = CutNode{node.l, node.g, tr.index(__float_as_int(la.w)), 0, 0};
        y = CutNode{node.g + 1, node.r, tr.index(__float_as_int(ra.w)), 0, 0};
    }
    for (uint64_t todo = cuts; todo; todo &= todo - 1) {
        const int s = __ffsll((unsigned long long)todo) - 1;
        const int l = __builtin_amdgcn_readlane(node.l, s), r = __builtin_amdgcn_readlane(node.r, s);
        const int g = __builtin_amdgcn_readlane(node.g, s);
        const uint64_t in = (uint64_t)readlane64((int64_t)node.in, s);
        const float4 a = readlane4(la, s), b = readlane4(lb, s), c = readlane4(ra, s), d = readlane4(rb, s);
        const uint64_t ml = ballot(q.test(a, b) && g >= from) & in;
        const uint64_t mr = ballot(q.test(c, d) && r >= from) & in;
        const uint64_t al = g - l >= kLeaves ? ballot(q.contains(a, b)) & ml : 0ull;
        const uint64_t ar = r - g > kLeaves ? ballot(q.contains(c, d)) & mr : 0ull;
        if (lane == s) {
            x.in = ml;
            x.all = al;
            y.in = mr;
            y.all = ar;
        }
    }
}

template <class Q>
__global__ __launch_bounds__(kCutBlock, 4) void k_cut(Tree tr, const float *__restrict__ queries, int m,
                                                      int packet_size, int least_width,
                                                      const int32_t *__restrict__ perm,
                                                      const int32_t *__restrict__ resume, QueryCtrl *ctrl,
                                                      HeavyPacket *__restrict__ heavy, uint32_t max_tasks,
                                                      Task *__restrict__ tasks, const Task *__restrict__ nodes)
{
    __shared__ CutList a, b;   // b: the parts of a's nodes, two places each
    __shared__ uint32_t s_sum[kCutWaves], s_first;
    __shared__ int s_cnt, s_level, s_longest[2];   // the longest range of a's nodes, by the level's parity
    __shared__ bool s_fits, s_more;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t n_heavy = ctrl->heavy;
    for (int64_t h = blockIdx.x; h < n_heavy; h += gridDim.x) {
        const uint64_t who = heavy[h].queries;
        const int number = heavy[h].packet;
        const int j = packet_query(number, packet_size, m, perm);
        Q q{};
        int from = 0;
        if (j >= 0 && ((who >> lane) & 1)) {
            q.load(queries, j);
            from = resume[j];
        }
        int cnt, most = kCutList;
        int64_t first;
        while (true) {
            int64_t width = least_width;
            auto wide = [&](const CutNode &x, int longest) {
                return (int64_t)x.r - x.l >= max(width, (int64_t)longest / kCutFirst);
            };
            // (no path has kPacketDepth nodes: that ends the loops on nodes that
            // are no tree, whose tasks' walks then report it)
            if (wv == 0) {
                int level = 0;
                bool more = true;
                cnt = most == kCutList ? heavy[h].nodes : 0;
                for (int k = lane; k < cnt; k += 64) {
                    const Task x = nodes[heavy[h].first_node + k];
                    a.put(k, CutNode{x.l, x.r, x.g, x.in, x.all});
                }
                if (cnt == 0) {
                    if (lane == 0) a.put(0, CutNode{0, tr.n - 1, tr.index(__float_as_int(tr.nodes[0].w)), who, 0});
                    cnt = 1;
                }
                for (; cnt > 0 && cnt <= min(kCutAlone, most / 4) && level < kPacketDepth; ++level) {
                    wave_sync();
                    CutNode x = a.get(lane < cnt ? lane : 0), y{};
                    wave_sync();
                    const uint64_t cuts = ballot(lane < cnt && wide(x, 0));
                    more = cuts != 0;
                    if (!more || __popcll(cuts) > kCutFew) break;
                    if (lane >= cnt) x.in = 0;
                    cut_nodes(tr, q, from, cuts, x, y);
                    const uint64_t mx = ballot(x.in != 0), my = ballot(y.in != 0);
                    const int at = (int)(lanes_below(mx) + lanes_below(my));
                    if (x.in) a.put(at, x);
                    if (y.in) a.put(at + (x.in ? 1 : 0), y);
                    cnt = __popcll(mx) + __popcll(my);
                }
                wave_sync();
                int longest = 0;
                for (int k = lane; k < cnt; k += 64) longest = max(longest, a.r[k] - a.l[k]);
                longest = wave_max(longest);
                if (lane == 0) {
                    s_cnt = cnt;
                    s_level = level;
                    s_more = more;
                    s_longest[level & 1] = longest;
                }
            }
            __syncthreads();
            cnt = s_cnt;
            for (int level = s_level; s_more && cnt > 0 && cnt <= most / 2 && level < kPacketDepth; ++level) {
                if (cnt > most / 4) width *= 4;
                const int e = lane * kCutWaves + wv;   // (neighbours, often cut together, in different waves)
                CutNode x{}, y{};
                if (e < cnt) x = a.get(e);
                const uint64_t cuts = ballot(e < cnt && wide(x, s_longest[level & 1]));
                if (tid == 0) s_longest[(level & 1) ^ 1] = 0;
                if (cuts) cut_nodes(tr, q, from, cuts, x, y);
                if (e < cnt) {
                    b.put(2 * e, x);
                    b.put(2 * e + 1, y);
                }
                const bool more = __syncthreads_or(cuts != 0);
                // the parts that have a query left, in order, back to a
                int out = 0;
                for (int c0 = 0; c0 < 2 * cnt; c0 += kCutBlock) {
                    const int k = c0 + tid;
                    const bool some = k < 2 * cnt && b.in[k] != 0;
                    const uint64_t mk = ballot(some);
                    if (lane == 0) s_sum[wv] = (uint32_t)__popcll(mk);
                    __syncthreads();
                    int at = out + (int)lanes_below(mk);
                    for (int w = 0; w < kCutWaves; ++w) {
                        if (w < wv) at += s_sum[w];
                        out += s_sum[w];
                    }
                    CutNode part{};
                    if (some) {
                        part = b.get(k);
                        a.put(at, part);
                    }
                    const int longest = wave_max(part.r - part.l);
                    if (lane == 0 && longest > 0) atomicMax(&s_longest[(level & 1) ^ 1], longest);
                    __syncthreads();
                }
                cnt = out;
                if (!more) break;
            }
            if (most == kOwnTasks) {
                first = (int64_t)max_tasks + h * kOwnTasks;
                break;
            }
            if (tid == 0) {
                s_first = 0u;
                s_fits = cnt == 0 || reserve_places(TaskCounter{ctrl}, (uint32_t)cnt, max_tasks, &s_first);
                if (!s_fits) ctrl->own = 1u;
            }
            __syncthreads();
            first = s_first;
            if (s_fits) break;
            most = kOwnTasks;
            __syncthreads();
        }
        for (int e = tid; e < cnt; e += kCutBlock)
            tasks[first + e] = Task{a.l[e], a.r[e], a.g[e], number, a.in[e], a.all[e]};
        if (tid == 0) {
            heavy[h].first = (int)first;
            heavy[h].tasks = cnt;
        }
        __syncthreads();
    }
}

// calls f(t, task) for every task, one wave per task
template <class F>
__device__ __forceinline__ void each_task(const QueryCtrl *ctrl, uint32_t max_tasks, const HeavyPacket *heavy,
                                          const Task *tasks, F &&f)
{
    const int64_t T = places_given(ctrl->tasks, ctrl->tasks_end, max_tasks);
    const int64_t own = ctrl->own ? (int64_t)ctrl->heavy * kOwnTasks : 0;
    for (int64_t k = blockIdx.x; k < T + own; k += gridDim.x) {
        int64_t t = k;
        if (k >= T) {
            t = (int64_t)max_tasks + (k - T);
            const HeavyPacket h = heavy[(k - T) / kOwnTasks];
            if ((uint32_t)h.first < max_tasks || (int)((k - T) % kOwnTasks) >= h.tasks) continue;
        }
        f(t, tasks[t]);
    }
}

// Hits of every task, per query of its packet: one wave per task.
template <class Q>
__global__ __launch_bounds__(kWalkBlock) void k_task_count(Tree tr, const float *__restrict__ queries, int m,
                                                           int packet_size, const int32_t *__restrict__ perm,
                                                           const int32_t *__restrict__ resume,
                                                           const QueryCtrl *ctrl, uint32_t max_tasks,
                                                           const HeavyPacket *__restrict__ heavy,
                                                           const Task *__restrict__ tasks,
                                                           int32_t *__restrict__ rows)
{
    __shared__ PacketLds<Q> lds;
    const int lane = threadIdx.x;
    each_task(ctrl, max_tasks, heavy, tasks, [&](int64_t t, const Task &x) {
        const int j = packet_query(x.packet, packet_size, m, perm);
        const bool mine = j >= 0 && ((x.in >> lane) & 1);   // every lane of x.in has a query
        Q q{};
        if (mine) q.load(queries, j);
        const PacketRun run{x.l, x.r, x.g, x.in, x.all, mine ? resume[j] : 0, nullptr, 0u, 0};
        uint64_t left;
        int rest;
        const int c = packet<Q, false>(tr, run, q, mine, mine, lds, nullptr, 0, 0, left, rest);
        if (lane < packet_size) rows[t * packet_size + lane] = mine ? c : 0;
    });
}

// Each task's place among its queries' hits (in place of the hits), and the
// queries' totals: one wave per heavy packet.
__global__ __launch_bounds__(kBlock) void k_task_places(const QueryCtrl *ctrl, int m,
                                                   int packet_size, const int32_t *__restrict__ perm,
                                                   const HeavyPacket *__restrict__ heavy,
                                                   const int32_t *__restrict__ light,
                                                   int32_t *__restrict__ rows, int32_t *__restrict__ places,
                                                   int32_t *__restrict__ counts)
{
    const int lane = threadIdx.x & 63;
    const int64_t n_heavy = ctrl->heavy;
    for (int64_t h = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6); h < n_heavy;
         h += (int64_t)gridDim.x * kWavesPerBlock) {
        const HeavyPacket x = heavy[h];
        const int j = packet_query(x.packet, packet_size, m, perm);
        const int64_t first = x.first;
        if (j < 0) continue;
        int run = light[j];
        constexpr int kAhead = 16;
        for (int k0 = 0; k0 < x.tasks; k0 += kAhead) {
            int32_t c[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                c[u] = k0 + u < x.tasks ? rows[(first + k0 + u) * packet_size + lane] : 0;
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                if (k0 + u < x.tasks) places[(first + k0 + u) * packet_size + lane] = run;
                run += c[u];
            }
        }
        counts[j] = run;
    }
}

// ------------------------------------------------------------------- fill

// The light walks' hits: a query with at most kHitCache of them has them in
// the cache, from where 16 lanes copy each row; the others walk again.
template <class Q>
__global__ __launch_bounds__(kWalkBlock) void k_fill_light(Tree tr, const float *__restrict__ queries, int m,
                                                           int packet_size, const int32_t *__restrict__ perm,
                                                           const QueryCtrl *ctrl,
                                                           const int32_t *__restrict__ light,
                                                           const int64_t *__restrict__ offsets,
                                                           const int32_t *__restrict__ cache,
                                                           int32_t *__restrict__ out)
{
    static_assert(kHitCache % 16 == 0, "whole rows of 16 lanes");
    __shared__ PacketLds<Q> lds;
    const int lane = threadIdx.x;
    const int j = packet_query(packet_of(blockIdx.x, gridDim.x), packet_size, m, ctrl->ordered ? perm : nullptr);
    const bool valid = j >= 0;
    const int c = valid ? light[j] : 0;
    const int64_t pos = c > 0 ? offsets[j] : 0;
    uint64_t rows = ballot(c > 0 && c <= kHitCache);
    while (rows) {
        constexpr int kRows = 2;   // rows per lane group and step
        int32_t v[kRows][kHitCache / 16];
        int n[kRows];
        int64_t p[kRows];
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            int src = 0;
            bool some = false;
#pragma unroll
            for (int g = 0; g < 4; ++g) {   // four rows, one per 16 lanes
                if (rows && (lane >> 4) == g) {
                    src = __ffsll((unsigned long long)rows) - 1;
                    some = true;
                }
                rows &= rows - 1;
            }
            const int row = __shfl(j, src);
            n[u] = __shfl(c, src);
            if (!some) n[u] = 0;
            p[u] = (int64_t)shfl64((uint64_t)pos, src);
#pragma unroll
            for (int w = 0; w < kHitCache / 16; ++w) {
                const int k = (lane & 15) + 16 * w;
                if (k < n[u]) v[u][w] = cache[(int64_t)row * kHitCache + k];
            }
        }
#pragma unroll
        for (int u = 0; u < kRows; ++u)
#pragma unroll
            for (int w = 0; w < kHitCache / 16; ++w) {
                const int k = (lane & 15) + 16 * w;
                if (k < n[u]) out[p[u] + k] = v[u][w];
            }
    }
    const bool again = c > kHitCache;
    if (ballot(again)) {
        Q q{};
        if (valid) q.load(queries, j);
        int rest;
        uint64_t left;
        PacketRun run{};
        run.l = -1;
        packet<Q, true>(tr, run, q, valid, again, lds, out, pos, c, left, rest);
    }
}

// The tasks' hits: walked again, each query's from its place on.
template <class Q>
__global__ __launch_bounds__(kWalkBlock) void k_fill_tasks(Tree tr, const float *__restrict__ queries, int m,
                                                           int packet_size, const int32_t *__restrict__ perm,
                                                           const int32_t *__restrict__ resume,
                                                           const QueryCtrl *ctrl, uint32_t max_tasks,
                                                           const HeavyPacket *__restrict__ heavy,
                                                           const Task *__restrict__ tasks,
                                                           const int32_t *__restrict__ rows,
                                                           const int32_t *__restrict__ places,
                                                           const int64_t *__restrict__ offsets,
                                                           int32_t *__restrict__ out)
{
    __shared__ PacketLds<Q> lds;
    const int lane = threadIdx.x;
    const int32_t *order = ctrl->ordered ? perm : nullptr;
    each_task(ctrl, max_tasks, heavy, tasks, [&](int64_t t, const Task &x) {
        const int j = packet_query(x.packet, packet_size, m, order);
        const bool whole = j >= 0 && ((x.in >> lane) & 1);
        int c = 0;
        int64_t pos = 0;
        if (whole) {
            c = rows[t * packet_size + lane];
            pos = offsets[j] + places[t * packet_size + lane];
        }
        const bool mine = c > 0;
        PacketRun run{x.l, x.r, x.g, x.in, x.all, mine ? resume[j] : 0, nullptr, 0u, 0};
        run.in &= ballot(mine);
        run.all &= run.in;
        if (run.in == 0) return;
        Q q{};
        if (whole) q.load(queries, j);
        uint64_t left;
        int rest;
        packet<Q, true>(tr, run, q, whole, mine, lds, out, pos, c, left, rest);
    });
}

}  // namespace
}  // namespace lbvh
