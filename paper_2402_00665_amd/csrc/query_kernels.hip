// Range queries on gfx950 (Alg. 1) and their CSR output.
//
// Alg. 1 walks the tree in preorder from the root: a node whose box passes
// the test sends the walk to its left child (internal node) or reports the
// primitive (leaf) and follows the rope; a node that fails sends it along
// the rope; the sentinel -1 ends it.  Its hits are the leaves whose boxes
// pass, in index order: both tests are monotone under box inclusion, so every
// ancestor of a passing leaf passes.  The kernels here report the same hits in
// the same order with the nodes visited by whole waves:
//
// * The queries are walked in packets of up to 64 by one wave each, in Morton
//   order of their centres when there are many (packet_size).
// * The rest of a packet that turns out heavy while few other waves are still
//   busy is cut into tasks, subtrees that other waves walk (one box query can
//   hit 10^5 primitives; alone it would be the critical path).
// * The count call keeps each query's first hits, and the places of the tasks'
//   hits; the fill call copies the kept ones and walks again only where a
//   query had more.
// No contraction: the sphere test is evaluated exactly as written.
#pragma clang fp contract(off)

#include <type_traits>

#include "query_walk.hpp"
#include "radix_sort.hpp"

namespace lbvh {
namespace {

// ------------------------------------------------------------ query order
//
// From kQOrderMin queries on (and with the "query_order" knob set) the count
// call first sorts the queries' numbers by a 16-bit Morton key of their centres
// (quantised in the root's box, clamped to it), so that the queries of a
// packet walk the same part of the tree.  Only the schedule changes: counts
// and hits are kept per caller's query.

// keys of the queries, their digit histograms (LDS, then one global add
// per digit and block), and the first sort pass's cleared look-back status
template <class Q>
__global__ __launch_bounds__(kBlock) void k_qorder_keys(Tree tr, const float *__restrict__ queries,
                                                   int m, uint32_t *__restrict__ keys,
                                                   uint32_t *hist, uint32_t *__restrict__ status0,
                                                   int64_t status_words)
{
    __shared__ uint32_t lh[kQOrderPasses * kRadix];
    for (int j = threadIdx.x; j < kQOrderPasses * kRadix; j += kBlock) lh[j] = 0u;
    const int64_t gid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t j = gid; j < status_words; j += stride) status0[j] = 0u;
    __syncthreads();
    float4 a, b;
    tr.load(0, a, b);   // the root's box (leaf 0's when n = 1)
    const float rlo[3] = {a.x, a.y, a.z}, rhi[3] = {b.x, b.y, b.z};
    float scale[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float ext = rhi[k] - rlo[k];
        scale[k] = ext > 0.0f ? 1024.0f / ext : 0.0f;
    }
    for (int64_t i = gid; i < m; i += stride) {
        Q q;
        q.load(queries, (int)i);
        float lo[3], hi[3];
        q.bounds(lo, hi);
        uint32_t c[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float t = ((lo[k] + hi[k]) * 0.5f - rlo[k]) * scale[k];
            c[k] = (uint32_t)fminf(fmaxf(t, 0.0f), 1023.0f);   // NaN -> 0
        }
        const uint32_t key = Code<uint32_t>::make(c[0], c[1], c[2]) >> 14;
        keys[i] = key;
        atomicAdd(&lh[key & (kRadix - 1)], 1u);
        atomicAdd(&lh[kRadix + (key >> kRadixBits)], 1u);
    }
    __syncthreads();
    for (int j = threadIdx.x; j < kQOrderPasses * kRadix; j += kBlock)
        if (lh[j]) atomicAdd(&hist[j], lh[j]);
}

// start of a count call: its control words, the scan's status words and
// (when reordering) the sort's histograms
__global__ __launch_bounds__(kBlock) void k_query_reset(QueryCtrl *ctrl, int ordered, uint64_t *scan_status,
                                                        int64_t scan_words, uint32_t *hist)
{
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) {
            QueryCtrl zero{};
            zero.ordered = ordered;
            *ctrl = zero;
        }
        if (ordered)
            for (int j = threadIdx.x; j < kQOrderPasses * kRadix; j += kBlock) hist[j] = 0u;
    }
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < scan_words; j += (int64_t)gridDim.x * kBlock)
        scan_status[j] = 0ull;
}

// ---------------------------------------------------------- first hit
//
// First hit of each ray: among the primitives it meets, the one with the
// smallest entry parameter, ties to the smallest leaf position (Morton
// order).  One lane per ray goes down from the root, the nearer child first,
// so that a close hit is found early and prunes what is behind it.  A node
// with the leaf range [l, r] and the split g has the children g and g + 1
// (leaves where the range ends there), so one step loads and tests both:
// usually neighbouring records.  The farther child waits on a stack.  A node
// is entered only if it can hold a better hit: an entry below the best one,
// or an equal one and leaves before the best hit's (a box inside a node's
// box never has a smaller entry parameter: the slab test is monotone under
// box inclusion).  The best hit is unique, so the order of the visits does
// not show.  An n = 0 tree gives every ray hit -1 and t = +inf (n = 0 never
// reaches here: the caller fills those).
//
// Bound by the latency of its scattered loads and then by its vector
// instructions, so what counts is waves per CU: the first kRayStack stack
// entries lie in LDS and the rest, rarely reached, in the call's workspace
// (2^20 rays on 2^24 clustered boxes: 0.96 ms with 6 entries in LDS, 1.04
// with 8, 1.00 with 10).  A wave owns `share` rays; once kRayRefill lanes
// have ended their rays, those lanes write their results and take the next
// rays together (1.02 ms for 2^20 rays without refills; writing each result
// as its ray ends, 1.00 instead of 0.92).  An entry on the stack carries its
// split, or its first step would load it (10^5 rays on 10^6 boxes 191 -> 163
// us).  Few rays are spread, down to one a wave: a wave takes the steps of
// its slowest ray and both sides of every branch (97 rays on 423177 boxes
// 136 -> 59 us).  One walk in preorder along the ropes per ray took 11.3 ms:
// it visits the children in index order, so most of what it visits lies
// behind the hit.
constexpr int kRayRefill = 16;

struct FirstHit {
    float best;
    int pos;   // leaf position of the best hit (kNoHit: none)
    // e of a box that was met is not NaN; no short circuit, so no branches
    __device__ bool better(float e, int l) const { return (e < best) | ((e == best) & (l < pos)); }
};
constexpr int kNoHit = 0x7fffffff;

__global__ __launch_bounds__(kRayBlock) void k_ray_first(Tree tr, const float *__restrict__ rays, int m,
                                                         int share, int32_t *__restrict__ hit,
                                                         float *__restrict__ t, int2 *__restrict__ deep)
{
    __shared__ int2 s_stack[kRayStack][kRayBlock];    // node, other end of its range
    __shared__ float s_enter[kRayStack][kRayBlock];   // its entry parameter
    __shared__ int s_split[kRayStack][kRayBlock];     // its split
    const int leaf0 = tr.leaf0(), tid = threadIdx.x;
    const int lanes = share < kRayBlock ? share : kRayBlock;   // that ever hold a ray
    const int64_t stride = (int64_t)gridDim.x * lanes;
    deep += (int64_t)blockIdx.x * lanes + tid;
    auto split_of = [&](int c) { return c >= leaf0 ? c - leaf0 : c; };
    float4 root_a, root_b;
    tr.load(0, root_a, root_b);
    const int root_g = split_of(__float_as_int(root_a.w));
    // this wave's rays not taken yet
    int64_t next = (int64_t)blockIdx.x * share;
    const int64_t end = next + share < m ? next + share : m;
    int j = -1, l = 0, r = 0, g = 0, sp = 0;
    int64_t budget = 0;
    FastRay q{};
    bool fast = true;
    FirstHit f{INFINITY, kNoHit};
    bool live = false;
    while (true) {
        const uint64_t idle = __ballot(!live);
        if (idle == ~0ull || (next < end && __popcll(idle) >= kRayRefill)) {
            // the rays that ended since: their results
            if (!live && j >= 0) {
                int prim = -1;
                float best = INFINITY;
                if (f.pos != kNoHit) {   // the entry parameter exactly as the test defines it
                    Ray x;
                    x.load(rays, j);
                    float4 a, b;
                    tr.load(leaf0 + f.pos, a, b);
                    x.enter(a, b, &best);
                    prim = __float_as_int(a.w);
                }
                hit[j] = prim;
                t[j] = best;
                j = -1;
            }
            if (next >= end) break;   // every lane is idle
            const int64_t mine = next + lanes_below(idle);
            next += __popcll(idle);
            if (!live && mine < end) {
                Ray x;
                x.load(rays, (int)mine);
                q = FastRay(x);
                fast = x.plain();
                f = FirstHit{INFINITY, kNoHit};
                budget = tr.walk_budget();
                sp = 0;
                l = 0;
                r = tr.n - 1;
                g = root_g;
                float e;
                const bool met = x.enter(root_a, root_b, &e);
                if (met && leaf0 > 0) {
                    j = (int)mine;
                    live = true;
                } else {
                    hit[mine] = met ? __float_as_int(root_a.w) : -1;
                    t[mine] = met ? e : INFINITY;
                }
            }
            continue;
        }
        if (live) {
            const bool lleaf = g == l, rleaf = g + 1 == r;
            float4 la, lb, ra, rb;
            tr.load(lleaf ? leaf0 + g : g, la, lb);
            tr.load(rleaf ? leaf0 + r : g + 1, ra, rb);
            float el, er;
            bool hl, hr;
            if (__ballot(!fast) == 0) {
                hl = q.enter(la, lb, &el);
                hr = q.enter(ra, rb, &er);
            } else {
                Ray x;
                x.load(rays, j);
                hl = x.enter(la, lb, &el);
                hr = x.enter(ra, rb, &er);
            }
            auto take = [&](bool now, float e, int leaf) {
                f.best = now ? e : f.best;
                f.pos = now ? leaf : f.pos;
            };
            hl = hl & f.better(el, l);
            take(hl & lleaf, el, l);
            hr = hr & f.better(er, g + 1);
            take(hr & rleaf, er, r);
            hl = hl & !lleaf & f.better(el, l);
            hr = hr & !rleaf;
            const int gl = split_of(__float_as_int(la.w)), gr = split_of(__float_as_int(ra.w));
            const bool lnear = hl && (!hr || el <= er);
            if (hl && hr) {
                const int2 far = lnear ? make_int2(g + 1, r) : make_int2(g, l);
                const float fe = lnear ? er : el;
                if (sp < kRayStack) {
                    s_stack[sp][tid] = far;
                    s_enter[sp][tid] = fe;
                    s_split[sp][tid] = lnear ? gr : gl;
                } else {
                    deep[(sp - kRayStack) * stride] = far;
                }
                ++sp;
            }
            bool go = hl || hr;
            l = lnear ? l : g + 1;
            r = lnear ? g : r;
            g = lnear ? gl : gr;
            if (!go) {
                int2 s = make_int2(0, 0);
                while (!go && sp > 0) {
                    --sp;
                    float e;
                    if (sp < kRayStack) {
                        s = s_stack[sp][tid];
                        e = s_enter[sp][tid];
                        g = s_split[sp][tid];
                    } else {   // its entry parameter and split are found again
                        s = deep[(sp - kRayStack) * stride];
                        Ray x;
                        x.load(rays, j);
                        float4 a, b;
                        tr.load(s.x, a, b);
                        x.enter(a, b, &e);
                        g = split_of(__float_as_int(a.w));
                    }
                    l = s.x < s.y ? s.x : s.y;
                    go = f.better(e, l);
                }
                r = s.x < s.y ? s.y : s.x;
            }
            if ((--budget < 0 || sp >= kRayDepth) && go) {   // (also where the nodes are no tree)
                tr.budget_spent();
                go = false;
            }
            live = go;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_ray_none(int64_t m, int32_t *__restrict__ hit,
                                                     float *__restrict__ t, uint32_t *err)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    const int64_t j0 = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j0 == 0) *err = 0u;
    for (int64_t j = j0; j < m; j += stride) {
        hit[j] = -1;
        t[j] = INFINITY;
    }
}

struct Scratch {
    QueryCtrl *ctrl;
    int32_t *light, *counts, *cache, *resume, *rows, *places, *perm, *qvals;
    int64_t *offsets;
    HeavyPacket *heavy;
    Task *tasks, *nodes;
    uint64_t *scan_status;
    uint32_t *qkeys[2], *qstatus[2], *qhist;
};

Scratch carve(char *ws, const QueryLayout &L)
{
    Scratch S;
    auto at = [&](auto *&p, size_t off) { p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(ws + off); };
    at(S.ctrl, L.ctrl);
    at(S.light, L.light);
    at(S.counts, L.counts);
    at(S.offsets, L.offsets);
    at(S.cache, L.cache);
    at(S.resume, L.resume);
    at(S.heavy, L.heavy);
    at(S.tasks, L.tasks);
    at(S.rows, L.rows);
    at(S.nodes, L.rows);
    at(S.places, L.places);
    at(S.scan_status, L.scan_status);
    at(S.perm, L.perm);
    for (int k = 0; k < 2; ++k) {
        at(S.qkeys[k], L.qkeys[k]);
        at(S.qstatus[k], L.qstatus[k]);
    }
    at(S.qvals, L.qvals);
    at(S.qhist, L.qhist);
    return S;
}

unsigned grid_for(int64_t items, int64_t most)
{
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((items + kBlock - 1) / kBlock, most));
}

// Queries in key order: keys, then two stable 8-bit passes.  From 2^18
// queries on in tiles of 1024 x 8, whose passes look back over a quarter of
// the tiles (a pass over 2^20 keys 26.2 -> 18.5 us); below, 512 x 4 makes
// enough blocks.
constexpr int64_t kQOrderLarge = 1 << 18;
constexpr int kSmallTree = 1 << 18;
constexpr int kMidTree = 1 << 21;

template <class Q, int T, int I>
void sort_keys(const Tree &tr, const float *q, int m, unsigned key_blocks, const Scratch &S, hipStream_t s)
{
    const unsigned tiles = (unsigned)(((int64_t)m + T * I - 1) / (T * I));
    hipLaunchKernelGGL((k_qorder_keys<Q>), dim3(key_blocks), dim3(kBlock), 0, s, tr, q, m, S.qkeys[0], S.qhist,
                       S.qstatus[0], (int64_t)tiles * kRadix);
    const SortSegs one{nullptr, nullptr, 1, 0};
    hipLaunchKernelGGL((k_onesweep<uint32_t, T, I, kRadixBits, true>), dim3(tiles), dim3(T), 0, s, S.qkeys[0],
                       S.qkeys[1], nullptr, S.qvals, (int64_t)m, one, 0, kRadixBits, S.qhist, S.qstatus[0],
                       S.qstatus[1], tiles, S.ctrl->sort_tile, tr.err, (const uint32_t *)nullptr);
    hipLaunchKernelGGL((k_onesweep<uint32_t, T, I, kRadixBits, true>), dim3(tiles), dim3(T), 0, s, S.qkeys[1],
                       S.qkeys[0], S.qvals, S.perm, (int64_t)m, one, kRadixBits, kRadixBits, S.qhist + kRadix,
                       S.qstatus[1], nullptr, 0u, S.ctrl->sort_tile + 1, tr.err, (const uint32_t *)nullptr);
}

template <class Q>
hipError_t run_count(Tree tr, const float *q, int m, int64_t *offsets, char *ws,
                     const QueryLayout &L, hipStream_t s)
{
    const Scratch S = carve(ws, L);
    tr.err = &S.ctrl->error;
    tr.budget = tune_get(TUNE_QBUDGET);
    const bool order = m > 1 && (tune_get(TUNE_QORDER) != 0 || L.packet > 1);
    prof_begin(K_QSPLIT, s);
    hipLaunchKernelGGL(k_query_reset, dim3(grid_for(scan_tiles(m), kQueryGridMax)), dim3(kBlock), 0, s, S.ctrl,
                       order ? 1 : 0, S.scan_status, scan_tiles(m), S.qhist);
    prof_end(K_QSPLIT, s);
    if (order) {
        // sort the queries' numbers by key (two stable 8-bit passes)
        prof_begin(K_QORDER, s);
        // few blocks, so that few global histogram adds meet on each word
        const unsigned gk = (unsigned)std::min<int64_t>(kQOrderKeyBlocks, (m + 16 * kBlock - 1) / (16 * kBlock));
        if (m < kQOrderLarge)
            sort_keys<Q, 512, kQOrderTile / 512>(tr, q, m, gk, S, s);
        else
            sort_keys<Q, 1024, 8>(tr, q, m, gk, S, s);
        prof_end(K_QORDER, s);
    }
    prof_begin(K_QCOUNT, s);
    const int32_t *perm = order ? S.perm : nullptr;
    const int size = L.packet;
    // steps a packet walks before it may leave its rest to others (48; 32 cuts
    // up too many short walks: a request of 10^4 queries 285 instead of 278 us,
    // 64 leaves 200 heavy spheres at 148 instead of 117 us), and leaves of a
    // task: wide enough that a packet of 64 makes few thousand of them, narrow
    // for packets of few queries, whose tasks are cheap
    // (twice as many where the queries fill the machine on a tree of less than
    // 2^18 primitives, whose long walks end soon by themselves: 909012 spheres
    // on 141193 boxes 258 -> 231 us, but boxes on 400000 228 -> 299)
    const int patience = (L.packets > kDrainWaves && tr.n < kSmallTree ? 6 : 3)
                         << std::min<int64_t>(std::max<int64_t>(0, tune_get(TUNE_QSPLIT2) - 3), 16);
    // (a quarter of that on trees below 2^21 primitives, which cannot fill the
    // pool: 900000 boxes on 300000 363 -> 315 us, but 2^20 on 2^24 770 -> 852)
    const int wider = tune_get(TUNE_QLEAF) == 1 ? 4 : 1;
    const int64_t spread = std::max<int64_t>(0, tune_get(TUNE_QSPLIT1) - (tr.n < kMidTree ? 9 : 7));
    const int width = wider * (int)std::max<int64_t>(512, (int64_t)size << spread);
    hipLaunchKernelGGL((k_walk<Q>), dim3((unsigned)L.packets), dim3(kWalkBlock), 0, s, tr, q, m, size, patience,
                       perm, S.ctrl, S.light, S.counts, S.cache, S.resume, S.heavy, S.nodes, L.max_nodes);
    prof_end(K_QCOUNT, s);
    prof_begin(K_QSPLIT, s);
    hipLaunchKernelGGL((k_cut<Q>), dim3((unsigned)std::min<int64_t>(L.packets, kCutGrid)), dim3(kCutBlock), 0, s, tr,
                       q, m, size, width, perm, S.resume, S.ctrl, S.heavy, L.max_tasks, S.tasks, S.nodes);
    prof_end(K_QSPLIT, s);
    prof_begin(K_QCOUNT, s);
    const unsigned gt = (unsigned)std::min<int64_t>((int64_t)L.max_tasks, kTaskGrid);
    hipLaunchKernelGGL((k_task_count<Q>), dim3(gt), dim3(kWalkBlock), 0, s, tr, q, m, size, perm, S.resume, S.ctrl,
                       L.max_tasks, S.heavy, S.tasks, S.rows);
    prof_end(K_QCOUNT, s);
    prof_begin(K_SCAN, s);
    hipLaunchKernelGGL(k_task_places, dim3(grid_for(64 * L.packets, kCutGrid)), dim3(kBlock), 0, s, S.ctrl,
                       m, size, perm, S.heavy, S.light, S.rows, S.places, S.counts);
    scan(S.counts, m, S.scan_status, &S.ctrl->scan_tile, offsets, S.offsets, tr.err, s);
    prof_end(K_SCAN, s);
    return hipGetLastError();
}

template <class Q>
hipError_t run_fill(const Tree &tr, const float *q, int m, int32_t *indices, char *ws, const QueryLayout &L,
                    hipStream_t s)
{
    const Scratch S = carve(ws, L);
    prof_begin(K_QFILL, s);
    hipLaunchKernelGGL((k_fill_light<Q>), dim3((unsigned)L.packets), dim3(kWalkBlock), 0, s, tr, q, m, L.packet,
                       S.perm, S.ctrl, S.light, S.offsets, S.cache, indices);
    hipLaunchKernelGGL((k_fill_tasks<Q>), dim3((unsigned)std::min<int64_t>((int64_t)L.max_tasks, kTaskGrid)),
                       dim3(kWalkBlock), 0, s, tr, q, m, L.packet, S.perm, S.resume, S.ctrl, L.max_tasks, S.heavy, S.tasks,
                       S.rows, S.places, S.offsets, indices);
    prof_end(K_QFILL, s);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_query(int qkind, int kind, const lbvh_node *nodes, const int32_t *leaf_perm, int n,
                        const float *q, int m, int64_t *offsets, int32_t *indices, bool fill,
                        char *ws, const QueryLayout &L, hipStream_t s)
{
    if (n == 0 || m == 0) {
        if (fill) return hipSuccess;
        const int64_t cnt = (int64_t)m + 1;
        hipLaunchKernelGGL(k_zero_i64, dim3((unsigned)((cnt + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                           s, offsets, cnt, reinterpret_cast<uint32_t *>(ws + L.ctrl + kQueryErrorByte));
        return hipGetLastError();
    }
    Tree tr{reinterpret_cast<const float4 *>(nodes), leaf_perm, n};
    tr.points = kind == LBVH_POINTS;
    if (fill) {
        if (qkind == 2) return run_fill<Ray>(tr, q, m, indices, ws, L, s);
        return qkind == 0 ? run_fill<Sphere>(tr, q, m, indices, ws, L, s)
                          : run_fill<QBox>(tr, q, m, indices, ws, L, s);
    }
    if (qkind == 2) return run_count<Ray>(tr, q, m, offsets, ws, L, s);
    return qkind == 0 ? run_count<Sphere>(tr, q, m, offsets, ws, L, s)
                      : run_count<QBox>(tr, q, m, offsets, ws, L, s);
}

hipError_t launch_ray_none(int64_t m, int32_t *hit, float *t, char *ws, const QueryLayout &L,
                           hipStream_t s)
{
    const Scratch S = carve(ws, L);
    hipLaunchKernelGGL(k_ray_none, dim3(grid_for(m, kQueryGridMax)), dim3(kBlock), 0, s, m, hit, t,
                       &S.ctrl->error);
    return hipGetLastError();
}

hipError_t launch_ray_first(const lbvh_node *nodes, int n, const float *rays, int m, int32_t *hit,
                            float *t, char *ws, const QueryLayout &L, hipStream_t s)
{
    if (m == 0) return hipSuccess;
    const Scratch S = carve(ws, L);
    Tree tr{reinterpret_cast<const float4 *>(nodes), nullptr, n, &S.ctrl->error, tune_get(TUNE_QBUDGET)};
    prof_begin(K_QCOUNT, s);
    hipLaunchKernelGGL(k_zero_i64, dim3(1), dim3(kBlock), 0, s, (int64_t *)nullptr, (int64_t)0, &S.ctrl->error);
    const int share = ray_share(m);
    const int64_t waves = ((int64_t)m + share - 1) / share;
    hipLaunchKernelGGL(k_ray_first, dim3((unsigned)waves), dim3(kRayBlock), 0, s, tr, rays, m, share, hit,
                       t, reinterpret_cast<int2 *>(ws + L.deep));
    prof_end(K_QCOUNT, s);
    return hipGetLastError();
}

}  // namespace lbvh
