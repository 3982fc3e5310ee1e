// Query-side device code shared by the single-tree and batched query
// translation units: the predicates (with their containment tests), the tree,
// the staged output of the batched fill and the CSR scan.
#pragma once
#pragma clang fp contract(off)

#include "device_common.hpp"

namespace lbvh {
namespace {

struct PlainSphere;
struct PointSphere;

struct Sphere {
    static constexpr int kFloats = 4;   // x, y, z, r
    using Plain = PlainSphere;
    using PlainPoint = PointSphere;
    __device__ bool plain() const { return cx == cx && cy == cy && cz == cz; }
    __device__ bool leaf(float4 lo, float4 hi) const { return test(lo, hi); }
    float cx, cy, cz, r, r2;
    __device__ void load(const float *q, int j)
    {
        const float4 v = reinterpret_cast<const float4 *>(q)[j];
        cx = v.x; cy = v.y; cz = v.z; r = v.w; r2 = v.w * v.w;
    }
    // a box around the query (only steers the schedule, never a result)
    __device__ void bounds(float lo[3], float hi[3]) const
    {
        lo[0] = cx - r; lo[1] = cy - r; lo[2] = cz - r;
        hi[0] = cx + r; hi[1] = cy + r; hi[2] = cz + r;
    }
    __device__ bool test(float4 lo, float4 hi) const
    {
        const float dx = fmaxf(fmaxf(lo.x - cx, cx - hi.x), 0.0f);
        const float dy = fmaxf(fmaxf(lo.y - cy, cy - hi.y), 0.0f);
        const float dz = fmaxf(fmaxf(lo.z - cz, cz - hi.z), 0.0f);
        return (dx * dx + dy * dy) + dz * dz <= r2;
    }
    // The box lies inside the ball: its farthest corner passes.  Every box
    // inside it then passes `test` too, also after rounding: each per-axis
    // term of `test` for an inner box is <= the corresponding far term here
    // (rounding is monotone), and squares and sums of non-negative terms
    // keep the order.
    __device__ bool contains(float4 lo, float4 hi) const
    {
        const float fx = fmaxf(cx - lo.x, hi.x - cx);
        const float fy = fmaxf(cy - lo.y, hi.y - cy);
        const float fz = fmaxf(cz - lo.z, hi.z - cz);
        return (fx * fx + fy * fy) + fz * fz <= r2;
    }
};

// Sphere::test with what it needs of the query alone
struct PlainSphere {
    float cx, cy, cz, r2;
    PlainSphere() = default;
    __device__ explicit PlainSphere(const Sphere &q) : cx(q.cx), cy(q.cy), cz(q.cz), r2(q.r2) {}
    __device__ bool test(float4 lo, float4 hi) const
    {
        const float dx = fmaxf(fmaxf(lo.x - cx, cx - hi.x), 0.0f);
        const float dy = fmaxf(fmaxf(lo.y - cy, cy - hi.y), 0.0f);
        const float dz = fmaxf(fmaxf(lo.z - cz, cz - hi.z), 0.0f);
        return (dx * dx + dy * dy) + dz * dz <= r2;
    }
    __device__ bool leaf(float4 lo, float4 hi) const { return test(lo, hi); }
};

// ... and, on a leaf of a tree of points (lo == hi): the larger of lo - c
// and c - lo is their magnitude, whose square is the same.  (For a centre
// without NaN; the maximum with zero would drop one.)
struct PointSphere : PlainSphere {
    using PlainSphere::PlainSphere;
    __device__ bool leaf(float4 lo, float4) const
    {
        const float dx = lo.x - cx, dy = lo.y - cy, dz = lo.z - cz;
        return (dx * dx + dy * dy) + dz * dz <= r2;
    }
};

struct QBox {
    static constexpr int kFloats = 6;   // lo.xyz, hi.xyz
    using Plain = QBox;
    using PlainPoint = QBox;
    __device__ bool leaf(float4 lo, float4 hi) const { return test(lo, hi); }
    __device__ bool plain() const { return true; }
    float lx, ly, lz, hx, hy, hz;
    __device__ void load(const float *q, int j)
    {
        const float2 *p = reinterpret_cast<const float2 *>(q + 6 * (int64_t)j);
        const float2 a = p[0], b = p[1], c = p[2];
        lx = a.x; ly = a.y; lz = b.x; hx = b.y; hy = c.x; hz = c.y;
    }
    __device__ bool test(float4 lo, float4 hi) const
    {
        return lx <= hi.x && lo.x <= hx && ly <= hi.y && lo.y <= hy && lz <= hi.z && lo.z <= hz;
    }
    __device__ void bounds(float lo[3], float hi[3]) const
    {
        lo[0] = lx; lo[1] = ly; lo[2] = lz;
        hi[0] = hx; hi[1] = hy; hi[2] = hz;
    }
    // The box lies inside the query box, so every box inside it overlaps.
    __device__ bool contains(float4 lo, float4 hi) const
    {
        return lx <= lo.x && hi.x <= hx && ly <= lo.y && hi.y <= hy && lz <= lo.z && hi.z <= hz;
    }
};

// Ray or segment: the points o + t*d with tmin <= t <= tmax (a segment from
// a to b is o = a, d = b - a, [0, 1]; a ray has tmax = +inf).  Sec. 1 counts
// the primitives a ray meets among the range searches a BVH answers.  Closed
// slab test in binary32: per axis, inv = 1/d correctly rounded; an axis with
// d = 0, or whose reciprocal overflows, passes iff o lies in the slab
// [lo, hi]; otherwise its parameter interval has the ends (lo - o)*inv and
// (hi - o)*inv.  enter = the largest of tmin and the intervals' lower ends,
// exit = the smallest of tmax and their upper ends; hit iff enter <= exit.
// Each step is a monotone function of lo (non-increasing) and hi
// (non-decreasing), also after rounding, so a box inside a passing box can
// only fail or pass with an entry parameter at least as large: Alg. 1's
// pruning is exact, and so is the first-hit walk's pruning on the entry.
struct FastRay;

struct Ray {
    static constexpr int kFloats = 8;   // o.xyz, tmin, d.xyz, tmax
    using Plain = FastRay;
    using PlainPoint = FastRay;
    __device__ bool leaf(float4 lo, float4 hi) const { return test(lo, hi); }
    float o[3], d[3], inv[3], tmin, tmax;
    bool par[3];
    // every value that the test takes is ordinary (FastRay's condition)
    __device__ bool plain() const
    {
        bool ok = tmin == tmin && tmax == tmax;
#pragma unroll
        for (int k = 0; k < 3; ++k) ok = ok && !par[k] && fabsf(o[k]) < INFINITY && fabsf(d[k]) < INFINITY;
        return ok;
    }
    __device__ void load(const float *q, int j)
    {
        const float4 *p = reinterpret_cast<const float4 *>(q) + 2 * (int64_t)j;
        const float4 a = p[0], b = p[1];
        o[0] = a.x; o[1] = a.y; o[2] = a.z; tmin = a.w;
        d[0] = b.x; d[1] = b.y; d[2] = b.z; tmax = b.w;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            inv[k] = __fdiv_rn(1.0f, d[k]);
            par[k] = d[k] == 0.0f || inv[k] == INFINITY || inv[k] == -INFINITY;
        }
    }
    // the entry parameter in *enter when the ray meets the box
    __device__ bool enter(float4 lo4, float4 hi4, float *enter) const
    {
        const float lo[3] = {lo4.x, lo4.y, lo4.z}, hi[3] = {hi4.x, hi4.y, hi4.z};
        float t_in = tmin, t_out = tmax;
        bool ok = true;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (par[k]) {
                ok = ok && lo[k] <= o[k] && o[k] <= hi[k];
            } else {
                const float t1 = (lo[k] - o[k]) * inv[k];
                const float t2 = (hi[k] - o[k]) * inv[k];
                const float nr = t1 < t2 ? t1 : t2;
                const float fr = t1 < t2 ? t2 : t1;
                t_in = nr > t_in ? nr : t_in;
                t_out = fr < t_out ? fr : t_out;
            }
        }
        *enter = t_in;
        return ok && t_in <= t_out;
    }
    __device__ bool test(float4 lo, float4 hi) const
    {
        float e;
        return enter(lo, hi, &e);
    }
    // A thin set contains no box of positive volume; claiming none only
    // forgoes a shortcut.
    __device__ bool contains(float4, float4) const { return false; }
    // the start point as a degenerate box: it keys the query order by where
    // the ray starts
    __device__ void bounds(float lo[3], float hi[3]) const
    {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float t = (tmin == -INFINITY || d[k] == 0.0f) ? 0.0f : tmin;
            lo[k] = hi[k] = o[k] + t * d[k];
        }
    }
};

// The slab test of Ray::enter with the hardware's minimum and maximum, for a
// ray whose origin and interval hold no NaN, whose origin and direction are
// finite and none of whose axes is parallel: then no product is NaN, the
// verdict is the same and the entry parameter equal (a zero may differ in
// sign).  Other rays take Ray::enter.
struct FastRay {
    float o[3], tmin, inv[3], tmax;
    FastRay() = default;
    __device__ explicit FastRay(const Ray &q) : o{q.o[0], q.o[1], q.o[2]}, tmin(q.tmin),
                                                inv{q.inv[0], q.inv[1], q.inv[2]}, tmax(q.tmax) {}
    __device__ bool enter(float4 lo, float4 hi, float *e) const
    {
        const float ax = (lo.x - o[0]) * inv[0], bx = (hi.x - o[0]) * inv[0];
        const float ay = (lo.y - o[1]) * inv[1], by = (hi.y - o[1]) * inv[1];
        const float az = (lo.z - o[2]) * inv[2], bz = (hi.z - o[2]) * inv[2];
        const float in = fmaxf(fmaxf(fmaxf(fminf(ax, bx), fminf(ay, by)), fminf(az, bz)), tmin);
        const float out = fminf(fminf(fminf(fmaxf(ax, bx), fmaxf(ay, by)), fmaxf(az, bz)), tmax);
        *e = in;
        return in <= out;
    }
    __device__ bool test(float4 lo, float4 hi) const
    {
        float e;
        return enter(lo, hi, &e);
    }
    __device__ bool leaf(float4 lo, float4 hi) const { return test(lo, hi); }
};

// Error word values of a query call (the count call's workspace).
constexpr uint32_t kQErrWalkBudget = 5;   // a walk ran out of its node-visit budget

struct Tree {
    const float4 *nodes;
    const int32_t *perm;   // leaf k -> primitive
    int n;
    uint32_t *err = nullptr;   // count calls: where a walk that ran out of budget is flagged
    int64_t budget = 0;        // node visits allowed per walk (a packet's, for range queries); 0: 2n
    bool points = false;       // a tree of points: every leaf box has hi == lo
    __device__ int64_t walk_budget() const { return budget > 0 ? budget : 2 * (int64_t)n; }
    // a walk stopped with its budget spent: its count is short; report it
    __device__ void budget_spent() const
    {
        if (err) __hip_atomic_store(err, kQErrWalkBudget, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ int leaf0() const { return n - 1; }
    __device__ int index(int v) const { return v >= n - 1 ? v - (n - 1) : v; }
    __device__ void load(int v, float4 &a, float4 &b) const
    {
        const float4 *p = nodes + 2 * (int64_t)v;
        a = p[0];
        b = p[1];
    }
    // the box of leaf record v for a test: in a tree of points the upper
    // corner equals the lower one, so only the record's first half is read
    // (b.w, the rope, is then not loaded)
    __device__ void load_leaf_box(int v, float4 &a, float4 &b) const
    {
        const float4 *p = nodes + 2 * (int64_t)v;
        a = p[0];
        b = points ? make_float4(a.x, a.y, a.z, 0.0f) : p[1];
    }
    // right bound of node v whose record half `b` holds the rope
    __device__ int right_bound(float4 b) const
    {
        const int r = __float_as_int(b.w);
        return r == -1 ? n - 1 : index(r) - 1;
    }
};

constexpr int kWavesPerBlock = kBlock / 64;

// set lanes of mask below this lane
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Staged output of a fill pass, per wave.  The 64 queries a wave takes at a
// time have consecutive output ranges (query order is output order), so the
// wave gathers their hits in its own LDS
// region and writes them out in one coalesced run:
//   1. each lane walks its query; a leaf hit goes to the stage at its offset
//      from the wave's first output slot (put), an all-hit leaf range
//      becomes a job: output slot, first leaf_perm entry, length;
//   2. the wave copies the jobs from leaf_perm, 64 entries per lane step,
//      with up to kCopyDepth independent loads per lane in flight (a dense
//      query's hits are mostly such ranges: copying them one dependent
//      load at a time is what made filling slower than counting);
//   3. the wave writes the stage to the output.
// Hits past the stage capacity, and jobs past the job list, are written
// straight to the output: every hit lands in the same slot either way.
// Only the wave synchronises with itself, so a long walk holds up its own
// wave and no other.
constexpr int kWaveHits = 1024;
constexpr int kWaveJobs = 128;
constexpr int kCopyDepth = 8;

struct HitJob {
    int32_t rel;              // output slot - the wave's first slot
    int32_t a, len;
};

struct WaveStageLds {
    int32_t hits[kWavesPerBlock][kWaveHits];
    HitJob jobs[kWavesPerBlock][kWaveJobs];
    int njobs[kWavesPerBlock];
};

struct HitStage {
    int32_t *hits;            // the wave's LDS [kWaveHits]
    HitJob *jobs;             // the wave's LDS [kWaveJobs]
    int *njobs;               // the wave's LDS counter
    int32_t *out;
    const int32_t *perm;      // leaf_perm that job ranges index
    int64_t base;             // output slot of the wave's first item

    __device__ void put(int64_t pos, int32_t v) const
    {
        const int64_t r = pos - base;
        if (r < kWaveHits) hits[r] = v;
        else out[pos] = v;
    }
    // perm[a .. a+len) go to output slots pos .. pos+len
    __device__ void range(int64_t pos, int32_t a, int32_t len) const
    {
        if (len <= 0) return;
        const int64_t rel = pos - base;
        const int j = rel <= INT32_MAX ? atomicAdd(njobs, 1) : kWaveJobs;
        if (j < kWaveJobs) {
            jobs[j] = HitJob{(int32_t)rel, a, len};
            return;
        }
        // no room: this lane copies the range, kCopyDepth loads at a time
        for (int k0 = 0; k0 < len; k0 += kCopyDepth) {
            int32_t v[kCopyDepth];
#pragma unroll
            for (int u = 0; u < kCopyDepth; ++u)
                if (k0 + u < len) v[u] = perm[a + k0 + u];
#pragma unroll
            for (int u = 0; u < kCopyDepth; ++u)
                if (k0 + u < len) put(pos + k0 + u, v[u]);
        }
    }
    // steps 2 and 3; every lane of the wave calls it
    __device__ void flush(int64_t total) const
    {
        const int lane = threadIdx.x & 63;
        wave_sync();
        const int nj = *njobs < kWaveJobs ? *njobs : kWaveJobs;
        // walk the jobs in 64-entry slices; each round loads up to
        // kCopyDepth slices (of one or more jobs) before storing any
        int j = 0, off = 0;   // next slice: job j from entry off (uniform)
        while (j < nj) {
            int32_t v[kCopyDepth];
            int64_t dst[kCopyDepth];
#pragma unroll
            for (int u = 0; u < kCopyDepth; ++u) {
                dst[u] = -1;
                if (j < nj) {
                    const HitJob jb = jobs[j];
                    const int k = off + lane;
                    if (k < jb.len) {
                        v[u] = perm[jb.a + k];
                        dst[u] = base + jb.rel + k;
                    }
                    off += 64;
                    if (off >= jb.len) { ++j; off = 0; }
                }
            }
#pragma unroll
            for (int u = 0; u < kCopyDepth; ++u)
                if (dst[u] >= 0) put(dst[u], v[u]);
        }
        wave_sync();
        const int staged = total < kWaveHits ? (int)total : kWaveHits;
        for (int k = lane; k < staged; k += 64) out[base + k] = hits[k];
        if (lane == 0) *njobs = 0;
        wave_sync();   // the stage is reused by the wave's next items
    }
};

__device__ __forceinline__ HitStage wave_stage(WaveStageLds &lds, int32_t *out, const int32_t *perm,
                                               int64_t base)
{
    const int w = threadIdx.x >> 6;
    return HitStage{lds.hits[w], lds.jobs[w], &lds.njobs[w], out, perm, base};
}

// Offsets of a count call with nothing to walk: all zero; and the call's
// error word cleared.
__global__ void k_zero_i64(int64_t *p, int64_t count, uint32_t *err)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < count) p[i] = 0;
    if (i == 0) *err = 0u;
}

// -------------------------------------------------------------- scan
//
// Exclusive scan of m int32 counts into int64 offsets[0..m] (offsets[m] =
// total), and into a second copy where `copy` is not null.  One launch: a
// block takes the next tile of kScanTile counts from a counter (so every
// tile it waits for is already running), publishes the tile's sum and adds
// up the earlier tiles' with a decoupled look-back, one wave reading 4 x 64
// status words at a time (bound by the latency of these reads, which cross
// the chip; with 64 at a time and offsets stored 64 bytes apart per lane,
// 2^20 counts took 24 instead of 16 us).  A status word holds two flag bits over a 62-bit
// sum, so it needs no fence.  Words and counter are zero on entry.  A wait
// that never ends (not expected) is cut and flagged.  Three launches
// (sums, their scan, the final pass) took 58 us over 2^20 counts and three
// scans, and about 10 us when there was nothing to scan.
constexpr uint64_t kScanSum = 1ull << 62, kScanPrefix = 2ull << 62, kScanValue = (1ull << 62) - 1;
constexpr uint32_t kQErrScan = 6;
constexpr int kScanAhead = 4;   // look-back words per lane in flight

inline int64_t scan_tiles(int64_t m) { return (m + kScanTile - 1) / kScanTile; }

__global__ __launch_bounds__(kBlock) void k_scan(const int32_t *__restrict__ counts, int64_t m,
                                                 uint64_t *status, uint32_t *counter,
                                                 int64_t *__restrict__ offsets,
                                                 int64_t *__restrict__ copy, uint32_t *err)
{
    __shared__ int64_t sh[kBlock / 64];
    __shared__ uint32_t s_tile;
    __shared__ int64_t s_before;
    __shared__ int64_t s_run[kBlock * (kScanItems + 1)];   // rows apart in the banks
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) s_tile = gridDim.x > 1 ? atomicAdd(counter, 1u) : 0u;
    __syncthreads();
    const int64_t tile = s_tile;
    const int64_t base = tile * kScanTile + (int64_t)threadIdx.x * kScanItems;
    int32_t c[kScanItems];
    int64_t sum = 0;
    if (base + kScanItems <= m) {   // counts is aligned to 16 bytes
#pragma unroll
        for (int k = 0; k < kScanItems; k += 4) {
            const int4 v = *reinterpret_cast<const int4 *>(counts + base + k);
            c[k] = v.x; c[k + 1] = v.y; c[k + 2] = v.z; c[k + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) c[k] = base + k < m ? counts[base + k] : 0;
    }
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) sum += c[k];
    int64_t x = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int64_t y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == 63) sh[wave] = x;
    __syncthreads();
    int64_t before = 0, all = 0;
    for (int w = 0; w < kBlock / 64; ++w) {
        if (w < wave) before += sh[w];
        all += sh[w];
    }
    if (gridDim.x > 1) {
        if (threadIdx.x == 0)
            __hip_atomic_store(status + tile, (tile == 0 ? kScanPrefix : kScanSum) | (uint64_t)all,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (wave == 0) {
            int64_t found = 0;
            uint32_t spins = 0;
            bool done = tile == 0;
            for (int64_t j = tile - 1; !done;) {   // word u of lane l: tile j - 64 u - l
                uint64_t s[kScanAhead];
#pragma unroll
                for (int u = 0; u < kScanAhead; ++u)
                    s[u] = j - 64 * u >= lane ? __hip_atomic_load(status + j - 64 * u - lane, __ATOMIC_RELAXED,
                                                                  __HIP_MEMORY_SCOPE_AGENT)
                                              : kScanPrefix;
#pragma unroll
                for (int u = 0; u < kScanAhead; ++u) {
                    const uint64_t empty = __ballot((s[u] >> 62) == 0), prefix = __ballot((s[u] >> 62) == 2);
                    const int upto = prefix ? __ffsll((unsigned long long)prefix) - 1 : 63;   // last lane to add
                    if (empty & (upto == 63 ? ~0ull : (2ull << upto) - 1ull)) {
                        if (++spins > (1u << 22)) {   // never expected: bounded wait
                            if (lane == 0)
                                __hip_atomic_store(err, kQErrScan, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            done = true;
                        }
                        __builtin_amdgcn_s_sleep(1);
                        break;
                    }
                    int64_t v = lane <= upto ? (int64_t)(s[u] & kScanValue) : 0;
#pragma unroll
                    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
                    found += v;
                    done = prefix != 0;
                    if (done) break;
                    j -= 64;
                    // the words after this one were read relative to the old j
                }
            }
            if (lane == 0) {
                s_before = found;
                __hip_atomic_store(status + tile, kScanPrefix | (uint64_t)(found + all), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
        before += s_before;
    }
    int64_t run = before + x - sum;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        s_run[threadIdx.x * (kScanItems + 1) + k] = run;
        run += c[k];
        if (base + k == m - 1) {
            offsets[m] = run;
            if (copy) copy[m] = run;
        }
    }
    __syncthreads();
    // a wave's offsets leave as one run
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int i = k * kBlock + threadIdx.x;
        const int64_t j = tile * kScanTile + i;
        if (j < m) {
            const int64_t v = s_run[i / kScanItems * (kScanItems + 1) + i % kScanItems];
            offsets[j] = v;
            if (copy) copy[j] = v;
        }
    }
}

// m >= 1; `status` holds scan_tiles(m) words
void scan(const int32_t *counts, int64_t m, uint64_t *status, uint32_t *counter, int64_t *offsets,
          int64_t *copy, uint32_t *err, hipStream_t s)
{
    hipLaunchKernelGGL(k_scan, dim3((unsigned)scan_tiles(m)), dim3(kBlock), 0, s, counts, m, status,
                       counter, offsets, copy, err);
}

}  // namespace
}  // namespace lbvh
