// Codes and sorted order of one scene by one block.
#pragma once
#pragma clang fp contract(off)

#include "device_common.hpp"
#include "radix_sort.hpp"

namespace lbvh {
namespace {

// ------------------------------------------------- one block per scene
//
// The other sort schedule of the batched build ("batch_sort_mode" 1), and the
// sort of a single small tree (seg_off null: n_one primitives): one block takes
// one whole scene (scenes in decreasing size, so the longest blocks start
// first) and runs every step up to the sorted codes itself:
// scene box and scale, the codes with every pass's digit histogram, then
// the sort.  A scene of one tile (T*I keys) is sorted on chip.  A larger
// scene is partitioned by its top digit in one pass over global memory and
// its runs of whole digit values, packed up to a tile, are sorted on chip;
// if one top-digit value holds more than a tile, each LSD pass runs over
// the scene in tiles instead.  A tile is ranked stably with wave64 ballots
// (as in the onesweep pass) and scattered through LDS so that global
// writes are runs of equal digits; the block's running start of each digit
// carries over from tile to tile, so no tile waits for another block (no
// look-back), and scenes need no tile plan.  Global writes of one pass are
// read by the next step of the same block after a workgroup barrier.
template <int KIND, typename K, int BITS, int T, int I>
__global__ __launch_bounds__(T) void k_scene_sort(
    const float *__restrict__ prims, const int64_t *__restrict__ seg_off,
    const int32_t *__restrict__ order, uint32_t n_one, int code_bits, float4 *__restrict__ scene_box, K *key_a,
    K *key_b, int32_t *val_a, int32_t *val_b, int32_t *__restrict__ perm_out, uint32_t *err)
{
    constexpr int R = 1 << BITS;
    constexpr int W = T / 64;
    constexpr int TILE = T * I;
    constexpr int DPT = (R + T - 1) / T;
    constexpr int PASSES = ((sizeof(K) == 4 ? 30 : 63) + BITS - 1) / BITS;
    static_assert(TILE < 65536, "16-bit per-wave digit counters");
    using Cnt = typename std::conditional<(BITS <= 9), uint32_t, uint16_t>::type;
    using P = Prims<KIND>;
    __shared__ __align__(16) Cnt s_wcnt[W][R];
    __shared__ uint32_t s_start[R];   // tile-local start of each digit run
    __shared__ uint32_t s_run[2][R];  // scene-local start of the digit's next run
    __shared__ uint32_t s_hist[R];    // one digit's counts over the scene
    __shared__ uint32_t s_scan[2][W];
    __shared__ K s_buf[TILE];
    __shared__ int32_t s_val[TILE];
    __shared__ float sh[W * 6];
    __shared__ float4 s_box[3];
    __shared__ uint32_t s_flag;       // some top digit holds more than a tile
    __shared__ uint32_t s_last[2];    // last digit of the current run group

    int s = 0;
    int64_t b0 = 0;
    uint32_t ns = n_one;
    if (seg_off) {
        s = order[blockIdx.x];
        b0 = seg_off[s];
        ns = (uint32_t)(seg_off[s + 1] - b0);   // a scene holds fewer than 2^30 primitives
        if (ns == 0) return;
    } else if (threadIdx.x == 0) {
        *err = 0u;   // a single tree's build starts here
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int j = tid; j < R; j += T) s_hist[j] = 0u;
    if (tid == 0) { s_flag = 0u; s_last[0] = 0u; }

    // scene box and scale (2^b / extent, correctly rounded; 0 when flat)
    float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (uint32_t i = tid; i < ns; i += T) {
        float lo[3], hi[3];
        P::one(prims, b0 + i, lo, hi);
#pragma unroll
        for (int a = 0; a < 3; ++a) { v[a] = fminf(v[a], lo[a]); v[3 + a] = fmaxf(v[3 + a], hi[a]); }
    }
    block_minmax6<T>(v, sh);
    if (tid == 0) {
        const float two_b = (float)(1u << (code_bits / 3));
        float sc[3];
        for (int a = 0; a < 3; ++a) {
            const float ext = v[3 + a] - v[a];
            sc[a] = ext > 0.0f ? __fdiv_rn(two_b, ext) : 0.0f;
        }
        s_box[0] = make_float4(v[0], v[1], v[2], 0.0f);
        s_box[1] = make_float4(v[3], v[4], v[5], 0.0f);
        s_box[2] = make_float4(sc[0], sc[1], sc[2], 0.0f);
        scene_box[3 * s + 0] = s_box[0];
        scene_box[3 * s + 1] = s_box[1];
        scene_box[3 * s + 2] = s_box[2];
    }
    __syncthreads();
    // codes in input order, and (scenes of several tiles) the top digit's
    // counts; the other digits are counted only if the scene needs them
    const int top = PASSES - 1;
    const int top_shift = top * BITS;
    {
        const float4 slo = s_box[0], sc = s_box[2];
        const bool count = ns > (uint32_t)TILE;
        for (uint32_t i = tid; i < ns; i += T) {
            float lo[3], hi[3];
            P::one(prims, b0 + i, lo, hi);
            const K c = code_of<KIND, K>(lo, hi, slo, sc);
            key_a[b0 + i] = c;
            if (count) atomicAdd(&s_hist[(uint32_t)((c >> top_shift) & (R - 1))], 1u);
        }
    }
    __threadfence_block();
    __syncthreads();

    const int d0 = tid * DPT;
    auto owns = [&](int k) { return d0 + k < R; };
    constexpr int kZeroWords = W * R * (int)sizeof(Cnt) / 4;
    auto zero_counts = [&]() {
        for (int j = tid; j < kZeroWords; j += T) reinterpret_cast<uint32_t *>(&s_wcnt[0][0])[j] = 0u;
    };
    // The tile ranking shared by both paths below: key k of this thread is
    // the tile's key lofs + 64k (rem keys in the tile); returns each key's
    // position in the tile's stable order by this pass's digit.  The wave
    // counters must be zero on entry (each caller clears them, after its
    // last read of the previous ranking and before a barrier).
    auto rank_tile = [&](const K (&key)[I], uint32_t rem, uint32_t lofs, int shift,
                         uint32_t (&pos)[I], uint32_t (&total)[DPT], uint32_t (&start)[DPT]) {
        uint32_t rank[I];
        // the wave's first key (a scalar: rows with no key in the tile are
        // skipped by a branch of the whole wave)
        const uint32_t wbase = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lofs - lane));
#pragma unroll
        for (int k = 0; k < I; ++k) {
            rank[k] = 0u;
            if (wbase + k * 64 >= rem) continue;
            const bool ok = lofs + k * 64 < rem;
            const uint32_t d = (uint32_t)(key[k] >> shift) & (R - 1);
            // bits of a narrower last digit are zero above it in every key
            const uint64_t peers = __ballot(ok) & ~digit_diff<BITS>(d);
            const uint32_t below = count_below(peers);
            const uint32_t cnt = s_wcnt[wave][d];
            rank[k] = cnt + below;
            if (ok && below == 0) s_wcnt[wave][d] = (Cnt)(cnt + (uint32_t)__popcll(peers));
        }
        __syncthreads();
        // per-wave exclusive offsets and the tile's digit totals
#pragma unroll
        for (int k = 0; k < DPT; ++k) {
            total[k] = 0;
            if (owns(k)) {
                const int d = d0 + k;
                uint32_t c[W];
#pragma unroll
                for (int w = 0; w < W; ++w) c[w] = s_wcnt[w][d];
#pragma unroll
                for (int w = 0; w < W; ++w) { s_wcnt[w][d] = (Cnt)total[k]; total[k] += c[w]; }
            }
        }
        digits_excl_scan<T, DPT>(total, start, s_scan[1]);
#pragma unroll
        for (int k = 0; k < DPT; ++k)
            if (owns(k)) s_start[d0 + k] = start[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < I; ++k) {
            pos[k] = 0u;
            if (wbase + k * 64 >= rem) continue;
            const uint32_t dk = (uint32_t)(key[k] >> shift) & (R - 1);
            pos[k] = s_start[dk] + s_wcnt[wave][dk] + rank[k];
        }
    };
    const uint32_t lofs = (uint32_t)(wave * 64 * I + lane);
    K *const kfinal = ((PASSES - 1) & 1) ? key_a : key_b;
    // Keys [off, off + cnt) of kin (cnt <= TILE) sorted on chip: each pass
    // reorders them through LDS and only the last pass writes, the sorted
    // codes to kfinal and the permutation to perm_out at the same places.
    // Values are vin's, or the scene-local index when vin is null.  kin may
    // be kfinal: every key is in registers before the first barrier.  The
    // caller's last barrier must follow its last read of the wave counters.
    auto sort_on_chip = [&](const K *kin, const int32_t *vin, uint32_t off, uint32_t cnt) {
        K key[I];
        int32_t val[I];
        zero_counts();
#pragma unroll
        for (int k = 0; k < I; ++k) {
            const bool ok = lofs + k * 64 < cnt;
            const int64_t at = b0 + off + lofs + k * 64;
            key[k] = ok ? kin[at] : (K)0;
            val[k] = vin ? (ok ? vin[at] : 0) : (int32_t)(off + lofs + k * 64);
        }
        __syncthreads();
        for (int p = 0; p < PASSES; ++p) {
            const int shift = p * BITS;
            uint32_t pos[I], total[DPT], start[DPT];
            rank_tile(key, cnt, lofs, shift, pos, total, start);
            if (p + 1 == PASSES) {
#pragma unroll
                for (int k = 0; k < I; ++k)
                    if (lofs + k * 64 < cnt) {
                        kfinal[b0 + off + pos[k]] = key[k];
                        perm_out[b0 + off + pos[k]] = val[k];
                    }
                break;
            }
#pragma unroll
            for (int k = 0; k < I; ++k)
                if (lofs + k * 64 < cnt) {
                    s_buf[pos[k]] = key[k];
                    s_val[pos[k]] = val[k];
                }
            __syncthreads();
            zero_counts();   // every position is read
#pragma unroll
            for (int k = 0; k < I; ++k) {
                const bool ok = lofs + k * 64 < cnt;
                key[k] = ok ? s_buf[lofs + k * 64] : (K)0;
                val[k] = ok ? s_val[lofs + k * 64] : 0;
            }
            __syncthreads();
        }
    };
    // One stable pass over the whole scene by the digit at `shift` (its
    // counts in s_hist), tile after tile through global memory.  The
    // running start of each digit alternates between the two rows of s_run
    // (tile t reads row t & 1 and its owner writes the next row), so no
    // barrier guards it; returns the row that ends up holding the
    // scene-local end of each digit's run.
    auto global_pass = [&](const K *kin, K *kout, const int32_t *vin, int32_t *vout, int shift) -> int {
        zero_counts();
        {   // the scene-local start of each digit in this pass
            uint32_t h[DPT], st[DPT];
#pragma unroll
            for (int k = 0; k < DPT; ++k) h[k] = owns(k) ? s_hist[d0 + k] : 0u;
            digits_excl_scan<T, DPT>(h, st, s_scan[0]);
#pragma unroll
            for (int k = 0; k < DPT; ++k)
                if (owns(k)) s_run[0][d0 + k] = st[k];
        }
        int row = 0;
        for (uint32_t base = 0; base < ns; base += TILE, row ^= 1) {
            const uint32_t rem = ns - base < (uint32_t)TILE ? ns - base : (uint32_t)TILE;
            K key[I];
            int32_t val[I];
#pragma unroll
            for (int k = 0; k < I; ++k) {
                const bool ok = lofs + k * 64 < rem;
                const int64_t at = b0 + base + lofs + k * 64;
                key[k] = ok ? kin[at] : (K)0;
                val[k] = vin ? (ok ? vin[at] : 0) : (int32_t)(base + lofs + k * 64);
            }
            // stable rank within the wave, as in the onesweep pass
            uint32_t pos[I], total[DPT], start[DPT];
            rank_tile(key, rem, lofs, shift, pos, total, start);
            // the next tile's runs of each digit follow this tile's
#pragma unroll
            for (int k = 0; k < DPT; ++k)
                if (owns(k)) s_run[row ^ 1][d0 + k] = s_run[row][d0 + k] + total[k];
#pragma unroll
            for (int k = 0; k < I; ++k)
                if (lofs + k * 64 < rem) {
                    s_buf[pos[k]] = key[k];
                    s_val[pos[k]] = val[k];
                }
            __syncthreads();
            zero_counts();
#pragma unroll
            for (int k = 0; k < I; ++k) {
                const uint32_t q = (uint32_t)(k * T + tid);
                if (q < rem) {
                    const K kk = s_buf[q];
                    const uint32_t dk = (uint32_t)(kk >> shift) & (R - 1);
                    const uint32_t out = s_run[row][dk] + q - s_start[dk];   // < ns by construction
                    if (out < ns) {
                        kout[b0 + out] = kk;
                        vout[b0 + out] = s_val[q];
                    } else {   // inconsistent counts: flag it rather than write outside
                        __hip_atomic_store(err, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
            }
            __syncthreads();
        }
        // this pass's writes are the next reads (same block)
        __threadfence_block();
        __syncthreads();
        return row;
    };

    if (ns <= (uint32_t)TILE) {   // one tile: all passes on chip
        sort_on_chip(key_a, nullptr, 0u, ns);
        return;
    }
    // Several tiles.  When no value of the top digit holds more than a
    // tile's keys, one global pass partitions the scene by the top digit
    // (most significant first), and runs of whole digit values, packed up to
    // a tile, are then sorted on chip by the whole code: the final order of
    // each run's keys lies inside the run, and both steps are stable, so
    // equal codes keep their input order.  Two global passes instead of one
    // per digit.  Otherwise every pass runs over the scene (least
    // significant digit first).
    const int top_bits = BITS < code_bits - top_shift ? BITS : code_bits - top_shift;
#pragma unroll
    for (int k = 0; k < DPT; ++k)
        if (owns(k) && s_hist[d0 + k] > (uint32_t)TILE) s_flag = 1u;
    __syncthreads();
    if (s_flag == 0u && top_bits > 0) {
        const uint32_t *end = s_run[global_pass(key_a, key_b, nullptr, val_a, top_shift)];
        // digit d's keys now lie in [end[d-1], end[d]) of key_b / val_a;
        // group g takes digits gb..last, the most that fit a tile (slot
        // g & 1 of s_last holds gb before the max)
        uint32_t gb = 0;
        for (int g = 0;; ++g) {
            const uint32_t gstart = gb == 0 ? 0u : end[gb - 1];
            if (gb >= (uint32_t)R || gstart >= ns) break;
#pragma unroll
            for (int k = 0; k < DPT; ++k) {
                const uint32_t d = (uint32_t)(d0 + k);
                if (owns(k) && d >= gb && end[d] - gstart <= (uint32_t)TILE) atomicMax(&s_last[g & 1], d);
            }
            __syncthreads();
            const uint32_t last = s_last[g & 1];
            const uint32_t gend = end[last];
            if (tid == 0) s_last[(g + 1) & 1] = last + 1;
            if (gend <= gstart || gend > ns || gend - gstart > (uint32_t)TILE) {   // not expected
                if (tid == 0) __hip_atomic_store(err, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            sort_on_chip(key_b, val_a, gstart, gend - gstart);
            gb = last + 1;
        }
        return;
    }
    for (int p = 0; p < PASSES; ++p) {
        const K *kin = (p & 1) ? key_b : key_a;
        K *kout = (p & 1) ? key_a : key_b;
        const int32_t *vin = p == 0 ? nullptr : ((p & 1) ? val_a : val_b);
        int32_t *vout = p + 1 == PASSES ? perm_out : ((p & 1) ? val_b : val_a);
        const int shift = p * BITS;
        // this digit's counts (the previous pass read s_hist before its
        // last barrier)
        for (int j = tid; j < R; j += T) s_hist[j] = 0u;
        __syncthreads();
        for (uint32_t i = tid; i < ns; i += T)
            atomicAdd(&s_hist[(uint32_t)((kin[b0 + i] >> shift) & (R - 1))], 1u);
        __syncthreads();
        global_pass(kin, kout, vin, vout, shift);
    }
}

}  // namespace
}  // namespace lbvh
