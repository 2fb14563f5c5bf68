// PiKV scheduling score (Section 3.4, Table 3 row H2O: u_i = a_i, the attention an entry
// received), kept as a running value u_i <- decay * u_i + a_i.
//
// The attention pass left the raw scores s_{h,i} of every visited entry and, per (query
// head, selected shard), a pair (shift, coef) with p_{h,i} = coef * exp(s_{h,i} - shift).
// This pass turns them into probabilities and sums them over the heads that read the
// entry, in fixed head order (no atomics, bit-reproducible).  Grid: (sequence, selected shard,
// slot tile) under per-token routing, (sequence, expert, slot tile) where the heads are routed one by one;
// blocks of shards nobody selected exit at once and leave u untouched.
//
// The tracked form also keeps the per-entry bookkeeping of Table 3's LRU / LRU+ rows in the
// same pass: an entry whose attention mass of this step exceeds a threshold has its
// last-access stamp set to the step counter and its access count raised by one.
#include "pikv_common.h"

#include <math.h>

namespace pikv {
namespace {

// Thread = (SPT slots, quarter of the heads): 64 * SPT slots per block, a wave per quarter, kUtilBatch heads' scores
// of each slot in flight per thread, the quarters' sums joined in LDS as (g0 + g1) + (g2 + g3).  Two trips to memory:
// selections and counts, then pairs, scores and old utilities together.  Bound by those trips, or by the score bytes once
// there are many.  With the counts, the selections, the pairs and each group's scores requested one after the other - up to
// seven trips - kernel trace: 10 sequences x 64 heads x 2 of 6 shards of 2560 slots 9.4 -> 4.8 us, 4 x 16 x 3 of 6
// ragged ones of 1501 4.8 -> 3.2, 1 x 256 x 4 of 8192 9.6 -> 8.1; heads routed one by one: 23 x 128 x 2 of 32 of 1536
// 27.2 -> 16.0, 1 x 4 x 2 of 4 of 256 3.1 -> 3.0.
constexpr int kUtilThreads = 256;
constexpr int kUtilBatch = 8;           // heads whose scores are in flight per thread ...
constexpr int kUtilFewBatch = 2;        // ... of up to kUtilFewHeads in all
constexpr int kUtilFewHeads = 4 * kUtilFewBatch;
// Heads routed one by one: those that meet a shard count, on average.  By all heads a block requested the same rows again and
// again for a batch it could not fill (in a graph, with a batch of 8 and with the one for those met: 76 sequences x 48 heads x 1 of 64
// shards of 61 slots 8.3 -> 6.2 us, 40 x 11 x 1 of 16 of 2363 10.2 -> 7.9, 24 x 32 x 2 of 16 of 2047 8.9 -> 6.2).
constexpr int kUtilSomeBatch = 4, kUtilSomeHeads = 4 * kUtilSomeBatch;
// Many heads in few blocks: a batch is a trip and what a CU has in flight bounds the rate (256 heads x 4 of 8192 slots, 32 MiB,
// batches of 8 8.1 us, 16 7.3, 32 7.1; 128 heads 5.1, 4.85, 4.9).
constexpr int kUtilManyHeads = 64, kUtilManyBatch = 16;
// Four slots per thread once one slot per thread makes more blocks than this (24 sequences x 32 heads x 2 of 16 shards of 2048
// slots, routed head by head, 17.4 us with one; the form before 13.6; now 9.4).
constexpr int kUtilManyBlocks = 1024;
// Head by head, from this many heads on, at twice the blocks: with 1024 - 2048 of them one slot per thread takes 0.87 of the time
// of four where shards are nearly empty (0.62 at best), 1.00 where they are half full and 1.04 where they are full (250 random shapes).
// Per token the line stays: full shards gain 1.2 from four slots (16 sequences x 128 heads x 4 of 16 shards of 4096 slots 23.2 us,
// in blocks of 64 slots 25.6), nearly empty ones lose where few blocks are left (85 x 224 x 2 of 2 of 1888, a sixteenth
// full, 17.4 against 10.3), and the host does not see the counts.
constexpr int kUtilSparseHeads = 128;

struct UtilParams {
    const float *scores;
    const float *slot_coef;
    const int32_t *n_valid;
    const int32_t *topk;
    float *utility;      // may be null in the tracked form
    FastDiv by_tiles, by_shards;     // selected shards of a sequence, or all
    int Hq, E, S, k, rr;
    float decay;
    // access bookkeeping (Table 3 rows LRU / LRU+): an entry whose attention mass of this
    // step exceeds `threshold` is accessed at step `now`
    int32_t *last_access;
    int32_t *freq;
    float threshold;
    int now;
};

// TOKEN: one routing decision per sequence - every head reads the selected shards.
// A thread's slots are consecutive (LINE: 16-byte loads of aligned rows) or 64 apart.
template <bool TRACK, int SPT, bool LINE, bool TOKEN, int BATCH>
__global__ __launch_bounds__(kUtilThreads) void utility_kernel(UtilParams p) {
    constexpr int kSlots = kUtilThreads / 4 * SPT;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tile, x;
    const int rest = fast_divide(p.by_tiles, blockIdx.x, &tile);
    const int b = fast_divide(p.by_shards, rest, &x);
    if constexpr (SPT == 4) {
        // Blocks go to the XCDs by id: where the tiles of a shard are a multiple of 8, or divide it, each XCD would have its own
        // ones, and shards that are not full leave the last XCDs idle.  So every fourth shard starts a tile further (half full:
        // 142 sequences x 128 heads x 4 of 4 shards of 1852 slots 73.6 -> 49.8 us).
        int turn;
        fast_divide(p.by_tiles, rest >> 2, &turn);
        tile += turn;
        if (tile >= (int)p.by_tiles.d) tile -= (int)p.by_tiles.d;
    }
    const int i0 = tile * kSlots;

    __shared__ int head_row[TOKEN ? 1 : 256];       // heads that selected the shard, ascending: (sequence, head, selection)
    __shared__ float2 head_w[256];      // their (shift, coef)
    __shared__ int wave_cnt[kUtilThreads / kWave];
    __shared__ float part_s[4][kSlots];

    // (one count per lane, the shard's own picked when it is needed: a load that is the same in all lanes is waited
    // for where it stands)
    const int n_of_lane = p.n_valid[(int64_t)b * p.E + min(lane, p.E - 1)];
    int e = x, n = 0, nact = p.Hq;
    if constexpr (TOKEN) {
        const int sel = p.topk[(int64_t)b * p.k + min(lane, p.k - 1)];
        e = __builtin_amdgcn_readlane(sel, x);
        // (of a shard selected twice the last selection counts)
        if (e < 0 || e >= p.E || __ballot(sel == e && lane > x && lane < p.k) != 0) return;
        n = __builtin_amdgcn_readlane(n_of_lane, e);
        if (i0 >= n) return;
    } else {
        if constexpr (SPT == 4) {        // many blocks: those past the count don't wait for selections
            n = __builtin_amdgcn_readlane(n_of_lane, e);
            if (i0 >= n) return;
        }
        constexpr int kSel = 4;          // selections requested at a time
        const int32_t *row = p.topk + ((int64_t)b * p.rr + min(tid, p.Hq - 1)) * p.k;
        int jj = -1;
        for (int j0 = 0; j0 < p.k; j0 += kSel) {
            int sel[kSel];
#pragma unroll
            for (int t = 0; t < kSel; ++t) sel[t] = row[min(j0 + t, p.k - 1)];
#pragma unroll
            for (int t = 0; t < kSel; ++t) jj = sel[t] == e ? min(j0 + t, p.k - 1) : jj;
        }
        if constexpr (SPT == 1) {
            n = __builtin_amdgcn_readlane(n_of_lane, e);
            if (i0 >= n) return;
        }
        const bool active = tid < p.Hq && jj >= 0;
        const uint64_t mask = __ballot(active);
        if (lane == 0) wave_cnt[wave] = __popcll(mask);
        __syncthreads();
        int before = 0;
        nact = 0;
#pragma unroll
        for (int w = 0; w < kUtilThreads / kWave; ++w) {
            if (w < wave) before += wave_cnt[w];
            nact += wave_cnt[w];
        }
        nact = __builtin_amdgcn_readfirstlane(nact);
        if (nact == 0) return;
        if (active) head_row[before + __popcll(mask & ((1ull << lane) - 1ull))] = (b * p.Hq + tid) * p.k + jj;
        __syncthreads();
    }
    auto row_of = [&](int t) { return TOKEN ? (b * p.Hq + t) * p.k + x : head_row[t]; };

    // the pairs, the scores, the old utilities: requested together, in this order (loads come back in order)
    const int64_t pair_at = (int64_t)row_of(min(tid, nact - 1)) * 2;
    const float shift = p.slot_coef[pair_at], coef = p.slot_coef[pair_at + 1];
    const int gsize = (nact + 3) / 4, lo = wave * gsize, hi = min(nact, lo + gsize);
    const int slot = LINE ? lane * SPT : lane;
    // the quarter's rows, at most 64: one trip to LDS instead of one per batch (55 sequences x 256 heads, 2 shards of 80 slots, 6.25 -> 5.75 us)
    const int row_of_lane = TOKEN ? 0 : head_row[min(lo + lane, nact - 1)];
    float sc[BATCH][SPT];
    auto fetch = [&](int t0) {           // (heads past the group's end and slots past the count are masked where they are used)
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int row = TOKEN ? row_of(min(t0 + u, nact - 1)) : __builtin_amdgcn_readlane(row_of_lane, t0 - lo + u);
            const float *from = p.scores + (int64_t)row * p.S;
            if constexpr (LINE) {
                // (no line past the last entry's: 35 x 128 x 10 of 16 of 780 slots, nearly empty, 26.8 us with whole tiles, now 13.1)
                const float4 v = *reinterpret_cast<const float4 *>(from + min(i0 + slot, (n - 1) & ~3));
                sc[u][0] = v.x, sc[u][1] = v.y, sc[u][2] = v.z, sc[u][3] = v.w;
            } else {
#pragma unroll
                for (int s = 0; s < SPT; ++s) sc[u][s] = from[min(i0 + slot + s * kWave, n - 1)];
            }
        }
    };
    fetch(lo);
    // the block's slots are written by the first wave, or a slot by every thread
    const int i = i0 + tid;
    const bool writes = (SPT == 4 || wave == 0) && i < n;
    const int64_t at = ((int64_t)b * p.E + e) * p.S + i;
    const bool scored = !TRACK || p.utility != nullptr;
    const float old = writes && scored ? p.utility[at] : 0.0f;
    if (tid < nact) head_w[tid] = make_float2(shift, coef);
    __syncthreads();

    float a[SPT];
#pragma unroll
    for (int s = 0; s < SPT; ++s) a[s] = 0.0f;
    for (int t0 = lo; t0 < hi; t0 += BATCH) {
        if (t0 != lo) fetch(t0);
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const float2 w = head_w[min(t0 + u, nact - 1)];
#pragma unroll
            for (int s = 0; s < SPT; ++s) {
                const float with = fmaf(w.y, __expf(sc[u][s] - w.x), a[s]);
                a[s] = t0 + u < hi ? with : a[s];
            }
        }
    }
#pragma unroll
    for (int s = 0; s < SPT; ++s) part_s[wave][slot + (LINE ? s : s * kWave)] = a[s];
    __syncthreads();
    if (!writes) return;
    const float mass = (part_s[0][tid] + part_s[1][tid]) + (part_s[2][tid] + part_s[3][tid]);
    if (scored) p.utility[at] = fmaf(p.decay, old, mass);
    if (TRACK && mass > p.threshold) {
        p.last_access[at] = p.now;
        p.freq[at] += 1;
    }
}

int launch_utility(const pikv_desc *desc, const float *scores, const float *slot_coef,
                   const int32_t *n_valid, const int32_t *topk_idx, int32_t k, float decay,
                   float *utility, bool track, float threshold, int32_t now,
                   int32_t *last_access, int32_t *freq, void *stream) {
    UtilParams p;
    p.scores = scores;
    p.slot_coef = slot_coef;
    p.n_valid = n_valid;
    p.topk = topk_idx;
    p.utility = utility;
    p.Hq = desc->Hq;
    p.E = desc->E;
    p.S = desc->S;
    p.k = k;
    p.rr = desc->route_rows_per_seq;
    const int shards = p.rr == 1 ? k : desc->E;
    auto blocks_of = [&](int slots) { return (int64_t)desc->B * shards * ((desc->S + slots - 1) / slots); };
    const bool wide = blocks_of(kUtilThreads / 4) > (p.rr != 1 && desc->Hq >= kUtilSparseHeads ? 2 : 1) * kUtilManyBlocks;
    const bool line = desc->S % 4 == 0 && reinterpret_cast<uintptr_t>(scores) % 16 == 0;
    const int tile_slots = wide ? kUtilThreads : kUtilThreads / 4;
    p.by_tiles = fast_div((desc->S + tile_slots - 1) / tile_slots);
    p.by_shards = fast_div(shards);
    p.decay = decay;
    p.last_access = last_access;
    p.freq = freq;
    p.threshold = threshold;
    p.now = now;
    const int64_t blocks = blocks_of(tile_slots);
    if (blocks > 0x7fffffff) return PIKV_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)blocks), block(kUtilThreads);
    hipStream_t st = as_stream(stream);
    auto launch = [&](auto tracks, auto spt, auto lines, auto token, auto batch) {
        constexpr bool TRACK = decltype(tracks)::value, LINE = decltype(lines)::value, TOKEN = decltype(token)::value;
        constexpr int SPT = decltype(spt)::value, BATCH = decltype(batch)::value;
        hipLaunchKernelGGL((utility_kernel<TRACK, SPT, LINE, TOKEN, BATCH>), grid, block, 0, st, p);
    };
    const std::integral_constant<int, 4> four{};
    const std::integral_constant<int, 1> one{};
    auto launch_wide = [&](auto tracks, auto token, auto batch) {
        if (wide && line) launch(tracks, four, std::true_type{}, token, batch);
        else if (wide) launch(tracks, four, std::false_type{}, token, batch);
        else launch(tracks, one, std::false_type{}, token, batch);
    };
    const std::integral_constant<int, kUtilFewBatch> few{};
    const std::integral_constant<int, kUtilSomeBatch> some{};
    const std::integral_constant<int, kUtilBatch> several{};
    const std::integral_constant<int, kUtilManyBatch> many{};
    auto launch_batch = [&](auto tracks) {
        if (p.rr != 1) {
            const int64_t met = ((int64_t)desc->Hq * k + desc->E - 1) / desc->E;      // heads that meet a shard, on average
            if (met <= kUtilFewHeads) launch_wide(tracks, std::false_type{}, few);
            else if (met <= kUtilSomeHeads) launch_wide(tracks, std::false_type{}, some);
            else launch_wide(tracks, std::false_type{}, several);
        } else {
            if (desc->Hq <= kUtilFewHeads) launch_wide(tracks, std::true_type{}, few);
            else if (desc->Hq > kUtilManyHeads && !wide) launch(tracks, one, std::false_type{}, std::true_type{}, many);
            else launch_wide(tracks, std::true_type{}, several);
        }
    };
    if (track) launch_batch(std::true_type{});
    else launch_batch(std::false_type{});
    return launch_status();
}

}  // namespace
}  // namespace pikv

using namespace pikv;

extern "C" int pikv_update_utility(const pikv_desc *desc, const float *scores,
                                   const float *slot_coef, const int32_t *n_valid,
                                   const int32_t *topk_idx, int32_t k, float decay,
                                   float *utility, void *stream) {
    const int rc = check_desc(desc);
    if (rc != PIKV_OK) return rc;
    if (!scores || !slot_coef || !n_valid || !topk_idx || !utility) return PIKV_ERR_INVALID;
    if (k < 1 || k > desc->E) return PIKV_ERR_INVALID;
    if (!(decay >= 0.0f) || decay > 3.0e38f) return PIKV_ERR_INVALID;
    if (desc->B == 0) return PIKV_OK;
    return launch_utility(desc, scores, slot_coef, n_valid, topk_idx, k, decay, utility, false, 0.0f,
                          0, nullptr, nullptr, stream);
}

extern "C" int pikv_update_utility_tracked(const pikv_desc *desc, const float *scores,
                                           const float *slot_coef, const int32_t *n_valid,
                                           const int32_t *topk_idx, int32_t k, float decay,
                                           float *utility, float threshold, int32_t now,
                                           int32_t *last_access, int32_t *freq, void *stream) {
    const int rc = check_desc(desc);
    if (rc != PIKV_OK) return rc;
    if (!scores || !slot_coef || !n_valid || !topk_idx || !last_access || !freq)
        return PIKV_ERR_INVALID;
    if (k < 1 || k > desc->E) return PIKV_ERR_INVALID;
    if (utility && (!(decay >= 0.0f) || decay > 3.0e38f)) return PIKV_ERR_INVALID;
    if (!(threshold >= 0.0f)) return PIKV_ERR_INVALID;
    if (desc->B == 0) return PIKV_OK;
    return launch_utility(desc, scores, slot_coef, n_valid, topk_idx, k, decay, utility, true,
                          threshold, now, last_access, freq, stream);
}
