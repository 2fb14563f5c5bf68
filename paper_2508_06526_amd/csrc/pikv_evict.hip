// PiKV scheduling under bounded memory (Algorithm 1, C <- S(C, q_t); Section 3.4) and the
// constant-time insert (Algorithm 1 Insert; Section 3.1 storage invariants).
//
//   evict_select : one block per (sequence, expert).  The entries to drop are the
//                  n - capacity smallest under (utility ascending, slot descending), i.e.
//                  the complement of the `capacity` best under (utility descending, slot
//                  ascending).  A histogram select over the order-preserving integer image
//                  of the fp32 utilities, held in registers, finds the cut value exactly
//                  (no floating-point comparison is ever redone in a different order),
//                  then one pass in slot order, driven by a block-wide prefix sum of the
//                  per-thread counts, emits the evicted slots ascending and (optionally)
//                  compacts the utilities in place.
//   evict_move   : one block per (shard, kv head, K or V, column slice) slides the kept rows down,
//                  a pass of rows at a time in ascending order (a destination never lies
//                  above its source, so holding a pass in registers before writing it is
//                  enough).
//   append_rows  : one block per (sequence, selected expert) writes the new entry.
#include "pikv_common.h"

namespace pikv {
namespace {

constexpr int kAppendThreads = 256;
// evict_select: 256 threads for shards of up to 2048 slots, 1024 beyond: a thread then owns a quarter of
// the slots, the lists and the compacted utilities leave as runs of 32 bytes per lane instead of 128, and
// four waves a SIMD cover each other's latencies; but a CU holds two such blocks, not eight.  Graph replay, capacity
// 3/4, with a copy of 3 us, 256 and 1024 threads: 64 shards of 1000 slots 8.3 and 8.9 us, of 2000 9.9 and 9.1, of 4096 14.8
// and 10.1; 1024 shards of 1000 10.1 and 25.1, of 2000 14.6 and 26.8, of 4096 24.0 and 29.6.
constexpr int kSelFewSlots = 2048;
constexpr int kSelCache = 32;        // keys a thread can keep in registers (n <= 32768)
constexpr int kSelBins = 1024;       // of a round of the select
constexpr int kSelBinBits = 10;

template <int THREADS>
struct SelShared {
    static constexpr int kWaves = THREADS / kWave;
    int hist[kSelBins];
    uint32_t low[16], high[16];      // per-wave extremes of the keys
    int least[2];                    // keys equal to the range's lower end; two buffers in turn
    int found[2][3];                 // the bin of the cut, the keys below it, the keys in it; two buffers in turn
    int scan[2][16];                 // per-wave totals of a block scan, two buffers in turn
    uint64_t wave_best[kWaves];
};
// The pairs of buffers are used in turn, which makes one barrier per use enough: a buffer
// is rewritten two uses later, and every wave has left the reads of use i before any wave
// passes the barrier of use i+1.

// Sum over the 16 lanes of a DPP row, in every one of them.
__device__ __forceinline__ int row_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true);    // lane ^ 1
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true);    // lane ^ 2
    v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true);   // mirror within 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, true);   // mirror within 16
    return v;
}

// Exclusive prefix sum of v over the block in thread order.
template <int THREADS>
__device__ __forceinline__ int block_scan_excl(int v, SelShared<THREADS> &sh, int &turn) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    // inclusive sums within the rows of 16 lanes, then the rows before (lane 15 of a row to the next, lane 31 to
    // the upper half), without LDS
    int incl = v;
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xf, 0xf, true);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xf, 0xf, true);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xf, 0xf, true);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xf, 0xf, true);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x142, 0xa, 0xf, false);
    incl += __builtin_amdgcn_update_dpp(0, incl, 0x143, 0xc, 0xf, false);
    int *slot = sh.scan[turn & 1];
    ++turn;
    if (lane == kWave - 1) slot[wave] = incl;
    __syncthreads();
    const int before = row_sum((lane & 15) < wave ? slot[lane & 15] : 0);
    return before + incl - v;
}

// Exclusive block-wide rank of a one-bit flag in thread order; *total receives the block sum.
template <int THREADS>
__device__ __forceinline__ int block_rank_flag(bool flag, SelShared<THREADS> &sh, int &turn, int *total) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const uint64_t votes = __ballot(flag);
    const int in_wave = __popcll(votes & ((1ull << lane) - 1ull));
    int *slot = sh.scan[turn & 1];
    ++turn;
    if (lane == 0) slot[wave] = __popcll(votes);
    __syncthreads();
    const int mine = (lane & 15) < SelShared<THREADS>::kWaves ? slot[lane & 15] : 0;
    *total = row_sum(mine);
    return row_sum((lane & 15) < wave ? mine : 0) + in_wave;
}

struct EvictParams {
    float *utility;
    int32_t *n_valid;
    const int32_t *sel_idx;
    int32_t *evicted_idx;
    int32_t *evicted_cnt;
    int E, S, capacity, sel_k, max_evict, compact;
};

// fp32 value whose order_key is `key` (a negative zero comes back as positive zero)
__device__ __forceinline__ float key_value(uint32_t key) {
    return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

// Minimum and maximum over the 64 lanes of a wave, in every lane.
__device__ __forceinline__ void wave_extremes(uint32_t &low, uint32_t &high) {
    auto take = [&](uint32_t l, uint32_t h) {
        low = min(low, l);
        high = max(high, h);
    };
#define PIKV_DPP(v, ctrl) (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(v), ctrl, 0xf, 0xf, true)
    take(PIKV_DPP(low, 0xB1), PIKV_DPP(high, 0xB1));         // lane ^ 1
    take(PIKV_DPP(low, 0x4E), PIKV_DPP(high, 0x4E));         // lane ^ 2
    take(PIKV_DPP(low, 0x141), PIKV_DPP(high, 0x141));       // mirror within 8
    take(PIKV_DPP(low, 0x140), PIKV_DPP(high, 0x140));       // mirror within 16
#undef PIKV_DPP
    auto l = __builtin_amdgcn_permlane16_swap(low, low, false, false), h = __builtin_amdgcn_permlane16_swap(high, high, false, false);
    low = min(l[0], l[1]), high = max(h[0], h[1]);
    l = __builtin_amdgcn_permlane32_swap(low, low, false, false), h = __builtin_amdgcn_permlane32_swap(high, high, false, false);
    low = min(l[0], l[1]), high = max(h[0], h[1]);
}

// The cut of the general case (drop the `ngone` worst of n) is the ngone-th smallest key: keys below it go, and of
// the keys equal to it the first keep_eq in slot order stay.  Rounds of a 1024-bin histogram over the
// range that still holds it - first the smallest to the largest key, then the bin the cut fell into - end
// when a bin is one value wide or goes as a whole.  Utilities spread over their range, so a bin of the first
// round holds a few dozen keys and the second or third ends it.  At most four rounds, of three barriers
// each.  Before, the cut was found two bits at a step, in 16 steps of a barrier and some 20 dependent lane
// and LDS operations (0.5 us each).  Measured (graph replay, capacity 3/4, no rows moved): 16 shards of 8192 slots
// 17.7 -> 10.6 us, 128 of 4096 13.4 -> 7.2, 64 of 1999 10.3 -> 6.9, 64 of 256 8.9 -> 5.1, 16 of 20000 32 -> 24, 8 of 60000
// (read from memory in every round) 218 -> 90; 16 of 8192, 70 % of them zero, 17.9 -> 9.0.
// `each(f)` calls f(key, real) for the thread's keys, in all lanes.
struct Cut {
    uint32_t key;
    int keep_eq;
};
template <int THREADS, class F>
__device__ __forceinline__ Cut find_cut(int ngone, F each, SelShared<THREADS> &sh, int &turn) {
    constexpr int kBins = kSelBins / THREADS;                 // a thread's, in the scan
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    uint32_t low = 0xffffffffu, high = 0;
    each([&](uint32_t key, bool valid) {
        low = min(low, valid ? key : 0xffffffffu);
        high = max(high, valid ? key : 0u);
    });
    wave_extremes(low, high);
    if (lane == 0) sh.low[wave] = low, sh.high[wave] = high;
#pragma unroll
    for (int i = 0; i < kBins; ++i) sh.hist[tid * kBins + i] = 0;
    if (tid == 0) sh.least[0] = 0;
    __syncthreads();
    low = sh.low[min(lane, SelShared<THREADS>::kWaves - 1)];
    high = sh.high[min(lane, SelShared<THREADS>::kWaves - 1)];
    wave_extremes(low, high);
    uint32_t width = high - low;                              // candidates: key - low <= width
    int remaining = ngone;
    for (int round = 0;; ++round) {
        const int bits = width == 0 ? 0 : 32 - __builtin_clz(width);
        const int shift = bits > kSelBinBits ? bits - kSelBinBits : 0;
        // Keys of the range's least value - entries that were never attended have utility zero - are counted by
        // the wave, and when they alone reach the cut it is that value.  (Other values that fill a wave
        // would queue for their bin: a wave that sees that for its first keys lets one lane count for
        // all that share the leader's bin.)
        int seen = 0, least = 0;
        bool crowded = false;
        each([&](uint32_t key, bool valid) {
            const uint32_t x = key - low;
            bool in = valid && x <= width;
            const int bin = (int)(x >> shift);
            least += __popcll(__ballot(in && x == 0));
            in = in && x != 0;
            if (seen++ == 0 || crowded) {
                const uint64_t who = __ballot(in);
                if (who != 0) {
                    const int leader = __builtin_ctzll(who), first = __builtin_amdgcn_readlane(bin, leader);
                    const uint64_t same = __ballot(in && bin == first);
                    crowded = __popcll(same) > 16;
                    if (crowded) {
                        if (lane == leader) atomicAdd(&sh.hist[first], __popcll(same));
                        in = in && bin != first;
                    }
                }
            }
            if (in) atomicAdd(&sh.hist[bin], 1);
        });
        if (lane == 0 && least > 0) {
            atomicAdd(&sh.hist[0], least);
            atomicAdd(&sh.least[round & 1], least);
        }
        __syncthreads();
        least = sh.least[round & 1];
        if (remaining <= least) return Cut{low, least - remaining};          // (the same in the whole block)
        if (tid == 0) sh.least[(round & 1) ^ 1] = 0;
        int count[kBins], sum = 0;
#pragma unroll
        for (int i = 0; i < kBins; ++i) {
            count[i] = sh.hist[tid * kBins + i];
            sum += count[i];
        }
        int below = block_scan_excl(sum, sh, turn);
        int *found = sh.found[round & 1];
        if (below < remaining && remaining <= below + sum) {
#pragma unroll
            for (int i = 0; i < kBins; ++i) {
                if (below < remaining && remaining <= below + count[i])
                    found[0] = tid * kBins + i, found[1] = below, found[2] = count[i];
                below += count[i];
            }
        }
#pragma unroll
        for (int i = 0; i < kBins; ++i) sh.hist[tid * kBins + i] = 0;     // (its own bins only)
        __syncthreads();
        const uint32_t offset = (uint32_t)found[0] << shift;
        remaining -= found[1];
        const int cand = found[2];
        low += offset;
        width = min(width - offset, (1u << shift) - 1u);
        if (shift == 0) return Cut{low, cand - remaining};
        if (remaining == cand) return Cut{low + width, 0};
    }
}

// Keys in registers: thread t owns the `per` consecutive slots from t * per (per a multiple
// of 4, at most NCH), so the rounds touch no memory and slot order is thread order.
template <int THREADS, int NCH>
__device__ __forceinline__ void select_cached(const EvictParams &p, int be, float *u, int n,
                                              int ngone, bool vec, SelShared<THREADS> &sh) {
    const int tid = threadIdx.x;
    const int per = (n + THREADS * 4 - 1) / (THREADS * 4) * 4;
    const int first = tid * per;
    // vec: the row is 16-byte aligned and S is a multiple of 4, so a group of four that starts
    // below n lies inside the row; groups past n re-read the first one.  Otherwise single slots,
    // clamped onto the last.  No branch around the loads: all of them are in flight together.
    uint32_t keys[NCH];
#pragma unroll
    for (int j0 = 0; j0 < NCH; j0 += 4) {
        const int i0 = first + j0;
        const bool any = j0 < per && i0 < n;
        const float4 v = vec ? *reinterpret_cast<const float4 *>(u + (any ? i0 : 0))
                             : make_float4(u[min(i0, n - 1)], u[min(i0 + 1, n - 1)], u[min(i0 + 2, n - 1)],
                                           u[min(i0 + 3, n - 1)]);
        keys[j0] = any ? order_key(v.x) : 0xffffffffu;
        keys[j0 + 1] = (any && i0 + 1 < n) ? order_key(v.y) : 0xffffffffu;
        keys[j0 + 2] = (any && i0 + 2 < n) ? order_key(v.z) : 0xffffffffu;
        keys[j0 + 3] = (any && i0 + 3 < n) ? order_key(v.w) : 0xffffffffu;
    }
    int turn = 0;
    const Cut found = find_cut<THREADS>(ngone, [&](auto take) {
#pragma unroll
        for (int j = 0; j < NCH; ++j)
            if (j < per) take(keys[j], first + j < n);
    }, sh, turn);
    const uint32_t cut = found.key;               // keys < cut go; of the keys == cut
    const int keep_eq = found.keep_eq;            // the first keep_eq in slot order stay

    constexpr int kWords = (NCH + 31) / 32;
    uint32_t gone[kWords];
#pragma unroll
    for (int w = 0; w < kWords; ++w) gone[w] = 0;
    int n_eq = 0, n_gone = 0;
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
        const bool valid = j < per && first + j < n;
        const bool g = valid && (keys[j] < cut || (keep_eq == 0 && keys[j] == cut));
        gone[j >> 5] |= (g ? 1u : 0u) << (j & 31);
        n_gone += g;
        n_eq += valid && keys[j] == cut;
    }
    if (keep_eq > 0) {                            // ties at the cut: the earliest keep_eq stay
        int eq_rank = block_scan_excl(n_eq, sh, turn);
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
            const bool valid = j < per && first + j < n;
            if (valid && keys[j] == cut) {
                if (eq_rank >= keep_eq) {
                    gone[j >> 5] |= 1u << (j & 31);
                    ++n_gone;
                }
                ++eq_rank;
            }
        }
    }
    int rank = block_scan_excl(n_gone, sh, turn);   // evicted slots before my first slot
    int32_t *out = p.evicted_idx + (int64_t)be * p.max_evict;
    // In-place compaction is safe here: every utility is already held as a key.
#pragma unroll
    for (int j0 = 0; j0 < NCH; j0 += 4) {
        if (j0 < per) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int j = j0 + t, i = first + j;
                if (i < n) {
                    if ((gone[j >> 5] >> (j & 31)) & 1u) {
                        if (rank < p.max_evict) out[rank] = i;
                        ++rank;
                    } else if (p.compact && rank > 0) {
                        u[i - rank] = key_value(keys[j]);
                    }
                }
            }
        }
    }
}

// More keys than the registers hold: every round re-reads them (slot i = tid + j * THREADS).
template <int THREADS>
__device__ __forceinline__ void select_stream(const EvictParams &p, int be, float *u, int n,
                                              int ngone, SelShared<THREADS> &sh) {
    const int tid = threadIdx.x;
    const int nchunk = (n + THREADS - 1) / THREADS;
    int turn = 0;
    const Cut found = find_cut<THREADS>(ngone, [&](auto take) {
        for (int j = 0; j < nchunk; ++j) {
            const int i = tid + j * THREADS;
            take(i < n ? order_key(u[i]) : 0u, i < n);
        }
    }, sh, turn);
    const uint32_t cut = found.key;
    const int keep_eq = found.keep_eq;
    int32_t *out = p.evicted_idx + (int64_t)be * p.max_evict;
    int eq_seen = 0, gone_seen = 0;       // running totals over the chunks already done
    for (int j = 0; j < nchunk; ++j) {
        const int i = tid + j * THREADS;
        const bool valid = i < n;
        const float ui = valid ? u[i] : 0.0f;
        const uint32_t key = order_key(ui);
        const bool is_eq = valid && key == cut, is_less = valid && key < cut;
        int eq_total, gone_total;
        const int eq_rank = eq_seen + block_rank_flag(is_eq, sh, turn, &eq_total);
        const bool gone = is_less || (is_eq && eq_rank >= keep_eq);
        const int gone_before = gone_seen + block_rank_flag(gone, sh, turn, &gone_total);
        if (valid) {
            if (gone) {
                if (gone_before < p.max_evict) out[gone_before] = i;
            } else if (p.compact && gone_before > 0) {
                u[i - gone_before] = ui;  // this chunk's reads ended before the barriers above
            }
        }
        eq_seen += eq_total;
        gone_seen += gone_total;
    }
}

template <int THREADS>
__global__ __launch_bounds__(THREADS) void evict_select(EvictParams p) {
    const int be = blockIdx.x;
    const int b = be / p.E, e = be - b * p.E;
    const int tid = threadIdx.x;

    __shared__ SelShared<THREADS> sh;

    bool selected = true;
    if (p.sel_idx) {
        selected = false;
        for (int j = 0; j < p.sel_k; ++j) selected |= (p.sel_idx[(int64_t)b * p.sel_k + j] == e);
    }
    const int n = p.n_valid[be];
    const int ngone = n - p.capacity;
    if (!selected || ngone <= 0 || ngone > p.max_evict) {
        if (tid == 0) p.evicted_cnt[be] = (selected && ngone > p.max_evict) ? -1 : 0;
        return;
    }
    float *u = p.utility + (int64_t)be * p.S;

    if (ngone == 1 && !p.compact) {
        // Streaming case: drop the single worst entry = minimum of (key, then largest slot).
        // One composite 64-bit value per entry orders both at once.
        uint64_t best = ~0ull;
        const int n4 = (p.S % 4 == 0) ? (n / 4) * 4 : 0;   // float4 reads need aligned rows
        for (int i = tid * 4; i < n4; i += THREADS * 4) {
            const float4 v = *reinterpret_cast<const float4 *>(u + i);
            const uint64_t c0 = evict_composite(v.x, i), c1 = evict_composite(v.y, i + 1);
            const uint64_t c2 = evict_composite(v.z, i + 2), c3 = evict_composite(v.w, i + 3);
            const uint64_t a = c0 < c1 ? c0 : c1, b2 = c2 < c3 ? c2 : c3;
            const uint64_t c = a < b2 ? a : b2;
            best = c < best ? c : best;
        }
        for (int i = n4 + tid; i < n; i += THREADS) {
            const uint64_t c = evict_composite(u[i], i);
            best = c < best ? c : best;
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const uint64_t o = __shfl_xor(best, off, kWave);
            best = o < best ? o : best;
        }
        if ((tid & (kWave - 1)) == 0) sh.wave_best[tid >> 6] = best;
        __syncthreads();
        if (tid == 0) {
            uint64_t m = sh.wave_best[0];
#pragma unroll
            for (int w = 1; w < THREADS / kWave; ++w) m = sh.wave_best[w] < m ? sh.wave_best[w] : m;
            p.evicted_idx[(int64_t)be * p.max_evict] = evict_composite_slot(m);
            p.evicted_cnt[be] = 1;
            p.n_valid[be] = p.capacity;
        }
        return;
    }

    // keys held per thread: the next size that covers n; beyond the largest, re-read in every round
    const bool vec = p.S % 4 == 0 && (reinterpret_cast<uintptr_t>(p.utility) & 15) == 0;
    if constexpr (THREADS == 256) {
        select_cached<THREADS, 8>(p, be, u, n, ngone, vec, sh);         // S <= kSelFewSlots
    } else if (n <= kSelFewSlots) {
        // Few entries in a large shard: as a small one.  (A barrier waits for the waves that are left.)
        __shared__ SelShared<256> few;
        if (tid >= 256) return;
        select_cached<256, 8>(p, be, u, n, ngone, vec, few);
    } else if (n <= 8 * THREADS) {
        select_cached<THREADS, 8>(p, be, u, n, ngone, vec, sh);
    } else if (n <= kSelCache * THREADS) {
        select_cached<THREADS, kSelCache>(p, be, u, n, ngone, vec, sh);
    } else {
        select_stream<THREADS>(p, be, u, n, ngone, sh);
    }
    if (tid == 0) {
        p.evicted_cnt[be] = ngone;
        p.n_valid[be] = p.capacity;
    }
}

struct MoveParams {
    void *const *K;
    void *const *V;
    const int32_t *n_valid;
    const int32_t *evicted_idx;
    const int32_t *evicted_cnt;
    int64_t stride_h_bytes, stride_s_bytes;
    int row_chunks;      // 16-byte chunks of a row that one block moves, a power of two up to 256
    int max_evict;
};

constexpr int kMaxRowChunks = 256;
constexpr int kMoveThreads = 1024;       // at most; 256 for shards of few slots (kMoveFewSlots) ...
constexpr int kMoveFewSlots = 1024;
constexpr int kMoveManyBlocks = 2048;    // ... or of one pass in this many blocks
constexpr int kMoveRows = 4;             // rows a thread carries per pass
constexpr int kMoveList = 8192;          // evicted slots of a shard kept in LDS (more: read from memory)
inline __host__ __device__ int move_pass_rows(int threads, int row_chunks) { return threads / row_chunks * kMoveRows; }
inline size_t move_lds_bytes(int threads, int row_chunks, int max_evict) {
    return ((size_t)2 * move_pass_rows(threads, row_chunks) + (max_evict < kMoveList ? max_evict : kMoveList)) * sizeof(int);
}

// Slides the kept rows of one (shard, kv head, K or V, column slice) down, a pass of destination
// rows at a time in ascending order.  Destination d takes the d-th kept slot, d + (how many evicted
// slots lie below it), found by binary search in the ascending list, one thread per row, while the
// rows of the pass before are on their way.  A pass's sources lie at or above its first destination:
// the rows of a pass can be requested before those of the pass before are written, so a block
// always has a pass of loads in flight; only the writes of a pass wait (a barrier) until the whole
// block holds its rows.  What bounded the form before - 256 threads, every pass a chain of four
// barriers and a trip to memory - were those chains (5 us per 256 rows).  Measured, 16 shards x 8
// heads, 8192 -> 6144 rows of 256 bytes: 161 -> 140 us (5.75 TB/s of
// reads and writes).
template <bool STREAM>
__global__ __launch_bounds__(kMoveThreads) void evict_move(MoveParams p) {
    // blockIdx.z: bit 0 picks K or V, the rest picks the column slice of the row
    const int be = blockIdx.x, hk = blockIdx.y;
    const bool is_v = blockIdx.z & 1;
    const int slice = blockIdx.z >> 1;
    const int tid = threadIdx.x, threads = blockDim.x;
    const int cnt = p.evicted_cnt[be];
    if (cnt <= 0) return;
    const int n_new = p.n_valid[be];
    const int32_t *gone = p.evicted_idx + (int64_t)be * p.max_evict;
    const int first = gone[0];               // rows below it stay
    if (first >= n_new) return;

    extern __shared__ int move_lds[];        // two tables of source rows, used in turn, and the list
    const int pass_rows = move_pass_rows(threads, p.row_chunks);
    const int list = 2 * pass_rows;
    const bool cached = cnt <= kMoveList;
    if (cached) {
        for (int i = tid; i < cnt; i += threads) move_lds[list + i] = gone[i] - i;   // kept slots below it
        __syncthreads();
    }
    auto fill = [&](int table, int base) {
        for (int x = tid; x < pass_rows; x += threads) {
            const int d = base + x;
            int lo = 0, hi = d < n_new ? cnt : 0;    // evicted slots below the d-th kept one
            if (cached) {
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (move_lds[list + mid] <= d) lo = mid + 1;
                    else hi = mid;
                }
            } else {
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (gone[mid] - mid <= d) lo = mid + 1;
                    else hi = mid;
                }
            }
            move_lds[table + x] = d < n_new ? d + lo : first;        // every entry is a row of the shard
        }
    };
    const int rsub = tid / p.row_chunks, csub = tid & (p.row_chunks - 1);
    const int group_rows = threads / p.row_chunks;      // rows covered by one sweep of the block
    char *Xb = static_cast<char *>(is_v ? p.V[be] : p.K[be]) + hk * p.stride_h_bytes +
               (slice * p.row_chunks + csub) * 16;
    struct Rows {
        uint4 v[kMoveRows];
    };
    auto load = [&](Rows &to, int table) {
        int row[kMoveRows];
#pragma unroll
        for (int r = 0; r < kMoveRows; ++r) row[r] = move_lds[table + r * group_rows + rsub];
#pragma unroll
        for (int r = 0; r < kMoveRows; ++r) {
            const char *from = Xb + row[r] * p.stride_s_bytes;
            to.v[r] = STREAM ? load16_stream(from) : load16(from);
        }
    };
    auto store = [&](char *to, const uint4 &v) {
        if (STREAM) store16_stream(to, v);
        else store16(to, v);
    };
    Rows rows[2];
    int base = first;
    // one pass: the next pass's rows are requested, this pass's written.  Nothing in it is
    // conditional, so a wait for rows is never a wait for the writes after them.
    auto pass = [&](Rows &cur, Rows &next, int next_table) {
        fill(next_table, base + pass_rows);
#pragma unroll
        for (int r = 0; r < kMoveRows; ++r)  // this wave's rows are here ...
            asm volatile("" : "+v"(cur.v[r].x), "+v"(cur.v[r].y), "+v"(cur.v[r].z), "+v"(cur.v[r].w));
        __syncthreads();                     // ... and so are the block's
        load(next, next_table);
#pragma unroll
        for (int r = 0; r < kMoveRows; ++r)
            store(Xb + (base + r * group_rows + rsub) * p.stride_s_bytes, cur.v[r]);
        base += pass_rows;
    };
    auto last = [&](Rows &cur) {             // a partial pass
#pragma unroll
        for (int r = 0; r < kMoveRows; ++r)
            asm volatile("" : "+v"(cur.v[r].x), "+v"(cur.v[r].y), "+v"(cur.v[r].z), "+v"(cur.v[r].w));
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kMoveRows; ++r) {
            const int d = base + r * group_rows + rsub;
            if (d < n_new) store(Xb + d * p.stride_s_bytes, cur.v[r]);
        }
    };
    fill(0, base);
    __syncthreads();
    load(rows[0], 0);
    while (base + 2 * pass_rows <= n_new) {
        pass(rows[0], rows[1], pass_rows);
        pass(rows[1], rows[0], 0);
    }
    if (base + pass_rows <= n_new) {
        pass(rows[0], rows[1], pass_rows);
        if (base < n_new) last(rows[1]);
    } else if (base < n_new) {
        last(rows[0]);
    }
}

struct AppendParams {
    const void *K_new;
    const void *V_new;
    const int32_t *topk;
    const int32_t *reuse_idx;
    const int32_t *reuse_cnt;
    void *const *K;
    void *const *V;
    float *utility;
    int32_t *n_valid;
    int64_t stride_h_bytes, stride_s_bytes;
    FastDiv by_k;
    int E, S, Hkv, k, row_chunks, row_bits, max_evict;      // chunks of a row: a power of two
};

// Two trips to memory: lane e of every wave takes shard e's count, reusable slot and addresses beside the
// selection, which picks among them, and the new rows come with those; then the writes.  (One after the other - selection, count,
// slot, addresses, rows - a block was four trips: kernel trace 2.95 -> 2.6 us for 12 rows of 4 fp32 heads, 3.25 -> 2.65 for 9.)
__global__ __launch_bounds__(kAppendThreads) void append_rows(AppendParams p) {
    int j;
    const int b = fast_divide(p.by_k, blockIdx.x, &j);
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int64_t be0 = (int64_t)b * p.E, be_lane = be0 + min(lane, p.E - 1);
    const int sel = p.topk[(int64_t)b * p.k + min(lane, p.k - 1)];
    const int n_lane = p.n_valid[be_lane];
    const uint64_t K_lane = reinterpret_cast<uint64_t>(p.K[be_lane]), V_lane = reinterpret_cast<uint64_t>(p.V[be_lane]);
    int cnt_lane = 0, idx_lane = 0;
    if (p.reuse_cnt) {                       // block-uniform
        cnt_lane = p.reuse_cnt[be_lane];
        idx_lane = p.reuse_idx[be_lane * p.max_evict];
    }
    const int total = p.Hkv * p.row_chunks;
    const char *Ks = static_cast<const char *>(p.K_new) + (int64_t)b * total * 16;
    const char *Vs = static_cast<const char *>(p.V_new) + (int64_t)b * total * 16;
    const int first = min(tid, total - 1);
    uint4 kv = load16(Ks + (int64_t)first * 16), vv = load16(Vs + (int64_t)first * 16);
    const int e = __builtin_amdgcn_readlane(sel, j);
    const int n = __builtin_amdgcn_readlane(n_lane, e);
    int slot = n;
    if (__builtin_amdgcn_readlane(cnt_lane, e) > 0) slot = __builtin_amdgcn_readlane(idx_lane, e);
    __syncthreads();                         // every thread has read n before it changes
    if (n >= p.S || slot < 0 || slot >= p.S) return;   // full shard: the entry is dropped
    auto address = [&](uint64_t of_lane) {
        const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)of_lane, e), hi = __builtin_amdgcn_readlane((int)(uint32_t)(of_lane >> 32), e);
        return reinterpret_cast<char *>(((uint64_t)hi << 32) | lo) + slot * p.stride_s_bytes;
    };
    char *Kd = address(K_lane), *Vd = address(V_lane);
    for (int idx = tid; idx < total; idx += kAppendThreads) {
        if (idx != tid) {
            kv = load16(Ks + (int64_t)idx * 16);
            vv = load16(Vs + (int64_t)idx * 16);
        }
        const int hk = idx >> p.row_bits, cc = idx & (p.row_chunks - 1);
        store16(Kd + hk * p.stride_h_bytes + cc * 16, kv);
        store16(Vd + hk * p.stride_h_bytes + cc * 16, vv);
    }
    if (tid == 0) {
        p.utility[(be0 + e) * p.S + slot] = 0.0f;
        p.n_valid[be0 + e] = n + 1;
    }
}

}  // namespace
}  // namespace pikv

using namespace pikv;

extern "C" int pikv_evict(const pikv_desc *desc, float *utility, int32_t *n_valid,
                          int32_t capacity, const int32_t *sel_idx, int32_t sel_k,
                          int32_t *evicted_idx, int32_t *evicted_cnt, int32_t max_evict,
                          int32_t compact, void *const *K_shards, void *const *V_shards,
                          void *stream) {
    const int rc = check_desc(desc);
    if (rc != PIKV_OK) return rc;
    if (!utility || !n_valid || !evicted_idx || !evicted_cnt) return PIKV_ERR_INVALID;
    if (capacity < 0 || max_evict < 1) return PIKV_ERR_INVALID;
    if (sel_idx && (sel_k < 1 || sel_k > desc->E)) return PIKV_ERR_INVALID;
    if (compact && (!K_shards || !V_shards)) return PIKV_ERR_INVALID;
    if (desc->B == 0) return PIKV_OK;
    const int row_chunks = desc_width(desc) * elem_bytes(desc->dtype) / 16;
    if (compact && (row_chunks < 1 || row_chunks > kMaxRowChunks)) return PIKV_ERR_UNSUPPORTED;
    hipStream_t st = as_stream(stream);
    EvictParams p;
    p.utility = utility;
    p.n_valid = n_valid;
    p.sel_idx = sel_idx;
    p.evicted_idx = evicted_idx;
    p.evicted_cnt = evicted_cnt;
    p.E = desc->E;
    p.S = desc->S;
    p.capacity = capacity;
    p.sel_k = sel_k;
    p.max_evict = max_evict;
    p.compact = compact ? 1 : 0;
    const dim3 shards(desc->B * desc->E);
    if (desc->S <= kSelFewSlots) hipLaunchKernelGGL(evict_select<256>, shards, dim3(256), 0, st, p);
    else hipLaunchKernelGGL(evict_select<1024>, shards, dim3(1024), 0, st, p);
    int lrc = launch_status();
    if (lrc != PIKV_OK || !compact) return lrc;
    MoveParams m;
    m.K = K_shards;
    m.V = V_shards;
    m.n_valid = n_valid;
    m.evicted_idx = evicted_idx;
    m.evicted_cnt = evicted_cnt;
    const int eb = elem_bytes(desc->dtype);
    m.stride_h_bytes = desc->stride_h * eb;
    m.stride_s_bytes = desc->stride_s * eb;
    // K and V move in separate blocks; rows are cut in column slices of whole 128-byte lines until there
    // are two blocks per CU (64-byte slices, two blocks on a line, cost 10 shards x 8 heads of 8192 rows
    // 131 -> 157 us), and of 64 bytes only to reach half the CUs (2 shards x 4 heads of 32768 rows 161 -> 147).
    const int64_t uncut = (int64_t)desc->B * desc->E * desc->Hkv * 2;
    int slices = 1;
    while (uncut * slices < 512 && row_chunks / slices >= 16) slices *= 2;
    while (uncut * slices < 128 && row_chunks / slices >= 8) slices *= 2;
    m.row_chunks = row_chunks / slices;
    m.max_evict = max_evict;
    // 1024 threads shorten the chain of passes; 256 where there is none: in small shards, and in those of
    // one pass with blocks enough to fill the chip (512 shards x 8 heads of 1108 rows of 32 bytes, 32 of the
    // shards selected, 92 -> 52 us: the blocks of the others only start and leave).
    const bool few = desc->S <= kMoveFewSlots ||
                     (uncut * slices >= kMoveManyBlocks && desc->S <= move_pass_rows(kMoveThreads, m.row_chunks));
    const int threads = few ? 256 : kMoveThreads;
    const dim3 grid(desc->B * desc->E, desc->Hkv, 2 * slices), block(threads);
    const size_t lds = move_lds_bytes(threads, m.row_chunks, max_evict);
    // From 512 MiB on, twice what the Infinity Cache holds, reads and writes go past it (512 MiB: 161 us
    // for the whole call against 187, 4 GiB 556 against 639).  Below, what a call moves may still be in it,
    // and half of it is where one entry leaves each shard (319 MB 61 us against 86, 470 MB 87 against 122).  Only
    // the shards that the call processes count.
    const int64_t shards_moved = (int64_t)desc->B * (sel_idx && sel_k < desc->E ? sel_k : desc->E);
    const int64_t cache_bytes = shards_moved * desc->Hkv * desc->S * row_chunks * 32;
    if (cache_bytes >= ((int64_t)512 << 20)) hipLaunchKernelGGL(evict_move<true>, grid, block, lds, st, m);
    else hipLaunchKernelGGL(evict_move<false>, grid, block, lds, st, m);
    return launch_status();
}

extern "C" int pikv_append(const pikv_desc *desc, const void *K_new, const void *V_new,
                           const int32_t *topk_idx, int32_t k, const int32_t *reuse_idx,
                           const int32_t *reuse_cnt, int32_t max_evict, void *const *K_shards,
                           void *const *V_shards, float *utility, int32_t *n_valid,
                           void *stream) {
    const int rc = check_desc(desc);
    if (rc != PIKV_OK) return rc;
    if (!K_new || !V_new || !topk_idx || !K_shards || !V_shards || !utility || !n_valid)
        return PIKV_ERR_INVALID;
    if (k < 1 || k > desc->E) return PIKV_ERR_INVALID;
    if ((reuse_idx == nullptr) != (reuse_cnt == nullptr)) return PIKV_ERR_INVALID;
    if (reuse_idx && max_evict < 1) return PIKV_ERR_INVALID;
    if (desc->B == 0) return PIKV_OK;
    AppendParams p;
    p.K_new = K_new;
    p.V_new = V_new;
    p.topk = topk_idx;
    p.reuse_idx = reuse_idx;
    p.reuse_cnt = reuse_cnt;
    p.K = K_shards;
    p.V = V_shards;
    p.utility = utility;
    p.n_valid = n_valid;
    const int eb = elem_bytes(desc->dtype);
    p.stride_h_bytes = desc->stride_h * eb;
    p.stride_s_bytes = desc->stride_s * eb;
    p.E = desc->E;
    p.S = desc->S;
    p.Hkv = desc->Hkv;
    p.k = k;
    p.by_k = fast_div(k);
    p.row_chunks = desc_width(desc) * eb / 16;
    p.row_bits = __builtin_ctz(p.row_chunks);
    p.max_evict = max_evict;
    hipLaunchKernelGGL(append_rows, dim3(desc->B * k), dim3(kAppendThreads), 0, as_stream(stream),
                       p);
    return launch_status();
}
