// One decode step of PiKV's hot path as three launches (Algorithm 1, one iteration of the
// loop: route, insert the new entry under bounded memory, attend, score):
//
//   step_pre   : per (sequence, selected position), a 1024-thread block routes the query
//                (Section 3.2), then for its selected shard evicts the minimum-utility entry
//                if the shard is full (Section 3.4) and inserts the new token's K/V rows in
//                O(1) (Section 3.1).  Everything that depends only on the selected expert id
//                (entry count, table pointers, the shard's utilities) is fetched in one round
//                trip; the new rows are fetched before the router result exists.
//   attention  : the split flash-decode pass over the selected shards (pikv_attn.hip).
//   step_post  : merge of the split partials with the router gates and the utility update
//                u <- decay * u + attention mass (Section 3.4, Table 3 H2O), in one launch
//                (two with many (head, shard) pairs: post_separate).
//
// With a scheduling policy (Table 3 rows SL, LRU, LRU+) step_pre takes its minimum over the
// policy's value, computed on the fly from the per-entry stamps and counts, and stamps the
// new entry; step_post marks the entries whose attention mass exceeds the access threshold.
//
// On MI355X even an empty kernel occupies the queue for ~1.5 us and each small kernel is a
// chain of dependent memory round trips; six launches cost more in dispatch and latency than
// in work next to a ~20 us attention pass.  The step is defined as exactly the sequence of
// the separate C-ABI calls and shares every reduction order with them (bit-identical).
#include "pikv_common.h"
#include "pikv_combine_dev.h"
#include "pikv_route_dev.h"
#include "pikv_policy_dev.h"
#include "pikv_penalty_dev.h"

namespace pikv {
namespace {

struct PreParams {
    const void *x;
    const void *W_r;
    const float *bias;
    int32_t *topk;
    float *gates;
    const void *K_new;
    const void *V_new;
    void *const *K;
    void *const *V;
    float *utility;
    int32_t *n_valid;
    int32_t *evicted_idx;
    int32_t *evicted_cnt;
    int64_t stride_h_bytes, stride_s_bytes;
    int64_t x_stride;    // elements between the routed vectors of consecutive sequences (>= d_r)
    int d_r, E, cpr, k, S, Hkv, row_chunks, row_bits, do_insert;   // chunks of a row: a power of two
    int flat_threads;    // fp32: 0 where rows of W_r are cpr aligned chunks, < 0 for single elements, else the threads of the flat form
    bool w_aligned;      // ... and whether W_r is 16-byte aligned
    bool words;          // bf16: see route_words_ok
    FastDiv by_k;
    int use_policy;      // the entry to evict is chosen by pol (Table 3) instead of the utility
    PolicyView pol;      // its arrays, when given, are also stamped for the new entry
};

// Minimum of a 64-bit key over the wavefront, every lane ends with it; the four low lane bits
// are exchanged inside the 16-lane rows (no LDS traffic).
__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v) {
    auto step = [&](auto bit) {
        constexpr int BIT = decltype(bit)::value;
        const uint32_t lo = __float_as_uint(lane_xchg<BIT>(__uint_as_float((uint32_t)v)));
        const uint32_t hi = __float_as_uint(lane_xchg<BIT>(__uint_as_float((uint32_t)(v >> 32))));
        const uint64_t o = ((uint64_t)hi << 32) | lo;
        v = o < v ? o : v;
    };
    step(std::integral_constant<int, 0>{});
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 3>{});
    step(std::integral_constant<int, 4>{});
    step(std::integral_constant<int, 5>{});
    return v;
}

// Grid: (sequence b, selected position j).  Every block of a sequence recomputes the routing
// decision (W_r is L2-resident and tiny next to the cache) so that the k evict/insert jobs
// run on k compute units at once instead of one after the other; block j == 0 publishes the
// decision.
// MOST: bf16, the router's experts at most (RouteTiles); 0 for fp32.
template <typename T, int MOST>
__global__ __launch_bounds__(kRouteThreads) void step_pre(PreParams p) {
    constexpr int kWaves = kRouteThreads / kWave;
    int j;
    const int b = fast_divide(p.by_k, blockIdx.x, &j);
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = tid >> 6;

    __shared__ uint64_t wave_best[kWaves];

    // neither the router's additive term, nor the entry counts of the sequence's shards (lane e
    // takes shard e's; the selected one is picked out of the register once the router has
    // spoken), nor the new rows depend on anything: requested now (the rows behind the router's sums for more than
    // 32 experts, which leave no registers for them: 20 bytes of scratch a lane)
    const float bias_e = route_bias_of_lane(p.bias, p.E, lane);
    const int n_of_lane = p.n_valid[(int64_t)b * p.E + min(lane, p.E - 1)];
    const int new_chunks = p.Hkv * p.row_chunks;
    uint4 knew = make_uint4(0, 0, 0, 0), vnew = knew;
    auto request_new = [&]() {
        if (p.do_insert && tid < new_chunks) {
            knew = load16(static_cast<const char *>(p.K_new) + ((int64_t)b * new_chunks + tid) * 16);
            vnew = load16(static_cast<const char *>(p.V_new) + ((int64_t)b * new_chunks + tid) * 16);
        }
    };
    if constexpr (MOST < 64) request_new();

    const T *xr = static_cast<const T *>(p.x) + (int64_t)b * p.x_stride;
    const T *W_r = static_cast<const T *>(p.W_r);
    float logit = 0.0f;                      // of expert `lane`, in the first wave
    if constexpr (MOST > 0) {
        __shared__ RouteShared<MOST, 1> sh;
        logit = route_logit_mfma<MOST>(xr, W_r, p.d_r, p.E, p.words, bias_e, sh);
        if constexpr (MOST == 64) request_new();
    } else {
        __shared__ float red[kWaves][64];
        __shared__ __attribute__((aligned(16))) float flat[kFlatFloats];
        if (p.flat_threads == 0) route_logits_vec(xr, W_r, p.d_r, p.cpr, red);
        else if (p.flat_threads < 0) route_logits_single<1>({xr}, W_r, p.d_r, p.E, route_flat_pow2(p.E), flat);
        else route_logits_flat(xr, W_r, p.d_r, p.E, p.flat_threads, p.w_aligned, flat, red);
        if (wave == 0)
            logit = p.flat_threads < 0 ? route_logit_single_of_lane(flat, bias_e, p.E, lane) : route_logit_of_lane(red[0], 64, bias_e, p.E, lane);
    }
    // The first wave ranks the experts and tells the others which shard is the block's (one LDS
    // word and a barrier): sixteen waves doing it side by side, four to a SIMD, take twice as
    // long as one wave alone plus the barrier.  The ranks come first - the shard to scan hangs
    // off them alone - and the softmax and the gates are formed, by that wave of the sequence's
    // first block, while the scan's requests are in flight.
    __shared__ int block_expert;
    int rank = 64;
    if (wave == 0) {
        rank = route_rank(logit, lane, p.E);
        const uint64_t owner = __ballot(rank == j);      // taken with every lane of the wave active
        if (lane == 0) block_expert = __builtin_ctzll(owner);
    }
    auto publish = [&]() {
        if (j == 0 && wave == 0) route_gates(logit, rank, lane, b, p.E, p.k, p.topk, p.gates, nullptr);
    };
    if (!p.do_insert) {
        publish();
        return;
    }
    __syncthreads();
    const int e = __builtin_amdgcn_readfirstlane(block_expert);
    const int n = __builtin_amdgcn_readlane(n_of_lane, e);
    const int64_t be = (int64_t)b * p.E + e;
    char *Kd = static_cast<char *>(p.K[be]);
    char *Vd = static_cast<char *>(p.V[be]);
    const float *u = p.utility + be * p.S;
    uint64_t best = ~0ull;
    if (p.use_policy) {
        publish();
        if (policy_vec_ok(p.pol, p.utility, p.S)) {
            for (int i = tid * 4; i < p.S; i += kRouteThreads * 4) {
                float v[4];
                policy_value4(p.pol, be * p.S + i, p.utility, v);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint64_t c0 = evict_composite(v[t], i + t);
                    best = c0 < best ? c0 : best;
                }
            }
        } else {
            for (int i = tid; i < p.S; i += kRouteThreads) {
                const uint64_t c0 = evict_composite(policy_value(p.pol, be * p.S + i, p.utility), i);
                best = c0 < best ? c0 : best;
            }
        }
    } else if ((p.S & 3) == 0) {
        // two 16-byte loads per thread and pass, both requested before either is used: up to
        // 8192 slots are one trip to memory, not one per 4096
        // (the first pass's requests are in flight while the gates are formed and published)
        constexpr int kScanLoads = 2;
        float4 v[kScanLoads];
        auto request = [&](int i0) {
#pragma unroll
            for (int t = 0; t < kScanLoads; ++t) {
                const int i = i0 + t * kRouteThreads * 4;
                v[t] = i < p.S ? *reinterpret_cast<const float4 *>(u + i) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        };
        request(tid * 4);
        publish();
        for (int i0 = tid * 4; i0 < p.S; i0 += kRouteThreads * 4 * kScanLoads) {
            if (i0 != tid * 4) request(i0);
            // The block's 16 waves share 4 vector units, so this phase costs its instruction
            // count times 16 cycles.  Where no value of the wave has its sign bit set (utilities
            // are sums of probabilities), the keys' order is the order of the raw bits and the
            // thread's slots ascend: one compare and two selects per value ("<=": of equal
            // values the higher slot goes) instead of building and comparing 64-bit composites
            // - the same minimum.  (Loads past the shard's end hold zeros and are left out; the
            // thread's first load is always inside.)
            uint32_t signs = 0;
#pragma unroll
            for (int t = 0; t < kScanLoads; ++t)
                signs |= (__float_as_uint(v[t].x) | __float_as_uint(v[t].y)) |
                         (__float_as_uint(v[t].z) | __float_as_uint(v[t].w));
            if (!__any((int)signs < 0)) {
                uint32_t low = 0xffffffffu;
                int at = 0;              // offset of the lowest value's slot from i0
                auto take = [&](bool inside, float value, int offset) {
                    const uint32_t bits = __float_as_uint(value);
                    const bool le = inside && bits <= low;
                    low = le ? bits : low;
                    at = le ? offset : at;
                };
#pragma unroll
                for (int t = 0; t < kScanLoads; ++t) {
                    const bool inside = i0 + t * kRouteThreads * 4 < p.S;
                    take(inside, v[t].x, t * kRouteThreads * 4);
                    take(inside, v[t].y, t * kRouteThreads * 4 + 1);
                    take(inside, v[t].z, t * kRouteThreads * 4 + 2);
                    take(inside, v[t].w, t * kRouteThreads * 4 + 3);
                }
                const uint64_t c0 = evict_composite(__uint_as_float(low), i0 + at);
                best = c0 < best ? c0 : best;
                continue;
            }
#pragma unroll
            for (int t = 0; t < kScanLoads; ++t) {
                const int i = i0 + t * kRouteThreads * 4;
                if (i < p.S) {
                    uint64_t c0 = evict_composite(v[t].x, i), c1 = evict_composite(v[t].y, i + 1);
                    uint64_t c2 = evict_composite(v[t].z, i + 2), c3 = evict_composite(v[t].w, i + 3);
                    c0 = c0 < c1 ? c0 : c1;
                    c2 = c2 < c3 ? c2 : c3;
                    c0 = c0 < c2 ? c0 : c2;
                    best = c0 < best ? c0 : best;
                }
            }
        }
    } else {
        publish();
        for (int i = tid; i < p.S; i += kRouteThreads) {
            const uint64_t c0 = evict_composite(u[i], i);
            best = c0 < best ? c0 : best;
        }
    }
    best = wave_min_u64(best);
    if (lane == 0) wave_best[wave] = best;
    __syncthreads();
    // what is left - the new rows and the bookkeeping - takes the block's first waves only: the
    // others leave, and with them their share of the SIMDs' issue slots
    if (wave != 0 && wave * kWave >= new_chunks) return;
    static_assert(kWaves <= 16, "one LDS word per lane of a row");
    uint64_t m = wave_min_u64(wave_best[lane & (kWaves - 1)]);
    const bool full = n >= p.S;
    const int slot = full ? evict_composite_slot(m) : n;

    // insert the new entry's rows (one 16-byte chunk per thread and pass)
    Kd += slot * p.stride_s_bytes;
    Vd += slot * p.stride_s_bytes;
    for (int idx = tid; idx < new_chunks; idx += kRouteThreads) {
        uint4 kv = knew, vv = vnew;
        if (idx >= kRouteThreads) {
            kv = load16(static_cast<const char *>(p.K_new) + ((int64_t)b * new_chunks + idx) * 16);
            vv = load16(static_cast<const char *>(p.V_new) + ((int64_t)b * new_chunks + idx) * 16);
        }
        const int hk = idx >> p.row_bits, cc = idx & (p.row_chunks - 1);
        *reinterpret_cast<uint4 *>(Kd + hk * p.stride_h_bytes + cc * 16) = kv;
        *reinterpret_cast<uint4 *>(Vd + hk * p.stride_h_bytes + cc * 16) = vv;
    }
    if (tid == 0) {
        if (full) p.evicted_idx[be] = slot;
        p.evicted_cnt[be] = full ? 1 : 0;
        p.utility[be * p.S + slot] = 0.0f;
        p.n_valid[be] = full ? p.S : n + 1;
        // the new entry's bookkeeping (Algorithm 1 Insert)
        if (p.pol.birth) p.pol.birth[be * p.S + slot] = p.pol.now;
        if (p.pol.last_access) p.pol.last_access[be * p.S + slot] = p.pol.now;
        if (p.pol.freq) p.pol.freq[be * p.S + slot] = 0;
    }
    // experts nobody selected report "nothing evicted" (block 0 of the sequence)
    if (j == 0 && tid < p.E && rank >= p.k) p.evicted_cnt[(int64_t)b * p.E + tid] = 0;
}

// The merge as a launch of its own with one block more, for the router's penalty update.
template <typename T, int THREADS>
__global__ __launch_bounds__(THREADS) void merge_with_penalty(CombineParams c, PenaltyParams fb) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // combine_smem_bytes()
    if (blockIdx.x == gridDim.x - 1) {
        if (threadIdx.x < kWave) penalty_wave(fb, threadIdx.x);
        return;
    }
    combine_head<T, THREADS>(c, blockIdx.x, smem);
}

// Post-attention stage of the fused step: the merge of the split partials (one block per
// query head, as in the stand-alone combine kernel) and the utility update in ONE launch.
// A utility block (256 slots of a visited shard x 4 groups of heads) cannot wait for the merge
// blocks, so it recomputes the per-head softmax statistics itself from the (max, sum) pairs of
// the partials - a few KiB from L2 and the same arithmetic, hence the same bits - while its
// score loads are already in flight.
// Beyond this many (head, shard) pairs - or heads, where the merge takes blocks of 1024 threads - the merge and the
// utility update run as two launches: every utility block of the single launch re-derives the statistics of all
// pairs from their partials, while the stand-alone kernel reads the merge's (shift, coef) pairs.  Kernel trace, one launch
// against both of the others (which are 0.7 us apart as well): 128 heads x 4 shards 13.9 against 4.7 + 5.2 us, in
// blocks of 256 threads 13.7 against 4.1 + 4.7, 16 sequences of them 18.4 against 5.8 + 7.5; 96 x 4 10.9 against 4.1 + 4.1, 96 x 2
// in blocks of 1024 9.9 and 4.1 + 4.2; the other side of the line: 64 x 4 7.1 against 4.0 + 3.7, 16 sequences 10.4 against
// 4.7 + 4.8, 128 x 2 in blocks of 256 9.5 against 4.6 + 4.2, 32 sequences 12.9 against 8.5 + 5.3, 16 x 16 5.6 against 4.4 + 3.1.
constexpr int kPostMostPairs = 256;
constexpr int kPostMostHeads = 255, kPostMostHeadsOf1024 = 64;
inline bool post_separate(int Hq, int k, int np) {
    return (int64_t)Hq * k > kPostMostPairs || Hq > (combine_threads(np) == 1024 ? kPostMostHeadsOf1024 : kPostMostHeads);
}

constexpr int kPostPrefetchHeads = 8;  // score loads each thread issues before the statistics
constexpr int kPostMaxTiles = 8;       // slot tiles one utility block walks through
constexpr int kPostStatsAhead = 4;     // many-pairs shape: passes of statistics whose loads are in flight
// Shapes of the kernel (template MODE): one slot tile per utility block and straight-line code;
// several tiles per block; many (head, shard) pairs or many heads per thread.
constexpr int kPostSingle = 0, kPostMulti = 1, kPostMany = 2;

struct PostParams {
    CombineParams c;
    const float *scores;
    const int32_t *n_valid;
    const int32_t *topk;
    float *utility;
    int B, E, S;
    int tiles;            // utility blocks per selected shard
    FastDiv by_tiles, by_k;
    int tiles_per_block;  // consecutive slot tiles each of them covers
    int util_first;       // the utility blocks take the grid's first block ids (they start first)
    float decay;
    int track;            // access bookkeeping: mass above pol.threshold stamps and counts the entry
    PolicyView pol;
    int small_scores;     // Hq * k * S < 2^31: a sequence's scores are addressed with 32-bit offsets
    int feedback;         // the grid's last block runs the router's penalty update (fb)
    PenaltyParams fb;
};

// LDS of a utility block: statistics of the Hq * k (head, shard) pairs, the gates, and two
// buffers of per-(head group, slot) sums used in turn.
inline __host__ __device__ int post_pairs_pad(int pairs) { return (pairs + 3) & ~3; }
inline size_t post_smem_bytes(int threads, int np, int pairs, int slots_per_thread, int decoder_bytes) {
    const size_t util = (size_t)(4 * post_pairs_pad(pairs) + 64 + 2 * slots_per_thread * threads) * 4;
    const size_t comb = combine_smem_bytes(threads, np, decoder_bytes);
    return util > comb ? util : comb;
}

// B*Hq blocks merge one query head each (the grid's first ids, or with util_first those after
// the utility blocks); the others update the utilities of
// tiles_per_block tiles of THREADS/4 slots of the j-th selected shard of a sequence.  THREADS
// is the merge's block size (combine_threads), so that the merge is bit-identical to the
// stand-alone kernel.
//
// SPT slots per thread: 1, or 4 consecutive ones (16-byte score loads, tiles of THREADS slots) when
// tiles of THREADS / 4 slots would take more than one round of blocks.  Those blocks were bound by
// their chain of trips and barriers, not by the score bytes: with four slots per thread a quarter
// of the blocks (or of the tiles a block walks through) has the same bytes in flight at once, and
// the statistics are formed a quarter as often.  Measured: 16 sequences x 32 heads x 2 shards of 4096
// slots 10.0 -> 7.2 us, with access bookkeeping 12.5 -> 8.4; 32 sequences, 2048 slots 11.7 -> 10.8; at
// one round of blocks or less it is no faster (4 shards of 8192 slots, 1 sequence: +1.5 us).  Several
// tiles per block take 151 - 159 registers, three blocks per CU instead of the four planned, and gain all
// the same (whole step, rows of 16 values: 32 sequences x 8 heads x 4 shards of 8192 slots 131.5 with one slot per
// thread -> 127 us, 64 x 4 x 8 of 8192 283 -> 257, 32 x 32 x 8 of 4096 436 -> 432; planned for three
// blocks: even).
//
// LANES: up to kWaveShards selected shards.  The (shift, coef) pair of a head comes out of the lanes that reduced its
// partials, without a trip through LDS between the statistics and the weights; in blocks of 256 threads, where a wave
// is a head group, each wave forms those of its own heads and no barrier stands before the scores' exponentials: the
// other waves' statistics are nothing it waits for.  What bounds these blocks is the chain of phases and, with the chip full of
// them, the instructions of a phase.  Kernel trace, with the merge's change below: 32 sequences x 32 heads x 2 shards of 2048
// slots 10.6 -> 8.2 us, 4 x 32 x 4 of 8192 a fourteenth full 6.5 -> 5.2, 8 x 32 x 2 of 4096 half full 5.7 -> 5.4, 1 x 32 x 4 of
// 8192 (blocks of 1024) 5.1 -> 4.8, 16 x 32 x 2 of 4096 codes of rank 32 8.3 -> 7.1.
template <typename T, int THREADS, int MODE, int SPT, bool LANES>
__global__ __launch_bounds__(THREADS) void step_post(PostParams p) {
    constexpr bool kOwnHeads = LANES && THREADS == 256;
    constexpr int kSlots = THREADS / 4 * SPT;
    const int ntiles = MODE != kPostSingle ? p.tiles_per_block : 1;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // post_smem_bytes()
    const int Hq = p.c.Hq, k = p.c.k, nsplit = p.c.nsplit;
    const int ncomb = p.B * Hq;
    // Blocks are dispatched in id order.  With more than 64 pairs, or 17 heads and more per thread, the utility
    // blocks are the long ones: they take the first ids, so that they do not queue behind the merge blocks.
    // (Blocks of 1024 threads never have as many: post_separate.)
    const bool util_first = (MODE == kPostMany || kOwnHeads) && p.util_first;
    const int mb = util_first ? (int)blockIdx.x - p.B * k * p.tiles : (int)blockIdx.x;
    if (mb >= 0 && mb < ncomb) {
        combine_head<T, THREADS>(p.c, mb, smem);
        return;
    }
    if (p.feedback && blockIdx.x == gridDim.x - 1) {   // Table 1 penalty for the next step
        if (threadIdx.x < kWave) penalty_wave(p.fb, threadIdx.x);
        return;
    }
    const int np = k * nsplit;
    int bid = util_first ? (int)blockIdx.x : (int)blockIdx.x - ncomb;
    int tile, j;
    bid = fast_divide(p.by_tiles, bid, &tile);
    const int b = fast_divide(p.by_k, bid, &j);
    const int tid = threadIdx.x;
    // Order of the requests: loads come back in the order they were issued, a value the
    // compiler knows to be the same in all lanes is waited for where it is loaded (it goes to a
    // scalar register at once), and nothing that is needed early may queue behind something
    // slow.  So the sequence's selections, entry counts and gates are read one per lane, first
    // (lane l takes selection l, shard l's count; the block's own are picked out of the registers when the pairs are
    // on their way); then the (max, sum) pairs of the statistics; then, once the count is here and the block
    // has not left for lack of entries, the scores, which come in while the statistics are formed.  (Requested with the
    // pairs, up to the shard's capacity, they gain nothing in full shards and cost nearly empty ones 5.3 -> 6.4 us: 4
    // sequences x 32 heads x 4 shards of 8192 slots, 573 entries each.)
    const int lane_id = tid & (kWave - 1);
    const int sel_of_lane = p.topk[(int64_t)b * k + min(lane_id, k - 1)];
    const int n_of_lane = p.n_valid[(int64_t)b * p.E + min(lane_id, p.E - 1)];
    // LANES: kp groups of 8 lanes per head, one for each shard (padded to a power of two)
    const int kp = pow2_at_least(k), kp_log2 = 31 - __builtin_clz(kp);
    const int gj = LANES ? min((tid >> 3) & (kp - 1), k - 1) : tid;
    const float gate_of_thread = (p.c.gates != nullptr && gj < k) ? p.c.gates[(int64_t)b * k + gj] : 1.0f;
    const int i0 = tile * kSlots * ntiles;

    const int pairs = post_pairs_pad(Hq * k);
    float *Mj_s = reinterpret_cast<float *>(smem), *Zj_s = Mj_s + pairs;
    float *shift_s = Zj_s + pairs, *coef_s = shift_s + pairs;
    float *g_s = coef_s + pairs;               // [64]
    float *part_s = g_s + 64;                  // [2][4][kSlots]
    float2 *pc_s = reinterpret_cast<float2 *>(smem);       // LANES: [Hq] (shift, coef) for the block's shard

    // thread = (SPT slots, head group); the heads are cut into 4 consecutive groups, each summed in
    // ascending order, the groups joined as (g0 + g1) + (g2 + g3) - the order the stand-alone
    // utility kernel uses too
    const int slot = (tid & (THREADS / 4 - 1)) * SPT, hg = tid / (THREADS / 4);
    const int gsize = (Hq + 3) / 4;
    const int h_lo = hg * gsize, h_hi = min(Hq, h_lo + gsize);
    float sc[kPostPrefetchHeads][SPT];
    auto load_scores = [&](float(&to)[SPT], const float *from) {
        if constexpr (SPT == 4) {
            const float4 v = *reinterpret_cast<const float4 *>(from);
            to[0] = v.x, to[1] = v.y, to[2] = v.z, to[3] = v.w;
        } else {
            to[0] = *from;
        }
    };
    // (unconditional loads from clamped, always valid addresses: heads past the group's end and
    // slots past the limit are masked where the values are used.  Loads under a lane-dependent
    // branch would make every later wait a wait for ALL loads in flight.)
    // Addresses = the sequence's block of scores (one 64-bit base, the same in every thread) plus
    // 32-bit element offsets built with adds and selects: as eight independent 64-bit products
    // they took some 130 instructions per wave, many of them quarter-rate multiplies, in front of
    // the block's first requests - and a block's 16 waves issue four to a SIMD, one after another.
    // (p.small_scores: a sequence's scores span less than 2^31 elements; else the long form.)
    const float *seq_scores = p.scores + (int64_t)b * Hq * k * p.S;
    const int h_first = min(h_lo, Hq - 1), t_last = Hq - 1 - h_first;
    const uint32_t kS = (uint32_t)k * (uint32_t)p.S;
    const uint32_t off_first = ((uint32_t)h_first * (uint32_t)k + (uint32_t)j) * (uint32_t)p.S;
    const uint32_t off_last = off_first + (uint32_t)t_last * kS;
    auto fetch = [&](int i, int limit, bool first) {
        const int ic = min(i, SPT == 4 ? p.S - 4 : limit - 1);      // (SPT = 4: S is a multiple of 4)
        // (the later tiles' requests keep the long form: its bases are set up once, after the
        // first requests have gone out, and a tile then costs one add per head; the shape with
        // several tiles per block keeps it throughout - there both forms side by side measured
        // 0.5-0.9 us slower on the streaming workload)
        if (MODE != kPostMulti && first && p.small_scores) {  // block-uniform
#pragma unroll
            for (int t = 0; t < kPostPrefetchHeads; ++t) {
                const uint32_t off = (t < t_last ? off_first + (uint32_t)t * kS : off_last) + (uint32_t)ic;
                load_scores(sc[t], seq_scores + off);
            }
        } else {
#pragma unroll
            for (int t = 0; t < kPostPrefetchHeads; ++t) {
                const int h = min(h_lo + t, Hq - 1);
                load_scores(sc[t], p.scores + (((int64_t)b * Hq + h) * k + j) * p.S + ic);
            }
        }
    };
    int i = i0 + slot;
    // softmax statistics of every (head, selected shard): 8 lanes each, pairs read from L2.  The
    // pairs of the first pass are requested before the scores: loads come back in order, and the
    // statistics must not wait for the scores' trip to memory
    const float *ml = p.c.part_ml + (int64_t)b * Hq * np * 2;
    const int pair0 = tid / 8;
    auto pair_of = [&](int t) {
        return [=](int sp) { return *reinterpret_cast<const float2 *>(ml + 2 * ((int64_t)t * nsplit + sp)); };
    };
    // With more pairs than groups of 8 lanes the statistics take several passes (kPostMany, blocks of 256
    // threads over more than 8 shards: up to 8 of them for 256 pairs), each a round trip to L2 if taken one after
    // the other: the pairs of kPostStatsAhead passes are requested ahead, and a pass that is done requests
    // those of the pass kPostStatsAhead later.
    constexpr int kAhead = MODE == kPostMany ? kPostStatsAhead : 1;
    constexpr int kPairsPerPass = THREADS / 8;
    const int npairs = LANES ? Hq << kp_log2 : Hq * k;
    // pair t: of head t / k and shard t % k, or by kp
    auto row_of = [&](int t) { return LANES ? (t >> kp_log2) * k + min(t & (kp - 1), k - 1) : t; };
    auto is_real = [&](int t) { return t < npairs && (!LANES || (t & (kp - 1)) < k); };
    auto load_pass = [&](int pass) {
        const int t = pass * kPairsPerPass + pair0;
        return shard_pairs_load(is_real(t) ? nsplit : 0, tid & 7, pair_of(row_of(min(t, npairs - 1))));
    };
    ShardPairs held[kAhead];
    // A wave's own heads: 8 >> kp_log2 of them per pass, each lane `per` pairs of a pass (1, 2 or 4: blocks of 256 threads
    // have at most 32 partials per head).  Four pairs are requested ahead: passes x per of them up to 32 heads.
    const int per_log2 = nsplit > 16 ? 2 : nsplit > 8 ? 1 : 0;
    const int own_head = lane_id >> (3 + kp_log2), own_shard = (lane_id >> 3) & (kp - 1);
    const uint32_t own_first = __umul24((uint32_t)min(own_shard, k - 1), (uint32_t)nsplit);
    float2 own[4];
    auto load_own = [&](int first) {         // pairs first .. first + 3 of the lane
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int pass = (first + x) >> per_log2, sp = (lane_id & 7) + 8 * ((first + x) & ((1 << per_log2) - 1));
            const int h = h_lo + (pass << (3 - kp_log2)) + own_head;
            const uint32_t at = __umul24((uint32_t)min(h, Hq - 1), (uint32_t)np) + own_first + (uint32_t)min(sp, nsplit - 1);
            const float2 v = reinterpret_cast<const float2 *>(ml)[at];
            const bool real = h < h_hi && own_shard < k && sp < nsplit;
            own[x].x = real ? v.x : -INFINITY;
            own[x].y = real ? v.y : 0.0f;
        }
    };
    if constexpr (kOwnHeads) {
        load_own(0);
    } else {
#pragma unroll
        for (int a = 0; a < kAhead; ++a) held[a] = load_pass(a);
    }
    const int e = __builtin_amdgcn_readlane(sel_of_lane, j);
    const int n = __builtin_amdgcn_readlane(n_of_lane, e);
    if (i0 >= n) return;     // block-uniform: no entries in this block's slots
    fetch(i, n, true);

    if constexpr (kOwnHeads) {
        const int pairs_own = __builtin_amdgcn_readfirstlane(((h_hi - h_lo + (8 >> kp_log2) - 1) >> (3 - kp_log2)) << per_log2);
        auto weigh = [&](int pass, float M, float Z) {
            const HeadWeights hw = head_weights_of_groups(kp, M, Z, gate_of_thread, p.c.combine);
            const int h = h_lo + (pass << (3 - kp_log2)) + own_head;
            if (own_shard == j && h < h_hi && (lane_id & 7) == 0) pc_s[h] = make_float2(hw.shift, hw.coef);
        };
        // (shard_stats8 over the `PER` pairs a lane has of a shard)
        auto pass_of = [&](auto per, int at) {
            constexpr int PER = decltype(per)::value;
#pragma unroll
            for (int x = 0; x < 4; x += PER) {
                if (at + x >= pairs_own) break;          // wave-uniform
                float M = -INFINITY, Z = 0.0f;
#pragma unroll
                for (int u = 0; u < PER; ++u) M = own[x + u].y > 0.0f ? fmaxf(M, own[x + u].x) : M;
                M = bits_max<0, 3>(M);
#pragma unroll
                for (int u = 0; u < PER; ++u) Z += own[x + u].y > 0.0f ? own[x + u].y * __expf(own[x + u].x - M) : 0.0f;
                weigh((at + x) >> per_log2, M, bits_sum<0, 3>(Z));
            }
        };
        for (int at = 0; at < pairs_own; at += 4) {      // wave-uniform
            if (at > 0) load_own(at);
            if (per_log2 == 0) pass_of(std::integral_constant<int, 1>{}, at);
            else if (per_log2 == 1) pass_of(std::integral_constant<int, 2>{}, at);
            else pass_of(std::integral_constant<int, 4>{}, at);
        }
        wave_lds_order();
    }
    const int passes = kOwnHeads ? 0 : (npairs + kPairsPerPass - 1) / kPairsPerPass;
    for (int pass0 = 0; pass0 < passes; pass0 += kAhead) {
#pragma unroll
        for (int a = 0; a < kAhead; ++a) {
            const int pass = pass0 + a;
            if (pass < passes) {                 // block-uniform
                const int t = pass * kPairsPerPass + pair0;
                const bool real = is_real(t);
                float M, Z;
                if (MODE == kPostMany || pass == 0)
                    shard_stats8(held[a], real ? nsplit : 0, tid & 7, pair_of(row_of(t)), &M, &Z);
                else
                    shard_stats8(real ? nsplit : 0, tid & 7, pair_of(row_of(t)), &M, &Z);
                if constexpr (LANES) {
                    const HeadWeights hw = head_weights_of_groups(kp, M, Z, gate_of_thread, p.c.combine);
                    if (real && (tid & 7) == 0 && (t & (kp - 1)) == j) pc_s[t >> kp_log2] = make_float2(hw.shift, hw.coef);
                } else if (real && (tid & 7) == 0) {
                    Mj_s[t] = M;
                    Zj_s[t] = Z;
                }
                if (MODE == kPostMany && pass + kAhead < passes) held[a] = load_pass(pass + kAhead);
            }
        }
    }
    float *urow = p.utility + ((int64_t)b * p.E + e) * p.S;
    // the utilities: with one slot per thread by the first head group, with four by every thread
    const int uslot = SPT == 4 ? tid : slot;
    const bool updates = SPT == 4 || hg == 0;
    int ui = i0 + uslot;
    float u_old = (ui < n && updates) ? urow[ui] : 0.0f;
    if constexpr (LANES) {
        if constexpr (!kOwnHeads) __syncthreads();
    } else {
        if (p.c.gates != nullptr && tid < k) g_s[tid] = gate_of_thread;
        __syncthreads();
        // (shift, coef) of every (head, shard) pair: an aligned group of kp lanes per head
        for (int h0 = 0; h0 < Hq; h0 += THREADS / kp) {
            const int h = h0 + tid / kp, jj = tid & (kp - 1);
            // a wave holds 64 / kp whole heads: one whose first head is past the end has nothing to
            // do and leaves the SIMD to the waves that have (wave-uniform branch)
            if (__builtin_amdgcn_readfirstlane(h) >= Hq) break;
            const bool mine = h < Hq && jj < k;
            const HeadWeights hw = head_weights(kp, mine ? Mj_s[h * k + jj] : 0.0f, mine ? Zj_s[h * k + jj] : 0.0f,
                                                (mine && p.c.gates) ? g_s[jj] : 1.0f, p.c.combine);
            if (mine) {
                shift_s[h * k + jj] = hw.shift;
                coef_s[h * k + jj] = hw.coef;
            }
        }
        __syncthreads();
    }
    auto weight_of = [&](int h) { return LANES ? pc_s[h] : make_float2(shift_s[h * k + j], coef_s[h * k + j]); };
    for (int it = 0; it < ntiles; ++it) {
        const bool live = i < n;
        float a[SPT];
#pragma unroll
        for (int x = 0; x < SPT; ++x) a[x] = 0.0f;
        // the prefetched heads, without branches: the group's head range is the same in the whole
        // wave (a scalar compare picks the sum or leaves it), heads past its end read a clamped,
        // valid pair, and lanes past the entry count compute on their clamped scores for nothing
        const int held_heads = __builtin_amdgcn_readfirstlane(h_hi - h_lo);
#pragma unroll
        for (int t = 0; t < kPostPrefetchHeads; ++t) {
            const int h = min(h_lo + t, Hq - 1);
            const float2 w = weight_of(h);
#pragma unroll
            for (int x = 0; x < SPT; ++x) {
                const float with = fmaf(w.y, __expf(sc[t][x] - w.x), a[x]);
                a[x] = t < held_heads ? with : a[x];
            }
        }
        if (live) {
            // more heads per group than were prefetched: batches of loads, same ascending order
            for (int hb = h_lo + kPostPrefetchHeads; hb < h_hi; hb += kPostPrefetchHeads) {
                float more[kPostPrefetchHeads][SPT];
#pragma unroll
                for (int t = 0; t < kPostPrefetchHeads; ++t)
                    load_scores(more[t], p.scores + (((int64_t)b * Hq + min(hb + t, h_hi - 1)) * k + j) * p.S + i);
#pragma unroll
                for (int t = 0; t < kPostPrefetchHeads; ++t) {
                    const int h = hb + t;
                    if (h < h_hi) {
                        const float2 w = weight_of(h);
#pragma unroll
                        for (int x = 0; x < SPT; ++x) a[x] = fmaf(w.y, __expf(more[t][x] - w.x), a[x]);
                    }
                }
            }
        }
        // the next tile's loads go out before this tile's sums meet in LDS
        const int i_next = i + kSlots;
        const int u_at = ui;
        const float u_cur = u_old;
        ui += kSlots;
        if (it + 1 < ntiles) {
            fetch(i_next, n, false);
            u_old = (ui < n && updates) ? urow[ui] : 0.0f;
        }
        float *part = part_s + (it & 1) * 4 * kSlots;    // rewritten two tiles later, after a barrier
#pragma unroll
        for (int x = 0; x < SPT; ++x) part[hg * kSlots + slot + x] = a[x];
        __syncthreads();
        if (updates && u_at < n) {
            const float total = (part[uslot] + part[kSlots + uslot]) +
                                (part[2 * kSlots + uslot] + part[3 * kSlots + uslot]);
            urow[u_at] = fmaf(p.decay, u_cur, total);
            if (p.track && total > p.pol.threshold) {
                const int64_t at = ((int64_t)b * p.E + e) * p.S + u_at;
                p.pol.last_access[at] = p.pol.now;
                p.pol.freq[at] += 1;
            }
        }
        i = i_next;
    }
}

}  // namespace
}  // namespace pikv

using namespace pikv;

static int decode_step(const pikv_desc *desc, const void *q, const void *W_r, const float *bias,
                       const void *K_new, const void *V_new, void *const *K_shards,
                       void *const *V_shards, const void *U_K, const void *U_V, int32_t *n_valid,
                       float *utility, int32_t k, int32_t combine, float scale, float decay,
                       int32_t *topk_idx, float *gates, int32_t *evicted_idx, int32_t *evicted_cnt,
                       float *y, float *row_max, float *row_norm, float *scores, float *slot_coef,
                       void *workspace, size_t workspace_bytes, void *stream,
                       const pikv_policy_args *pa, const pikv_router_feedback *fb) {
    const int rc = check_desc(desc);
    if (rc != PIKV_OK) return rc;
    PolicyView pol = {};
    bool use_policy = false, track = false;
    if (pa != nullptr) {
        const int prc = check_policy(pa->policy, pa->window, pa->protect, pa->lambda, pa->birth,
                                     pa->last_access, pa->freq, utility);
        if (prc != PIKV_OK) return prc;
        track = pa->last_access != nullptr && pa->freq != nullptr;
        if (track && !(pa->threshold >= 0.0f)) return PIKV_ERR_INVALID;
        pol.policy = pa->policy;
        pol.now = pa->now;
        pol.window = pa->window;
        pol.protect = pa->protect;
        pol.lambda = pa->lambda;
        pol.threshold = pa->threshold;
        pol.birth = pa->birth;
        pol.last_access = pa->last_access;
        pol.freq = pa->freq;
        use_policy = pa->policy != PIKV_POLICY_H2O || pa->protect > 0;
    }
    if (!q || !W_r || !K_shards || !V_shards || !n_valid || !utility || !topk_idx || !gates || !y ||
        !scores || !slot_coef)
        return PIKV_ERR_INVALID;
    PenaltyParams pen = {};
    if (fb != nullptr) {
        const int frc = check_penalty(fb->mode, fb->load, fb->miss, fb->coef, fb->bias, desc->E);
        if (frc != PIKV_OK) return frc;
        pen.mode = fb->mode;
        pen.topk = topk_idx;
        pen.n_sel = desc->B * k;
        pen.E = desc->E;
        pen.load = fb->load;
        pen.miss = fb->miss;
        pen.coef = fb->coef;
        pen.bias = fb->bias;
    }
    if ((K_new == nullptr) != (V_new == nullptr)) return PIKV_ERR_INVALID;
    if (K_new && (!evicted_idx || !evicted_cnt)) return PIKV_ERR_INVALID;
    if (k < 1 || k > desc->E) return PIKV_ERR_INVALID;
    if (!(decay >= 0.0f) || decay > 3.0e38f) return PIKV_ERR_INVALID;
    if (combine != PIKV_COMBINE_LSE && combine != PIKV_COMBINE_LOCAL) return PIKV_ERR_INVALID;
    if (desc->route_rows_per_seq != 1) return PIKV_ERR_UNSUPPORTED;
    // the attention pass's own checks come before the first launch as well: a rejected call
    // leaves the cache (rows, utilities, entry counts, policy arrays) exactly as it was
    AttnPlan checked;
    const int arc = check_attn_args(desc, q, K_shards, V_shards, U_K, U_V, n_valid, topk_idx, k, combine,
                                    scale, y, workspace, workspace_bytes, &checked);
    if (arc != PIKV_OK) return arc;
    hipStream_t st = as_stream(stream);
    if (profile_events_set()) {
        // an event record inside a captured graph would replay with every launch of the graph
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &cs) != hipSuccess) return PIKV_ERR_HIP;
        if (cs != hipStreamCaptureStatusNone) return PIKV_ERR_INVALID;
    }
    if (desc->B == 0) return PIKV_OK;

    PreParams p;
    p.x = q;
    p.W_r = W_r;
    p.bias = bias;
    p.topk = topk_idx;
    p.gates = gates;
    p.K_new = K_new;
    p.V_new = V_new;
    p.K = K_shards;
    p.V = V_shards;
    p.utility = utility;
    p.n_valid = n_valid;
    p.evicted_idx = evicted_idx;
    p.evicted_cnt = evicted_cnt;
    const int eb = elem_bytes(desc->dtype);
    p.stride_h_bytes = desc->stride_h * eb;
    p.stride_s_bytes = desc->stride_s * eb;
    // a multi-query step is routed by its first query alone: the leading d_r values of q[b]
    const int tq = desc->tq > 1 ? desc->tq : 1;
    if (desc->Hq % tq != 0) return PIKV_ERR_UNSUPPORTED;
    p.d_r = desc->Hq / tq * desc->D;
    p.x_stride = (int64_t)desc->Hq * desc->D;
    p.E = desc->E;
    p.cpr = 0;
    p.flat_threads = 0;
    if (desc->dtype == PIKV_F32 && !route_vec_ok(W_r, desc->E, &p.cpr))
        p.flat_threads = route_single_ok(p.d_r, desc->E) ? -1 : route_flat_threads(p.d_r, desc->E);
    p.w_aligned = reinterpret_cast<uintptr_t>(W_r) % 16 == 0;
    p.words = route_words_ok(q, p.x_stride, W_r, p.d_r, desc->E);
    p.k = k;
    p.S = desc->S;
    p.Hkv = desc->Hkv;
    p.row_chunks = desc_width(desc) * eb / 16;
    p.row_bits = __builtin_ctz(p.row_chunks);
    p.by_k = fast_div(k);
    p.do_insert = K_new != nullptr;
    p.use_policy = use_policy;
    p.pol = pol;
    const dim3 pre_grid(desc->B * k), pre_block(kRouteThreads);
    if (desc->dtype == PIKV_F32) {
        hipLaunchKernelGGL((step_pre<float, 0>), pre_grid, pre_block, 0, st, p);
    } else {
        switch (route_experts_most(desc->E)) {
            case 8: hipLaunchKernelGGL((step_pre<bf16, 8>), pre_grid, pre_block, 0, st, p); break;
            case 16: hipLaunchKernelGGL((step_pre<bf16, 16>), pre_grid, pre_block, 0, st, p); break;
            case 32: hipLaunchKernelGGL((step_pre<bf16, 32>), pre_grid, pre_block, 0, st, p); break;
            default: hipLaunchKernelGGL((step_pre<bf16, 64>), pre_grid, pre_block, 0, st, p); break;
        }
    }
    int lrc = launch_status();
    if (lrc != PIKV_OK) return lrc;
    AttnPlan plan;
    CombineParams c;
    lrc = launch_attn_partial(desc, q, K_shards, V_shards, U_K, U_V, n_valid, topk_idx, gates, k,
                              combine, scale, y, row_max, row_norm, scores, slot_coef, workspace,
                              workspace_bytes, stream, &checked, &plan, &c);
    if (lrc != PIKV_OK) return lrc;
    const int np = k * plan.nsplit;
    const int threads = combine_threads(np);
    const bool f32 = desc->dtype == PIKV_F32;
    if (post_separate(desc->Hq, k, np)) {
        if (fb == nullptr) {
            lrc = pikv_sharded_attn_merge(desc, &c, stream);
        } else {
            const dim3 mgrid(desc->B * desc->Hq + 1);
            const size_t mlds = combine_smem_bytes(threads, np, c.decoder_bytes);
            if (threads == 256 && f32) hipLaunchKernelGGL((merge_with_penalty<float, 256>), mgrid, dim3(256), mlds, st, c, pen);
            else if (threads == 256) hipLaunchKernelGGL((merge_with_penalty<bf16, 256>), mgrid, dim3(256), mlds, st, c, pen);
            else if (f32) hipLaunchKernelGGL((merge_with_penalty<float, 1024>), mgrid, dim3(1024), mlds, st, c, pen);
            else hipLaunchKernelGGL((merge_with_penalty<bf16, 1024>), mgrid, dim3(1024), mlds, st, c, pen);
            lrc = launch_status();
        }
        if (lrc != PIKV_OK) return lrc;
        if (track)
            return pikv_update_utility_tracked(desc, scores, slot_coef, n_valid, topk_idx, k, decay,
                                               utility, pol.threshold, pol.now, pol.last_access,
                                               pol.freq, stream);
        return pikv_update_utility(desc, scores, slot_coef, n_valid, topk_idx, k, decay, utility, stream);
    }
    PostParams pp;
    pp.c = c;
    pp.scores = scores;
    pp.n_valid = n_valid;
    pp.topk = topk_idx;
    pp.utility = utility;
    pp.track = track;
    pp.pol = pol;
    pp.small_scores = (int64_t)desc->Hq * k * desc->S < ((int64_t)1 << 31);
    pp.B = desc->B;
    pp.E = desc->E;
    pp.S = desc->S;
    // Utility blocks: enough of them to fill the GPU once (256 CUs x the blocks a CU holds),
    // each walking through several slot tiles rather than a new block per tile - the
    // statistics of the sequence's (head, shard) pairs are then computed once per block.
    const int64_t want_blocks = threads == 256 ? 1024 : 256;
    auto tiles_of = [&](int slots) { return (int64_t)(desc->S + slots - 1) / slots; };
    auto tiles_per_block = [&](int64_t tiles) {
        const int64_t t = ((int64_t)desc->B * k * tiles + want_blocks - 1) / want_blocks;
        return t < 1 ? 1 : t > kPostMaxTiles ? (int64_t)kPostMaxTiles : t;
    };
    const bool lanes = k <= kWaveShards;
    // more (head, shard) pairs than a pass takes, or many heads per thread: the utility blocks start first, and without
    // lane statistics (blocks of 256 threads) it takes the shape that keeps several passes of them in flight
    const bool many = desc->Hq * k > 2 * (threads / 8) || (desc->Hq + 3) / 4 > 2 * kPostPrefetchHeads;
    // four slots per thread as soon as one slot per thread needs more than one round of blocks (in
    // blocks of 1024 threads only where the loop-free shape takes it: the others would spill)
    bool wide = (int64_t)desc->B * k * tiles_of(threads / 4) > want_blocks && desc->S % 4 == 0 &&
                reinterpret_cast<uintptr_t>(scores) % 16 == 0;
    if (threads == 1024 && tiles_per_block(tiles_of(threads)) > 1) wide = false;
    const int64_t slot_tiles = tiles_of(wide ? threads : threads / 4);
    const int64_t tpb = tiles_per_block(slot_tiles);
    pp.tiles_per_block = (int)tpb;
    pp.tiles = (int)((slot_tiles + tpb - 1) / tpb);
    pp.by_tiles = fast_div(pp.tiles);
    pp.by_k = fast_div(k);
    pp.util_first = many ? 1 : 0;
    pp.decay = decay;
    pp.feedback = fb != nullptr;
    pp.fb = pen;
    const int64_t blocks = (int64_t)desc->B * desc->Hq + (int64_t)desc->B * k * pp.tiles + (fb ? 1 : 0);
    if (blocks > 0x7fffffff) return PIKV_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)blocks);
    const size_t lds = post_smem_bytes(threads, np, desc->Hq * k, wide ? 4 : 1, c.decoder_bytes);
    const bool multi = tpb > 1;
    // (several tiles of four slots per thread: blocks of 256 threads only, see `wide`)
    auto launch = [&](auto type, auto th, auto mode, auto with_lanes) {
        typedef decltype(type) T;
        constexpr int TH = decltype(th)::value, MODE = decltype(mode)::value;
        constexpr bool LANES = decltype(with_lanes)::value;
        constexpr int kWide = TH == 256 || MODE == kPostSingle ? 4 : 1;
        if (wide) hipLaunchKernelGGL((step_post<T, TH, MODE, kWide, LANES>), grid, dim3(TH), lds, st, pp);
        else hipLaunchKernelGGL((step_post<T, TH, MODE, 1, LANES>), grid, dim3(TH), lds, st, pp);
    };
    auto launch_mode = [&](auto type, auto th, auto with_lanes) {
        constexpr bool kHasMany = decltype(th)::value == 256 && !decltype(with_lanes)::value;
        if constexpr (kHasMany) {
            if (many) return launch(type, th, std::integral_constant<int, kPostMany>{}, with_lanes);
        }
        if (multi) launch(type, th, std::integral_constant<int, kPostMulti>{}, with_lanes);
        else launch(type, th, std::integral_constant<int, kPostSingle>{}, with_lanes);
    };
    auto launch_type = [&](auto type) {
        const std::integral_constant<int, 256> small{};
        const std::integral_constant<int, 1024> large{};
        if (threads == 256) lanes ? launch_mode(type, small, std::true_type{}) : launch_mode(type, small, std::false_type{});
        else lanes ? launch_mode(type, large, std::true_type{}) : launch_mode(type, large, std::false_type{});
    };
    if (f32) launch_type(float{});
    else launch_type(bf16{});
    return launch_status();
}

extern "C" int pikv_decode_step(const pikv_desc *desc, const void *q, const void *W_r,
                                const float *bias, const void *K_new, const void *V_new,
                                void *const *K_shards, void *const *V_shards, const void *U_K,
                                const void *U_V, int32_t *n_valid, float *utility, int32_t k,
                                int32_t combine, float scale, float decay, int32_t *topk_idx,
                                float *gates, int32_t *evicted_idx, int32_t *evicted_cnt, float *y,
                                float *row_max, float *row_norm, float *scores, float *slot_coef,
                                void *workspace, size_t workspace_bytes, void *stream) {
    return decode_step(desc, q, W_r, bias, K_new, V_new, K_shards, V_shards, U_K, U_V, n_valid, utility,
                       k, combine, scale, decay, topk_idx, gates, evicted_idx, evicted_cnt, y, row_max,
                       row_norm, scores, slot_coef, workspace, workspace_bytes, stream, nullptr, nullptr);
}

extern "C" int pikv_decode_step_policy(const pikv_desc *desc, const void *q, const void *W_r,
                                       const float *bias, const void *K_new, const void *V_new,
                                       void *const *K_shards, void *const *V_shards, const void *U_K,
                                       const void *U_V, int32_t *n_valid, float *utility, int32_t k,
                                       int32_t combine, float scale, float decay, int32_t *topk_idx,
                                       float *gates, int32_t *evicted_idx, int32_t *evicted_cnt,
                                       float *y, float *row_max, float *row_norm, float *scores,
                                       float *slot_coef, void *workspace, size_t workspace_bytes,
                                       void *stream, const pikv_policy_args *policy,
                                       const pikv_router_feedback *feedback) {
    return decode_step(desc, q, W_r, bias, K_new, V_new, K_shards, V_shards, U_K, U_V, n_valid, utility,
                       k, combine, scale, decay, topk_idx, gates, evicted_idx, evicted_cnt, y, row_max,
                       row_norm, scores, slot_coef, workspace, workspace_bytes, stream, policy, feedback);
}

