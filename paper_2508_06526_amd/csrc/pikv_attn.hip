// Routed attention over the selected expert shards (PiKV Algorithm 1, the f_attn step over
// C[g_t]; Section 3.2: only the k selected shards are fetched; Section 3.3: rank-r codes are
// decoded inside the kernel) as a split flash-decode for gfx950:
//
//   attn_partial : grid over (sequence, head group, selected shard, split).  Each wave64
//                  streams whole K rows and V rows with 16-byte lane loads (a wave load is
//                  1 KiB of consecutive bytes), keeps a running max / sum / output in fp32
//                  registers and never revisits a byte.  A block of 4 waves merges its
//                  waves through LDS and writes one (max, sum, acc[width]) partial.
//   attn_combine : one block per (sequence, query head) merges the k * nsplit partials with
//                  the router gates, applies the value decoder for rank-r codes, and emits
//                  y, the row statistics and the (shift, coef) pairs the utility pass needs.
//
// Low-rank entries are never materialised: s_i = scale * <U_K q, code_i> and
// y = (sum_i p_i code_i) U_V, so the streamed bytes are the codes and the decode costs
// O(rank) per entry (the paper's T_decode is linear in the compressed width, eq. 2).
#include "pikv_common.h"
#include "pikv_combine_dev.h"

#include <math.h>

namespace pikv {

namespace {

constexpr int kWavesPerBlock = 4;

// Shape of the plain-ALU kernel by row size and heads per block.  16-byte loads each lane keeps
// in flight per K (or V) tile: 8, or kShortRowLoads for one head over rows of at most 128 bytes (rank-r codes):
// that kernel then fits 128 registers, a CU holds four of its 4-wave blocks instead of three, and
// 1024 (sequence, head, shard) units run in one round of resident blocks instead of one and a third.
constexpr int kShortRowLoads = 4;
constexpr bool plain_short_rows(int row_bytes, int gb) { return gb == 1 && row_bytes <= 128; }
constexpr int plain_loads_per_tile(int row_bytes, int gb) { return plain_short_rows(row_bytes, gb) ? kShortRowLoads : 8; }

struct AttnParams {
    const void *q;
    const void *const *K;
    const void *const *V;
    const void *U_K;
    const int32_t *n_valid;
    const int32_t *topk;
    float *part_acc;
    float *part_ml;
    float *scores;
    int B, Hq, G, D, E, S, k, rr, rank;
    int64_t stride_h, stride_s;
    FastDiv by_nsplit, by_k, by_groups, by_G;   // head groups (Hq / the heads of a block), heads of a group
    FastDiv by_draft;   // rows of one draft query per kv head (G / tq)
    int heads;          // query heads of one draft query (Hq / tq)
    int nsplit, chunk;  // splits per shard, and the most rows one of them takes
    uint32_t nsplit_rcp;   // 2^32 / nsplit, rounded up (0: nsplit == 1)
    int tq;             // draft queries per sequence: q is [B, tq, Hq / tq, D] (1: plain [B, Hq, D])
    int stage_scores;   // keep the block's scores in LDS, write them in one burst at the end
    int stream_scores;  // ... with non-temporal stores
    float scale;
};

// Raw scores of at most this many bytes per block are staged in LDS (plain-ALU kernel).
constexpr int kScoreStageBytes = 16384;
// Resolve the j-th selected shard of a routing row with ONE round trip to memory: the
// expert id is fetched while lanes 0..E-1 fetch the entry count and the K/V base address of
// every expert of the sequence; the selected lane's values are then broadcast.
struct ShardRef {
    int e, n;
    const char *K, *V;
};
__device__ __forceinline__ ShardRef resolve_shard(const AttnParams &p, int b, int route_row, int j,
                                                  int lane) {
    const int l = min(lane, p.E - 1);
    const int64_t s = (int64_t)b * p.E + l;
    const int nv = p.n_valid[s];
    const uint64_t kp = reinterpret_cast<uint64_t>(p.K[s]);
    const uint64_t vp = reinterpret_cast<uint64_t>(p.V[s]);
    const int e = __builtin_amdgcn_readfirstlane(p.topk[(int64_t)route_row * p.k + j]);
    ShardRef out;
    out.e = e;
    out.n = __builtin_amdgcn_readlane(nv, e);
    const uint32_t klo = __builtin_amdgcn_readlane((int)(uint32_t)kp, e);
    const uint32_t khi = __builtin_amdgcn_readlane((int)(uint32_t)(kp >> 32), e);
    const uint32_t vlo = __builtin_amdgcn_readlane((int)(uint32_t)vp, e);
    const uint32_t vhi = __builtin_amdgcn_readlane((int)(uint32_t)(vp >> 32), e);
    out.K = reinterpret_cast<const char *>(((uint64_t)khi << 32) | klo);
    out.V = reinterpret_cast<const char *>(((uint64_t)vhi << 32) | vlo);
    return out;
}

// Rows [r0, r1) of split `split` of a shard that holds n entries.  The split count is planned for
// full shards; the rows are cut by what the shard holds, so that a young cache - a few hundred
// entries in shards of thousands - still spreads over the splits instead of leaving all but the
// first of them empty.  A split takes whole rounds of tiles, one per wave: with uneven waves it
// runs as long as one of more rows (32 splits of 136 rows in blocks of 160: 23.0 us, of 256: 21.6).
// (4 sequences, 8 kv heads, 4 of 16 shards of 8192 slots, 573 entries each: pass and merge 20.1 -> 16.3 us.)
template <int TILE>
__device__ __forceinline__ void split_rows(const AttnParams &p, int n, int split, int *r0, int *r1) {
    const int m = min(n, p.S);
    int per = p.chunk;
    if (p.nsplit_rcp != 0) {
        constexpr int ROUND = kWavesPerBlock * TILE;
        per = (int)__umulhi((uint32_t)(m + p.nsplit - 1), p.nsplit_rcp);
        per = min((max(per, 1) + ROUND - 1) / ROUND * ROUND, p.chunk);   // chunk: nsplit * chunk >= S
    }
    *r0 = split * per;
    *r1 = min(m, *r0 + per);
}

// Work item of a group kernel's block: its unit (sequence, head group, shard) and split.
// Workgroups go to the 8 XCDs round-robin by id.  Giving each XCD a contiguous range of units, whose splits share
// score rows and partial lines, measures 1.3 % faster than spreading neighbours over all XCDs.
__device__ __forceinline__ int group_block(const AttnParams &p, int *split) {
    const int id = blockIdx.x, grid = gridDim.x;
    const int item = (grid & 7) == 0 ? (id & 7) * (grid >> 3) + (id >> 3) : id;
    return fast_divide(p.by_nsplit, item, split);
}

// Where the caller keeps the query of internal row `row` of kv head hk of sequence b, in rows of D values.
// Internally the rows of a sequence are ordered (kv head, draft query, head of the group), so
// that all rows reading one kv head are adjacent; the caller's q is [B, tq, heads, D].  (The rows of a
// lane differ: by_draft, the heads of a draft query per kv head, saves three compiler divisions of vectors per row: pass and merge of 8 drafts 45.7 -> 44.2 us, nearly empty shards 23.3 -> 21.4.)
__device__ __forceinline__ int64_t query_row(const AttnParams &p, int b, int hk, int row) {
    if (p.tq <= 1) return (int64_t)b * p.Hq + hk * p.G + row;
    const int g = (int)p.by_draft.d;
    int t = (int)__umulhi((uint32_t)row, p.by_draft.rcp), gg = row - t * g;      // t: the quotient or one less
    if (gg >= g) ++t, gg -= g;
    return (int64_t)b * p.Hq + t * p.heads + hk * g + gg;
}

// 4-wave blocks of the plain-ALU kernel that the split plan counts per CU, and that the launch bounds
// hold the compiler to at the least.  The registers allow more in places (fp32: 119 registers at one head over
// rows of 256 bytes and more, 140 at two, 252 - 254 at eight; bf16: 131 at one head over 256 bytes, 154 - 164
// at two); the counts were measured with the kernel before its loop lost registers, and a plan for
// more has not been.
constexpr int plain_blocks_per_cu(int row_bytes, int gb) {
    return plain_short_rows(row_bytes, gb) ? 4 : gb == 1 ? 3 : (gb <= 4 ? 2 : 1);
}

// The most a CU is let hold: over short rows a sixth block fits and costs more than it gives (32 heads
// over fp32 codes of rank 16, 1 GiB of them: 1646 us with five, 1780 with six).
constexpr int plain_blocks_most(int row_bytes, int gb) { return plain_short_rows(row_bytes, gb) ? 5 : 8; }

template <typename T, int W, int GB>
__global__ __launch_bounds__(kWavesPerBlock *kWave)
__attribute__((amdgpu_waves_per_eu(plain_blocks_per_cu(W * (int)sizeof(T), GB), plain_blocks_most(W * (int)sizeof(T), GB)))) void
attn_partial(AttnParams p) {
    constexpr int EPL = Pack16<T>::N;        // elements per lane per load
    constexpr int LPR = W / EPL;             // lanes covering one row
    constexpr int RPL = kWave / LPR;         // rows covered by one wave load
    constexpr int NL = plain_loads_per_tile(W * (int)sizeof(T), GB);
    constexpr int TILE = RPL * NL;           // rows per wave iteration
    constexpr int CB = ilog2(LPR);           // lane bits that index the column chunk
    constexpr bool APART = GB <= 4 && !(EPL == 8 && W == 128);  // a wave's last tile: see the streaming loop
    static_assert(LPR >= 1 && LPR <= 32 && (LPR & (LPR - 1)) == 0, "row must be 16..512 bytes");

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid >> 6;
    const int c = lane & (LPR - 1);
    const int r = lane >> CB;

    int split, j, hg, group_head;
    int bid = fast_divide(p.by_nsplit, blockIdx.x, &split);
    bid = fast_divide(p.by_k, bid, &j);
    const int b = fast_divide(p.by_groups, bid, &hg);
    const int h0 = hg * GB;
    const int hk = fast_divide(p.by_G, h0, &group_head);
    const int route_row = b * p.rr + (p.rr == 1 ? 0 : h0);
    const ShardRef sh = resolve_shard(p, b, route_row, j, lane);
    int r0, r1;
    split_rows<TILE>(p, sh.n, split, &r0, &r1);

    __shared__ float q_s[GB][W];
    __shared__ float sm_acc[kWavesPerBlock][GB][W];
    __shared__ float sm_m[kWavesPerBlock][GB];
    __shared__ float sm_l[kWavesPerBlock][GB];
    // Raw scores of the block's rows, [GB][chunk], when p.stage_scores: scattered 128-byte
    // score writes in the middle of the K/V stream cost far more HBM time than their bytes
    // (each one turns a channel around); one contiguous burst per block at the end does not.
    extern __shared__ __attribute__((aligned(16))) float score_stage[];

    const int64_t part_base = (((int64_t)b * p.Hq + h0) * p.k + j) * p.nsplit + split;
    const int64_t part_head_stride = (int64_t)p.k * p.nsplit;

    if (r0 >= r1) {  // nothing valid in this split (short or empty shard)
        for (int idx = tid; idx < GB * W; idx += blockDim.x) {
            const int g = idx / W, d = idx - g * W;
            p.part_acc[(part_base + g * part_head_stride) * W + d] = 0.0f;
            if (d == 0) {
                p.part_ml[(part_base + g * part_head_stride) * 2 + 0] = -INFINITY;
                p.part_ml[(part_base + g * part_head_stride) * 2 + 1] = 0.0f;
            }
        }
        return;
    }

    const T *Kb = reinterpret_cast<const T *>(sh.K) + (int64_t)hk * p.stride_h + c * EPL;
    const T *Vb = reinterpret_cast<const T *>(sh.V) + (int64_t)hk * p.stride_h + c * EPL;

    // A wave owns tiles t0, t0 + 4*TILE, ... of the block's row range.  The loads of a tile
    // are issued one phase ahead of their use (K of the next tile while the softmax of this
    // one runs, V of the next tile after this tile's PV), so every wave always has 8 KiB in
    // flight; the first tile's loads go out before the query is staged.
    uint4 kr[NL], vr[NL];
    auto load_tile = [&](uint4(&dst)[NL], const T *base, int t0) {
#pragma unroll
        for (int t = 0; t < NL; ++t) {
            // rows past the end are clamped onto the last valid row (always in bounds) and
            // masked out of the softmax below, so the loads need no branches
            const int row = min(t0 + t * RPL + r, r1 - 1);
            dst[t] = load16_stream(base + (int64_t)row * p.stride_s);
        }
    };
    int t0 = r0 + wave * TILE;
    if (!APART || t0 < r1) {                  // (past the end: the last row)
        load_tile(kr, Kb, t0);
        load_tile(vr, Vb, t0);
    }

    // Stage the (scaled) query in LDS; for rank-r codes it is the projected query U_K q.
    const T *qp = static_cast<const T *>(p.q) + ((int64_t)b * p.Hq + h0) * p.D;
    if (p.rank == 0) {
        for (int idx = tid; idx < GB * W; idx += blockDim.x)
            q_s[idx / W][idx % W] = p.scale * load_scalar<T>(qp, idx);   // W == D here
    } else {
        // 8 lanes per (head, code column): 16-byte loads of the decoder row and of q, all
        // independent, joined by an xor butterfly (fixed order)
        const T *U = static_cast<const T *>(p.U_K) + (int64_t)hk * p.rank * p.D;
        const int chunks = p.D / EPL;
        const int sub = tid & 7;
        for (int idx0 = 0; idx0 < GB * W; idx0 += (kWavesPerBlock * kWave) / 8) {
            const int idx = idx0 + (tid >> 3);
            const bool real = idx < GB * W;
            const int g = real ? idx / W : 0, col = real ? idx - g * W : 0;
            float a = 0.0f;
            for (int ch = sub; ch < chunks; ch += 8) {
                float uf[EPL], qv[EPL];
                Pack16<T>::widen(load16(U + (int64_t)col * p.D + ch * EPL), uf);
                Pack16<T>::widen(load16(qp + (int64_t)g * p.D + ch * EPL), qv);
#pragma unroll
                for (int i = 0; i < EPL; ++i) a = fmaf(uf[i], qv[i], a);
            }
            a += __shfl_xor(a, 1, kWave);
            a += __shfl_xor(a, 2, kWave);
            a += __shfl_xor(a, 4, kWave);
            if (real && sub == 0) q_s[g][col] = p.scale * a;
        }
    }
    __syncthreads();

    float qf[GB][EPL];
#pragma unroll
    for (int g = 0; g < GB; ++g)
#pragma unroll
        for (int i = 0; i < EPL; ++i) qf[g][i] = q_s[g][c * EPL + i];

    float m[GB], l[GB], acc[GB][EPL];
#pragma unroll
    for (int g = 0; g < GB; ++g) {
        m[g] = -INFINITY;
        l[g] = 0.0f;
#pragma unroll
        for (int i = 0; i < EPL; ++i) acc[g][i] = 0.0f;
    }

    // No request under a condition: with the next tile's K under `if (tnext < r1)` the compiler had
    // to allow for the path without it and waited, before a tile's V was used, for everything in
    // flight.  (Pass and merge: fp32 rows x 4 heads, 512 MiB 104 -> 97 us, x 8 heads 163 -> 147; bf16
    // shards a fifth full 44.6 -> 41.4; rank-32 codes 54.4 -> 53.5.)  Instead a wave's last tile has a
    // pass of its own that requests nothing: a tile requested past the end is a trip to memory that the
    // block's end waits for (32 sequences x 64 heads over 16 kv heads x 3 shards of 64 fp32 codes: 31.8 ->
    // 28.8 us; the longer code costs 4 heads x 1501 rows 17.2 -> 17.5).  Not with eight heads
    // per block, which its arithmetic bounds (147 -> 152 us), nor over bf16 rows of 128 values (it spills):
    // there the request past the end is the last row once more.
#pragma unroll
    for (int pass = APART ? 0 : 1; pass < 2; ++pass)
    while (APART && pass == 0 ? t0 + kWavesPerBlock * TILE < r1 : t0 < r1) {
        const bool more = !APART || pass == 0;
        const int tnext = t0 + kWavesPerBlock * TILE;

        // scores: each lane's partial dot over its EPL columns, summed over the row's lanes
        float s[NL][GB];
#pragma unroll
        for (int t = 0; t < NL; ++t) {
            float kf[EPL];
            Pack16<T>::widen(kr[t], kf);
            const bool valid = (t0 + t * RPL + r) < r1;
#pragma unroll
            for (int g = 0; g < GB; ++g) {
                float d = 0.0f;
#pragma unroll
                for (int i = 0; i < EPL; ++i) d = fmaf(qf[g][i], kf[i], d);
                d = bits_sum<0, CB>(d);
                s[t][g] = valid ? d : -INFINITY;
            }
        }
        if (more) load_tile(kr, Kb, tnext);

        if (p.scores != nullptr) {  // raw scores for the utility pass, one row per lane
#pragma unroll
            for (int g = 0; g < GB; ++g) {
                float *dst = p.scores + (((int64_t)b * p.Hq + h0 + g) * p.k + j) * p.S;
#pragma unroll
                for (int u = 0; u < NL; u += LPR) {
                    float v = s[u][g];
#pragma unroll
                    for (int t = 1; t < LPR && u + t < NL; ++t) v = (c == t) ? s[u + t][g] : v;
                    const int row = t0 + (u + c) * RPL + r;
                    if (u + c < NL && row < r1) {
                        if (p.stage_scores) score_stage[g * p.chunk + row - r0] = v;
                        else dst[row] = v;
                    }
                }
            }
        }

        // online softmax update (wave-uniform running max per head)
#pragma unroll
        for (int g = 0; g < GB; ++g) {
            float tm = s[0][g];
#pragma unroll
            for (int t = 1; t < NL; ++t) tm = fmaxf(tm, s[t][g]);
            tm = bits_max<CB, 6>(tm);
            const float mn = fmaxf(m[g], tm);
            const float corr = __expf(m[g] - mn);
            m[g] = mn;
            l[g] *= corr;
#pragma unroll
            for (int i = 0; i < EPL; ++i) acc[g][i] *= corr;
#pragma unroll
            for (int t = 0; t < NL; ++t) {
                const float pt = __expf(s[t][g] - mn);
                s[t][g] = pt;
                l[g] += pt;
            }
        }

        // acc += p * V rows
#pragma unroll
        for (int t = 0; t < NL; ++t) {
            float vf[EPL];
            Pack16<T>::widen(vr[t], vf);
#pragma unroll
            for (int g = 0; g < GB; ++g)
#pragma unroll
                for (int i = 0; i < EPL; ++i) acc[g][i] = fmaf(s[t][g], vf[i], acc[g][i]);
        }
        if (more) load_tile(vr, Vb, tnext);
        t0 = tnext;
    }

    // merge the row groups of the wave (same column chunk c, different r) ...
#pragma unroll
    for (int off = LPR; off < kWave; off <<= 1) {
#pragma unroll
        for (int g = 0; g < GB; ++g) {
            l[g] += __shfl_xor(l[g], off, kWave);
#pragma unroll
            for (int i = 0; i < EPL; ++i) acc[g][i] += __shfl_xor(acc[g][i], off, kWave);
        }
    }
    if (r == 0) {
#pragma unroll
        for (int g = 0; g < GB; ++g)
#pragma unroll
            for (int i = 0; i < EPL; ++i) sm_acc[wave][g][c * EPL + i] = acc[g][i];
    }
    if (lane == 0) {
#pragma unroll
        for (int g = 0; g < GB; ++g) {
            sm_m[wave][g] = m[g];
            sm_l[wave][g] = l[g];
        }
    }
    __syncthreads();

    if (p.scores != nullptr && p.stage_scores) {   // the block's scores, one contiguous burst
        const int rows = r1 - r0;
#pragma unroll
        for (int g = 0; g < GB; ++g) {
            float *dst = p.scores + (((int64_t)b * p.Hq + h0 + g) * p.k + j) * p.S + r0;
            const float *src = score_stage + g * p.chunk;
            if ((p.S & 3) == 0 && (reinterpret_cast<uintptr_t>(p.scores) & 15) == 0) {   // r0, chunk: multiples of the tile
                const int rows4 = rows & ~3;
                // Bursts that land while later blocks still stream K/V (more than one round
                // of blocks) go out non-temporally: a dirty line parked in L2 is evicted on
                // its own later and interrupts a read stream each time.  With a single round
                // all bursts come at the very end and ordinary stores are cheaper.
                if (p.stream_scores) {
                    for (int i = tid * 4; i < rows4; i += blockDim.x * 4)
                        store16_stream(dst + i, *reinterpret_cast<const uint4 *>(src + i));
                } else {
                    for (int i = tid * 4; i < rows4; i += blockDim.x * 4)
                        *reinterpret_cast<float4 *>(dst + i) = *reinterpret_cast<const float4 *>(src + i);
                }
                if (tid < rows - rows4) dst[rows4 + tid] = src[rows4 + tid];
            } else {
                for (int i = tid; i < rows; i += blockDim.x) dst[i] = src[i];
            }
        }
    }

    // ... then the waves of the block, and write the block's partial.
    for (int idx = tid; idx < GB * W; idx += blockDim.x) {
        const int g = idx / W, d = idx - g * W;
        float M = sm_m[0][g];
#pragma unroll
        for (int w = 1; w < kWavesPerBlock; ++w) M = fmaxf(M, sm_m[w][g]);
        float a = 0.0f, L = 0.0f;
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) {
            const float f = sm_m[w][g] == -INFINITY ? 0.0f : __expf(sm_m[w][g] - M);
            a = fmaf(sm_acc[w][g][d], f, a);
            L = fmaf(sm_l[w][g], f, L);
        }
        p.part_acc[(part_base + g * part_head_stride) * W + d] = a;
        if (d == 0) {
            p.part_ml[(part_base + g * part_head_stride) * 2 + 0] = M;
            p.part_ml[(part_base + g * part_head_stride) * 2 + 1] = L;
        }
    }
}

// ---------------------------------------------------------------------------------------
// Grouped-query variant on the matrix cores (bf16 rows of W values, one routing decision per
// token, 2..64 query rows per kv head: the heads of the group times the draft queries of a
// multi-query step).  With G query rows sharing every K/V byte the plain-ALU kernel above
// spends ~G times more instructions per byte and stops being memory-bound; here the G rows
// (padded to whole tiles of 16) form one dimension of 16x16x32 bf16 MFMA tiles, so the
// instruction count per byte does not depend on G within a row tile.
//
// Per wave and per tile of entries (sub-tiles of 32):
//   * K rows arrive with coalesced 16-byte lane loads and make one trip through a padded
//     wave-private LDS tile (write row-major, read one entry per lane); Q sits in registers.
//     S^T[entry][row] = K . Q^T: lane (query row c = lane % 16, group r = lane / 16) ends up
//     with the scores of entries 4r..4r+3 and 16+4r..16+4r+3 of the sub-tile.
//   * The order of the contraction index of an MFMA is free as long as both operands agree on
//     it.  With entry order e(r, 0..7) = {4r..4r+3, 16+4r..16+4r+3} those scores, turned into
//     probabilities, ARE the lane's slice of the operand P^T[entry][row] of the second product:
//     nothing moves between lanes.  (They are split into bf16 parts, see kProbParts.)
//   * O^T[d][row] += V^T . P^T.  V needs no transpose either: lane (c, r) loads the rows e(r, t)
//     of the sub-tile, W/8 bytes of each, and output set i takes the i-th value of each of its
//     own 8 rows (packed by byte-permutes).  The accumulators of lane (c, r) belong to query row
//     c, like the lane's scores: the online-softmax rescale is lane-local.
// Bound by memory up to 16 rows per kv head; by then the plain-ALU kernel is bound by vector issue.
// Measured, pass and merge, 128 MiB of K/V (64 MiB for rank 16 and the 64-row group), against the
// kernel that took the shape before: rows of 64 values x 8 heads 55.2 -> 33.8 us, x 3 heads (which
// streamed K/V once per head) 56.9 -> 30.6, x 32 heads 430 -> 53, x 64 heads 318 -> 43; rank-32
// codes x 4 heads 42.7 -> 37.8, x 16 heads 127 -> 34; rank 64 x 4 heads (256 MiB) 69.7 -> 58.8, rank
// 16 x 4 heads 28.9 -> 25.1; even at 2 heads.  Rows of 128 values (before: probabilities through
// LDS) x 4 heads 29.7 -> 29.1, 8 heads 35.0 -> 31.8, 64 rows 45.1 -> 41.6.
constexpr int kSubTile = 32;
constexpr int gqa_tile(int width, int row_tiles) {
    if (width == 128 || (width == 64 && row_tiles == 4)) return kSubTile;
    return kSubTile * (width == 16 ? 4 : 2);
}

// Bytes per staged K row: the row plus 16 of padding, so that the 16 lanes reading one 16-byte
// column of 16 different rows do not all start in the same bank.
template <int W, int RT>
struct RowShape {
    static constexpr int kRowBytes = 2 * W;
    static constexpr int kPitch = kRowBytes + 16;
    static constexpr int kKLanes = kRowBytes / 16;         // lanes of a K load that cover one row
    static constexpr int kKRows = kWave / kKLanes;         // rows of a K load
    // sub-tiles per tile: 16 KiB of K and V rows in flight per wave, 8 KiB for codes of rank 32
    // and 16 (four blocks per CU instead of three, as in the plain-ALU kernel)
    static constexpr int kTile = gqa_tile(W, RT);
    static constexpr int kSubs = kTile / kSubTile;
    static constexpr int kKLoads = kTile / kKRows;
    // V per sub-tile: 8 loads of W/8 bytes.  W = 16: 2 bytes would be left for a lane; there lanes
    // m < 8 and m + 8 load the same word of two neighbouring rows (4 loads) and swap halves.
    static constexpr bool kPairs = W == 16;
    static constexpr int kVLoads = kPairs ? 4 : 8;
    static constexpr int kVWords = kPairs ? 1 : kRowBytes / 64;      // 32-bit words per load
    static constexpr int kSets = W / 16;                   // output sets
    static constexpr int kQSteps = W >= 32 ? W / 32 : 1;   // MFMA steps of a score
    // row t of the lane's loads, relative to its first (entry e(r, t) or, in pairs, e(r, 2t))
    static constexpr int v_step(int t) { return kPairs ? (t & 1) * 2 + (t >> 1) * 16 : (t & 3) + (t >> 2) * 16; }
};

// A lane's slice of an MFMA operand with contraction length 32 (8 values), or 16 for rows of 16
// values (4 values).
template <int W>
struct OperandOf {
    typedef uint4 type;
};
template <>
struct OperandOf<16> {
    typedef uint2 type;
};

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// max over the four lanes c, c + 16, c + 32, c + 48, in all of them, without LDS: the swaps leave
// the two halves (then the two rows of each half) side by side in two registers.
__device__ __forceinline__ float group_max(float x) {
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
    const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

// fp32 values (8 for uint4, 4 for uint2) as PARTS bf16 operands whose sum they are: each part
// rounds what the parts before it left (2 parts carry 16 bits of a value, 3 parts all 24).
template <int PARTS, typename OP>
__device__ __forceinline__ void split_bf16(const float *v, OP (&out)[PARTS]) {
    constexpr int NW = sizeof(OP) / 4;
    struct Words {
        uint32_t w[NW];
    } words[PARTS];
#pragma unroll
    for (int u = 0; u < NW; ++u) {
        f32x2_t rest = {v[2 * u], v[2 * u + 1]};
#pragma unroll
        for (int k = 0; k < PARTS; ++k) {
            const bf16x2_t part = __builtin_convertvector(rest, bf16x2_t);
            words[k].w[u] = __builtin_bit_cast(uint32_t, part);
            if (k + 1 < PARTS) rest = rest - f32x2_t{(float)part[0], (float)part[1]};
        }
    }
#pragma unroll
    for (int k = 0; k < PARTS; ++k) out[k] = __builtin_bit_cast(OP, words[k]);
}

// 8 probabilities as 3 parts, each the leading 8 bits of what is left: all 24 bits, none of the parts
// negative, and one that would be zero is the smallest normal number.  An infinite value of V then
// gives the infinity of the unsplit product, where a zero or a negative part would make it NaN.
// (The lift adds 2^-126 of a value of V.)
__device__ __forceinline__ void split_bf16_up(const float *v, uint4 (&out)[3]) {
    typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
    auto upper = [](float hi, float lo) { return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u); };
    auto rest = [](float x) { return x - __uint_as_float(__float_as_uint(x) & 0xffff0000u); };
    auto lift = [](uint32_t part) {
        const u16x2_t least = {0x0080, 0x0080};
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, part), least));
    };
    uint32_t w[3][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const float a = v[2 * u], b = v[2 * u + 1], a1 = rest(a), b1 = rest(b);
        w[0][u] = upper(b, a);
        w[1][u] = lift(upper(b1, a1));
        w[2][u] = lift(upper(rest(b1), rest(a1)));
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) out[k] = make_uint4(w[k][0], w[k][1], w[k][2], w[k][3]);
}


// Consecutive bf16 query values as an operand; a caller's q need not be 16-byte aligned.
template <typename OP>
__device__ __forceinline__ OP load_query(const bf16 *q, bool aligned) {
    if (aligned) return *reinterpret_cast<const OP *>(q);
    struct {
        uint16_t v[sizeof(OP) / 2];
    } parts;
#pragma unroll
    for (unsigned i = 0; i < sizeof(OP) / 2; ++i) parts.v[i] = q[i].bits;
    return __builtin_bit_cast(OP, parts);
}

__device__ __forceinline__ void hold_operand(uint4 &v) {
    asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
}
__device__ __forceinline__ void hold_operand(uint2 &v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }

// RT = number of 16-row tiles the query group occupies (group rows = query heads per kv head
// times the draft queries of a multi-query step): 1, 2 or 4.  Every row tile reuses the K tile
// staged in LDS and the V rows in registers, so the streamed bytes do not grow with RT; the
// accumulators do (W/4 registers per row tile), which is why a CU holds 3 blocks at RT = 1 and 2
// above.  For RT = 4 the query operands live in LDS instead of registers.
// (The least; rows of 32 values at two row tiles without scores have registers for one more.)
constexpr int gqa_blocks_per_cu(int width, int row_tiles, bool codes) {
    if (codes && width == 64 && row_tiles == 4) return 1;      // 96 registers of query operand
    if (width <= 32) return row_tiles == 1 ? 4 : row_tiles == 2 ? 3 : 2;
    return row_tiles == 1 ? 3 : 2;
}
// LONG: rows of 128 values in the plan of a block per CU.  A wave takes up to 256 rows in a row, fewer of its weights are its
// running maximum - which is 1, and exact in any number of parts - and with two parts y would be further off 64 bits than in
// short blocks (64 units of 4096 slots 2.0e-6 against 1.8e-6).  A third part makes it 2.0e-7; its registers are there
// where a CU holds two blocks.  (Fused step 37.0 us in short blocks, 36.2 in long ones, so 36.6; half full 29.4, 27.4, 27.9.
// For every plan of these rows it would cost 1 - 2 %: 1 x 8 x 4 units of 8192 slots 36.4 -> 36.9.)
constexpr int kGqaLongBlocksPerCu = 2;
// CODES: the rows are rank-W codes.  Their query is U_K q, formed in fp32 by MFMAs in the kernel's
// prologue - W/16 tiles of (code column, query row), whose result layout is again the operand
// layout up to the order of the contraction index - and split into 3 bf16 parts, so that its
// products with the codes stay exact to 24 bits.
template <int W, int RT, bool CODES, bool LONG>
struct GqaShape {
    static constexpr bool kQueryInLds = W == 128 && RT > 2;
    // W = 128, RT = 4: the 128 accumulator registers leave no room to hold the next K tile across
    // the whole tile's arithmetic; K is then loaded where it is used and the CU's other waves hide
    // the latency (at four row tiles the kernel is bound by the matrix cores, not by memory).
    static constexpr bool kPrefetchK = !kQueryInLds;
    static constexpr int kQueryParts = CODES ? 3 : 1;
    // The lane's part of the row addresses is formed again for each tile instead of held (4 registers):
    // where the shape would spill otherwise.
    static constexpr bool kLeanAddresses = CODES && ((W == 64 && RT == 1) || (W == 16 && RT == 4));
    // Probabilities: 3 parts are the fp32 value, 2 parts differ from it by 2^-17.  Rows of 128
    // values have always used 2 (y is 1.8e-6 off 64 bits), but for LONG blocks; the narrower rows were summed in fp32
    // on the vector units and keep that: y against 64 bits 1.5 - 1.8e-7 (64 values) and 1.8 - 2.5e-7
    // (codes), from 1.5 - 1.8e-7 and 2.0 - 2.6e-7, with the two small parts summed apart from the
    // running output (added to it part by part: up to 2.8e-7).  At one row tile, whose waves take up to 8 tiles
    // in a row, the large part is summed apart too: 128 units of 4096 slots of 64 values 1.76e-7, accumulated onto the
    // small parts 2.02e-7, onto the running output 2.16e-7; rank-16 codes 2.00, 2.22 and 2.36e-7, rank 64 2.39, 2.61, 2.68e-7.
    static constexpr int kProbParts = W == 128 && !LONG ? 2 : 3;
};

// LDS a block holds besides the score stage: a K tile per wave and the wave statistics, and the
// query tile at four row tiles.
constexpr size_t gqa_static_lds(int width, int tile, int row_tiles) {
    return (size_t)kWavesPerBlock * (tile * (2 * width + 16) + 2 * 16 * 4) +
           (width == 128 && row_tiles == 4 ? (size_t)64 * (2 * width + 16) : 16);
}

// SC: what happens to the raw scores - kScoresNone (not asked for), kScoresStaged (kept in LDS,
// one burst per row at the block's end) or kScoresDirect (written from the loop).  A template
// parameter and not a run-time branch: each form costs registers, and a value spilled for one
// of them is reloaded inside the loop by a scratch load, which the wait counters cannot tell
// from the tile loads in flight - the wave then waits for all of them.  (One form of the 44 still
// spills: rank-16 codes at four row tiles with scores written from the loop, 24 bytes.)
constexpr int kScoresNone = 0, kScoresStaged = 1, kScoresDirect = 2;
template <int W, int RT, int SC, bool CODES, bool LONG>
__global__ __launch_bounds__(kWavesPerBlock *kWave, LONG ? kGqaLongBlocksPerCu : gqa_blocks_per_cu(W, RT, CODES)) void attn_partial_gqa(
    AttnParams p) {
    using Row = RowShape<W, RT>;
    constexpr int TILE = Row::kTile, SUBS = Row::kSubs, SETS = Row::kSets, PITCH = Row::kPitch;
    using Shape = GqaShape<W, RT, CODES, LONG>;
    typedef typename OperandOf<W>::type Operand;
    constexpr bool QLDS = Shape::kQueryInLds;
    constexpr bool KPRE = Shape::kPrefetchK;
    constexpr int PP = Shape::kProbParts, QP = Shape::kQueryParts, KS = Row::kQSteps;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid >> 6;
    const int c = lane & 15;
    const int r = lane >> 4;
    const int gb = p.G;                       // rows per block = the whole query group

    // (the plain-ALU kernel above measures 2.6 % slower with a contiguous range per XCD)
    int split, j, hk;
    int bid = group_block(p, &split);
    int b;
    if constexpr (RT < 4) {
        bid = fast_divide(p.by_k, bid, &j);
        b = fast_divide(p.by_groups, bid, &hk);
    } else {                                  // (two registers spill here with fast_divide)
        j = bid % p.k;
        bid /= p.k;
        const int hgroups = p.Hq / gb;
        hk = bid % hgroups;
        b = bid / hgroups;
    }
    const int h0 = hk * gb;

    // Query operand of row tile rt: lane (row c, group r) holds Q[row rt*16 + c][32 s + 8 r .. +7]
    // (codes: columns 32 s + 4 r .. +3 and 32 s + 16 + 4 r .. +3; rows of 16 values: 4 r .. +3).
    // The group's rows are the query rows h0 .. h0 + gb - 1 of the sequence; query_row() maps a
    // group row to where the caller keeps it.  Rows past the group repeat the last one; nothing
    // reads what they lead to.
    const bool q_aligned = (reinterpret_cast<uintptr_t>(p.q) & 15) == 0;
    auto query = [&](int rt) {
        return static_cast<const bf16 *>(p.q) + query_row(p, b, hk, min(rt * 16 + c, gb - 1)) * p.D;
    };
    constexpr int DS = CODES ? 4 : 1;          // steps of 32 over the head dimension (D <= 128)
    Operand qop[QLDS ? 1 : RT][KS][QP];
    uint4 q_raw[CODES ? RT : 1][DS], u_raw[CODES ? W / 16 : 1][DS];
    if constexpr (CODES) {
        // what the projection reads is requested ahead of everything: loads come back in order,
        // and behind a tile's rows it would hold the first scores up (31.7 -> 31.4 us for 128 MiB
        // of rank-32 codes; the plain query, requested here, costs 0.7 us instead)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int s = 0; s < DS; ++s) q_raw[rt][s] = load_query<uint4>(query(rt) + min(32 * s + 8 * r, p.D - 8), q_aligned);
        const bf16 *U = static_cast<const bf16 *>(p.U_K) + ((int64_t)hk * W + c) * p.D;
#pragma unroll
        for (int ct = 0; ct < W / 16; ++ct)
#pragma unroll
            for (int s = 0; s < DS; ++s) u_raw[ct][s] = load16(U + (int64_t)16 * ct * p.D + min(32 * s + 8 * r, p.D - 8));
    }
    const ShardRef sh = resolve_shard(p, b, b, j, lane);
    int r0, r1;
    split_rows<TILE>(p, sh.n, split, &r0, &r1);

    __shared__ __attribute__((aligned(16))) unsigned char lds_k[kWavesPerBlock][TILE * PITCH];
    __shared__ float sm_m[kWavesPerBlock][16];
    __shared__ float sm_l[kWavesPerBlock][16];
    __shared__ __attribute__((aligned(16))) unsigned char lds_q[QLDS ? RT * 16 * PITCH : 16];
    // Raw scores of the block's rows, [rows of the group][chunk], when p.stage_scores (see
    // attn_partial): written to memory in one contiguous burst per row after the streaming loop.
    extern __shared__ __attribute__((aligned(16))) float gqa_stage[];

    const int64_t part_base = (((int64_t)b * p.Hq + h0) * p.k + j) * p.nsplit + split;
    const int64_t part_head_stride = (int64_t)p.k * p.nsplit;

    if (r0 >= r1) {
        for (int idx = tid; idx < gb * (W / 4); idx += blockDim.x) {
            const int g = idx / (W / 4), d = (idx - g * (W / 4)) * 4;
            const int64_t at = part_base + g * part_head_stride;
            *reinterpret_cast<float4 *>(p.part_acc + at * W + d) = make_float4(0.f, 0.f, 0.f, 0.f);
            if (d == 0) *reinterpret_cast<float2 *>(p.part_ml + at * 2) = make_float2(-INFINITY, 0.f);
        }
        return;
    }

    const char *Kb = sh.K + (int64_t)hk * p.stride_h * 2;
    const char *Vb = sh.V + (int64_t)hk * p.stride_h * 2;
    // Byte offsets of the lane's rows from the kv head's base, in 32 bits (the host admits this
    // kernel only where a shard's fit): rows past the end are clamped onto the last valid row - one
    // minimum per load, no branch around any - and masked out of the softmax.  The requests run up to
    // five tiles past the end, so the sums saturate instead of wrapping: with terms of at most the
    // S - 1 rows below a shard's last, a sum that does not fit lies past it.  (Two forms of the loads, full tiles from
    // a wave-uniform base and clamped ones for the last tile, cost 20 registers more: 124 bytes of
    // spills at one row tile of 128 values.)
    const uint32_t rb = (uint32_t)(p.stride_s * 2);
    const int k_row = lane / Row::kKLanes;
    const uint32_t k_col = 16u * (lane & (Row::kKLanes - 1));
    const uint32_t last = (uint32_t)(r1 - 1) * rb;

    // (Each tile's offset is hidden from the optimiser: it would otherwise carry one running
    // address per load through the loop, 16 registers instead of one.)
    auto opaque = [](uint32_t v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    uint4 kr[Row::kKLoads];
    uint32_t vr[SUBS][Row::kVLoads][Row::kVWords];
    const int row_most = p.S - 1;
    auto rows_bytes = [&](int rows) { return (uint32_t)min(rows, row_most) * rb; };
    auto sum = [](uint32_t a, uint32_t b) { return __builtin_elementwise_add_sat(a, b); };
    auto load_k = [&](int t0) {
        const int ln = Shape::kLeanAddresses ? opaque(lane) : lane;
        const uint32_t col = 16u * (ln & (Row::kKLanes - 1));
        const uint32_t at = opaque(sum(rows_bytes(t0), rows_bytes(ln / Row::kKLanes) + col));
#pragma unroll
        for (int t = 0; t < Row::kKLoads; ++t)
            kr[t] = load16_stream(Kb + (size_t)min(sum(at, rows_bytes(t * Row::kKRows)), last + col));
    };
    auto load_v = [&](int t0) {
        const int ln = Shape::kLeanAddresses ? opaque(lane) : lane;
        const uint32_t col = 4u * Row::kVWords * (ln & (Row::kPairs ? 7 : 15));
        const uint32_t at = opaque(sum(rows_bytes(t0), rows_bytes(4 * (ln >> 4) + (Row::kPairs ? (ln & 15) >> 3 : 0)) + col));
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
            for (int t = 0; t < Row::kVLoads; ++t)
                load_words_stream<Row::kVWords>(
                    vr[sub][t], Vb + (size_t)min(sum(at, rows_bytes(sub * kSubTile + Row::v_step(t))), last + col));
    };
    if constexpr (!CODES && !QLDS) {         // ahead of the tile's rows: loads come back in order
        auto load_q = [&](auto aligned) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    qop[rt][s][0] = load_query<Operand>(query(rt) + 32 * s + (W >= 32 ? 8 : 4) * r, aligned);
        };
        if (q_aligned) load_q(std::true_type{});
        else load_q(std::false_type{});
    }
    int t0 = r0 + __builtin_amdgcn_readfirstlane(wave) * TILE;
    if constexpr (KPRE) load_k(t0);           // (a wave without rows loads the last one)
    load_v(t0);

    if constexpr (CODES) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            float proj[W / 4];               // proj[4 ct + x]: code column 16 ct + 4 r + x of row c
#pragma unroll
            for (int ct = 0; ct < W / 16; ++ct) {
                f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < DS; ++s) {
                    uint4 qv = q_raw[rt][s];
                    if (32 * s + 8 * r >= p.D) qv = make_uint4(0, 0, 0, 0);
                    acc = mfma_rows(u_raw[ct][s], qv, acc);
                }
#pragma unroll
                for (int x = 0; x < 4; ++x) proj[4 * ct + x] = acc[x] * p.scale;
            }
#pragma unroll
            for (int s = 0; s < KS; ++s) split_bf16(proj + 8 * s, qop[rt][s]);
        }
    } else if constexpr (QLDS) {
        for (int idx = tid; idx < RT * 16 * (W / 8); idx += blockDim.x) {     // (row, 16-byte chunk)
            const int row = idx / (W / 8), ch = idx % (W / 8);
            *reinterpret_cast<uint4 *>(lds_q + row * PITCH + 16 * ch) = load_query<uint4>(
                static_cast<const bf16 *>(p.q) + query_row(p, b, hk, min(row, gb - 1)) * W + 8 * ch, q_aligned);
        }
        __syncthreads();
    }
    // Every operand the loop keeps is complete here: a wait for it inside the loop would be a wait
    // for the tile loads requested after it.
    if constexpr (!QLDS) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int k = 0; k < QP; ++k) hold_operand(qop[rt][s][k]);
    }
    // the same slice of a staged K row
    auto k_operand = [&](const unsigned char *row, int s) {
        Operand a;
        if constexpr (W == 16) {
            a = *reinterpret_cast<const uint2 *>(row + 8 * r);
        } else if constexpr (CODES) {
            const uint2 lo = *reinterpret_cast<const uint2 *>(row + 64 * s + 8 * r);
            const uint2 hi = *reinterpret_cast<const uint2 *>(row + 64 * s + 32 + 8 * r);
            a = make_uint4(lo.x, lo.y, hi.x, hi.y);
        } else {
            a = *reinterpret_cast<const uint4 *>(row + 64 * s + 16 * r);
        }
        return a;
    };

    float m[RT], lsum[RT];                  // running max / partial sum of row rt*16 + c
    f32x4_t oacc[RT][SETS];                 // oacc[rt][i][x] = O[row rt*16 + c][out_col(x, i)]
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        m[rt] = -INFINITY;
        lsum[rt] = 0.0f;
#pragma unroll
        for (int i = 0; i < SETS; ++i) oacc[rt][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }

    auto out_col = [&](int x, int i) {
        const int mm = 4 * r + x;
        return Row::kPairs ? 2 * (mm & 7) + (mm >> 3) : SETS * mm + i;
    };
    const uint32_t pair_sel = c < 8 ? 0x05040100u : 0x03020706u;   // W = 16: low halves, or high halves

    unsigned char *kst = lds_k[wave];
    // The order of a wave's requests is the same on every path - K of the next tile, V of the next
    // tile, K ... - and no request sits under a condition inside the loop: the wait for a tile's K
    // is then a wait for those loads alone, with its V still in flight.  (With the two prefetches
    // under `if (tnext < r1)` the compiler had to allow for K without V and waited for both.)
    if (t0 < r1) do {
        const int tnext = t0 + kWavesPerBlock * TILE;

        // K rows -> LDS (row-major, padded), then the next tile's K loads reuse the registers
        if constexpr (!KPRE) {
            load_k(t0);                      // K where it is used
        }
#pragma unroll
        for (int t = 0; t < Row::kKLoads; ++t)
            *reinterpret_cast<uint4 *>(kst + (t * Row::kKRows + k_row) * PITCH + k_col) = kr[t];
        if constexpr (KPRE) load_k(tnext);   // past the end: the clamped last row once more
        wave_lds_order();

#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            if (rt * 16 >= gb) break;        // row tiles past the group (wave-uniform)
            // S^T = K Q^T, 16 entries at a time; sv[8 sub + 4 hb + x] is the score of entry
            // t0 + 32 sub + 16 hb + 4 r + x
            float sv[8 * SUBS];
#pragma unroll
            for (int hb = 0; hb < 2 * SUBS; ++hb) {
                f32x4_t sc = f32x4_t{0.f, 0.f, 0.f, 0.f};
                Operand a[KS];
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    a[s] = k_operand(kst + (16 * hb + c) * PITCH, s);
                    if constexpr (QLDS)
                        sc = mfma_rows(a[s], *reinterpret_cast<const uint4 *>(lds_q + (rt * 16 + c) * PITCH + 64 * s + 16 * r),
                                       sc);
                }
                if constexpr (QP > 1) {
                    // The small parts first, and kept finite: an infinite code against a part that is zero
                    // or of the other sign is NaN, where the unsplit query scores an infinity (-Inf: the
                    // entry drops out of the softmax).  (The median of a NaN and two numbers is a number.)
#pragma unroll
                    for (int k = QP - 1; k >= 1; --k)
#pragma unroll
                        for (int s = 0; s < KS; ++s) sc = mfma_rows(a[s], qop[rt][s][k], sc);
#pragma unroll
                    for (int x = 0; x < 4; ++x) sc[x] = __builtin_amdgcn_fmed3f(sc[x], -3e38f, 3e38f);
                }
                if constexpr (!QLDS) {
#pragma unroll
                    for (int s = 0; s < KS; ++s) sc = mfma_rows(a[s], qop[rt][s][0], sc);
                }
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int row = t0 + 16 * hb + 4 * r + x;
                    const float score = CODES ? sc[x] : sc[x] * p.scale;
                    sv[4 * hb + x] = row < r1 ? score : -INFINITY;
                }
            }
            const int row_g = rt * 16 + c;   // row of the group this lane's scores belong to
            if (SC == kScoresStaged && row_g < gb) {
                // [row of the group][row of the block]: chunk is a multiple of the tile, so the
                // float4 stores stay aligned
                float *dst = gqa_stage + row_g * p.chunk + (t0 - r0) + 4 * r;
#pragma unroll
                for (int hb = 0; hb < 2 * SUBS; ++hb)
                    *reinterpret_cast<float4 *>(dst + 16 * hb) =
                        make_float4(sv[hb * 4], sv[hb * 4 + 1], sv[hb * 4 + 2], sv[hb * 4 + 3]);
            } else if (SC == kScoresDirect) {
                // Whole 128-byte lines: lanes c and c + 8 swap halves, so that one store covers
                // 32 entries of 8 rows instead of 16 entries of 16.
                const bool upper = c >= 8;
#pragma unroll
                for (int sub = 0; sub < SUBS; ++sub) {
                    float va[4], vb[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const float lo = sv[8 * sub + x], hi = sv[8 * sub + 4 + x];
                        const float got = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(upper ? lo : hi), 0x128, 0xf, 0xf, true));
                        va[x] = upper ? got : lo;
                        vb[x] = upper ? hi : got;
                    }
                    const int first = 32 * sub + (upper ? 16 : 0) + 4 * r;
                    const int row = t0 + first;
                    float *dst = p.scores + (((int64_t)b * p.Hq + h0 + rt * 16 + (c & 7)) * p.k + j) * p.S + row;
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        const float *v = half ? vb : va;
                        float *to = dst + (int64_t)half * 8 * p.k * p.S;
                        if (rt * 16 + half * 8 + (c & 7) < gb) {
                            if (row + 4 <= r1 && (p.S & 3) == 0) {
                                *reinterpret_cast<float4 *>(to) = make_float4(v[0], v[1], v[2], v[3]);
                            } else {
#pragma unroll
                                for (int x = 0; x < 4; ++x)
                                    if (row + x < r1) to[x] = v[x];
                            }
                        }
                    }
                }
            }

            // online softmax for row c of this tile (its entries are spread over the 4 lane groups)
            float tm = sv[0];
#pragma unroll
            for (int x = 1; x < 8 * SUBS; ++x) tm = fmaxf(tm, sv[x]);
            const float mn = fmaxf(m[rt], group_max(tm));
            if (__any(mn > m[rt])) {         // else the factor is 1 in every lane
                const float corr = __expf(m[rt] - mn);
                m[rt] = mn;
                lsum[rt] *= corr;
#pragma unroll
                for (int i = 0; i < SETS; ++i)
#pragma unroll
                    for (int x = 0; x < 4; ++x) oacc[rt][i][x] *= corr;
            }
#pragma unroll
            for (int x = 0; x < 8 * SUBS; ++x) sv[x] = __expf(sv[x] - mn);
            // At one row tile the tile's weights and products are summed apart and meet the running sums in one addition: a
            // wave's rows may be many (blocks of 512 KiB, which are planned for one row tile alone), and each rounding of a
            // running sum is one of the whole sum's size.  At two and four the temporaries cost registers: rows of 16 values
            // x 64 heads 57.7 us, apart 80.8 (224 bytes of scratch), rank-32 codes 74.7 and 99.7.  (Rows of 128 values have
            // them for the weights.)
            if constexpr (RT == 1 || W == 128) {
                float tl = 0.f;
#pragma unroll
                for (int x = 0; x < 8 * SUBS; x += 4) tl += (sv[x] + sv[x + 1]) + (sv[x + 2] + sv[x + 3]);
                lsum[rt] += tl;
            } else {
#pragma unroll
                for (int x = 0; x < 8 * SUBS; ++x) lsum[rt] += sv[x];
            }
            // O^T += V^T P^T, output set i takes the i-th value of each of the lane's 8 V rows
#pragma unroll
            for (int sub = 0; sub < SUBS; ++sub) {
                uint4 pop[PP];
                if constexpr (PP == 3) split_bf16_up(sv + 8 * sub, pop);
                else split_bf16(sv + 8 * sub, pop);
                const auto &v = vr[sub];
#pragma unroll
                for (int i = 0; i < SETS; ++i) {
                    uint4 vop;
                    if constexpr (Row::kPairs) {
                        auto both = [&](uint32_t mine) {
                            const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mine, 0x128, 0xf, 0xf, true);
                            return __builtin_amdgcn_perm(other, mine, pair_sel);
                        };
                        vop = make_uint4(both(v[0][0]), both(v[1][0]), both(v[2][0]), both(v[3][0]));
                    } else {
                        const uint32_t sel = (i & 1) ? 0x07060302u : 0x05040100u;
                        vop = make_uint4(__builtin_amdgcn_perm(v[1][i >> 1], v[0][i >> 1], sel),
                                         __builtin_amdgcn_perm(v[3][i >> 1], v[2][i >> 1], sel),
                                         __builtin_amdgcn_perm(v[5][i >> 1], v[4][i >> 1], sel),
                                         __builtin_amdgcn_perm(v[7][i >> 1], v[6][i >> 1], sel));
                    }
                    if constexpr (PP == 3) {
                        f32x4_t small = mfma_rows(vop, pop[2], f32x4_t{0.f, 0.f, 0.f, 0.f});
                        small = mfma_rows(vop, pop[1], small);
                        // (onto zero: what a product adds to its third operand it cuts to that operand's last place)
                        if constexpr (RT == 1) oacc[rt][i] += mfma_rows(vop, pop[0], f32x4_t{0.f, 0.f, 0.f, 0.f}) + small;
                        else oacc[rt][i] = mfma_rows(vop, pop[0], oacc[rt][i]) + small;
                    } else {
                        oacc[rt][i] = mfma_rows(vop, pop[0], mfma_rows(vop, pop[1], oacc[rt][i]));
                    }
                }
            }
        }
        wave_lds_order();                    // the K tile is rewritten by the next iteration
        load_v(tnext);
        t0 = tnext;
    } while (t0 < r1);

    __syncthreads();
    if (SC == kScoresStaged) {   // the block's scores: one burst per row of the group
        const int rows = r1 - r0, rows4 = rows & ~3;
        for (int g = wave; g < gb; g += kWavesPerBlock) {      // a row per wave
            float *dst = p.scores + (((int64_t)b * p.Hq + h0 + g) * p.k + j) * p.S + r0;
            const float *src = gqa_stage + g * p.chunk;
            if ((p.S & 3) == 0 && (reinterpret_cast<uintptr_t>(p.scores) & 15) == 0) {
                // (Non-temporal stores where blocks run in several rounds, as in attn_partial, are 3 %
                // faster there, 508 -> 491 us, but the second form costs the single round 1 us of 42.)
                for (int i = lane * 4; i < rows4; i += kWave * 4)
                    *reinterpret_cast<float4 *>(dst + i) = *reinterpret_cast<const float4 *>(src + i);
                if (lane < rows - rows4) dst[rows4 + lane] = src[rows4 + lane];
            } else {
                for (int i = lane; i < rows; i += kWave) dst[i] = src[i];
            }
        }
    }

    // per row tile: wave results -> LDS (the wave's own K staging area is free now), then merge
    // the waves and write the block's partial.  Rows are padded by 4 floats (banks).
    constexpr int AP = W + 4;
    static_assert(16 * AP * 4 <= TILE * PITCH, "the wave's results fit its K staging area");
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        if (rt * 16 >= gb) break;
        const int rows_here = min(16, gb - rt * 16);
        float ls = lsum[rt];
        ls += __shfl_xor(ls, 16, kWave);
        ls += __shfl_xor(ls, 32, kWave);
        float *wacc = reinterpret_cast<float *>(kst) + c * AP;
        if (c < rows_here) {
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int i = 0; i < SETS; ++i) wacc[out_col(x, i)] = oacc[rt][i][x];
        }
        if (r == 0) {
            sm_m[wave][c] = m[rt];
            sm_l[wave][c] = ls;
        }
        __syncthreads();
        // Four values per thread: value by value the factors were formed four times as often and the partials, 16 KiB
        // per block at 32 rows of 128 values, left in 4-byte stores (pass and merge, 1 x 8 kv heads x 4 shards of 8192: 32 rows
        // 48.1 -> 45.7 us, 64 rows over 4 kv heads 42.7 -> 39.4, 4 rows 30.3 -> 30.2; with the query rows found without
        // compiler divisions 44.2 and 38.3).
        constexpr int V = 4;
        typedef float values __attribute__((ext_vector_type(V)));
        for (int idx = (int)opaque((uint32_t)tid); idx < rows_here * (W / V); idx += blockDim.x) {
            const int g = idx / (W / V), d = (idx - g * (W / V)) * V;
            float M = sm_m[0][g];
#pragma unroll
            for (int w2 = 1; w2 < kWavesPerBlock; ++w2) M = fmaxf(M, sm_m[w2][g]);
            values a = 0.0f;
            float L = 0.0f;
#pragma unroll
            for (int w2 = 0; w2 < kWavesPerBlock; ++w2) {
                const float f = sm_m[w2][g] == -INFINITY ? 0.0f : __expf(sm_m[w2][g] - M);
                const values o = *reinterpret_cast<const values *>(reinterpret_cast<const float *>(lds_k[w2]) + g * AP + d);
#pragma unroll
                for (int i = 0; i < V; ++i) a[i] = fmaf(o[i], f, a[i]);
                L = fmaf(sm_l[w2][g], f, L);
            }
            const int64_t at = part_base + (rt * 16 + g) * part_head_stride;
            *reinterpret_cast<values *>(p.part_acc + at * W + d) = a;
            if (d == 0) *reinterpret_cast<float2 *>(p.part_ml + at * 2) = make_float2(M, L);
        }
        if (rt + 1 < RT) __syncthreads();    // the staging areas are rewritten by the next row tile
    }
}

// ---------------------------------------------------------------------------------------
// Grouped queries over fp32 rows on the matrix cores: up to 16 heads of a group share every K/V byte as
// one side of 16x16x4 fp32 products (full fp32 multiply-adds, one routing decision per token).
//
// Per wave and 16 entries, lane (c, r) = (lane % 16, lane / 16):
//   * S^T[entry][head] = K . Q^T.  The order of the contraction is free: product i of step s takes the
//     dimensions {16 s + 4 r + i}, so that a lane's operands are 16-byte pieces of row c - K is requested in
//     that form (64 bytes of a row per load, the next load the line's other half) and needs no LDS.  The four i, and
//     the steps, are summed apart and joined pairwise.
//   * The lane's scores are those of entries 4r .. 4r+3 and head c, and product i of the second
//     contraction takes the entries {4 r + i}: its operand is the lane's own i-th probability.  The
//     operand of V is the i-th of four rows, loaded as such.
//   * The four products of 16 entries are summed apart, pairwise, and then added to the running output (in one
//     chain: y 1.89 - 2.42e-7 off 64 bits; so 1.82 - 2.32e-7, the plain kernel 1.83 - 2.39e-7).
// Codes: the projected query U_K q comes out of the same products in operand form, each wave over a quarter
// of the head dimension, joined in LDS.
// The plain kernel above spends 4 multiply-adds and a reduction over 4 - 32 lanes per head and row piece:
// with 4 and 8 heads it was bound by vector issue, and at 8 it left one wave per SIMD (252 registers);
// groups of other than 2, 4 and 8 heads streamed K/V once per head.
// Measured, pass and merge with scores, against the plain kernel: 8 heads over rows of 128 values (512 MiB) 146 -> 107 us,
// of 64 127 -> 110, 3 heads of 128 169 -> 97, 16 heads 1030 -> 115, 6 heads (256 MiB) 134 -> 59, 32 heads (128 MiB) 387 -> 62;
// rank-64 codes x 8 heads (100 MiB) 51 -> 39.  Groups of two and four stay there, see kGqa32Heads.
constexpr int gqa32_tile(int width) { return width >= 128 ? 16 : width == 64 ? 32 : 64; }
constexpr int kGqa32BlocksPerCu = 3;
// Rows of 4 floats more than W: banks.
constexpr size_t gqa32_merge_bytes(int width) { return (size_t)kWavesPerBlock * 16 * (width + 4) * sizeof(float); }

template <int W, int SC, bool CODES>
__global__ __launch_bounds__(kWavesPerBlock *kWave, kGqa32BlocksPerCu) void attn_partial_gqa32(AttnParams p, int gb) {
    constexpr int TILE = gqa32_tile(W), SUBS = TILE / 16, KS = W / 16, SETS = W / 16;
    constexpr int VW = SETS < 4 ? SETS : 4, VL = SETS / VW;   // floats of a V load, loads per row
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid >> 6;
    const int c = lane & 15;
    const int r = lane >> 4;

    int split, j, hg, group_head;
    int bid = group_block(p, &split);
    bid = fast_divide(p.by_k, bid, &j);
    const int b = fast_divide(p.by_groups, bid, &hg);
    const int h0 = hg * gb;
    const int hk = fast_divide(p.by_G, h0, &group_head);

    // Query operand: q[head c][16 s + 4 r + i]; heads past the group repeat the last one, nothing reads
    // what they lead to.
    const float *q = static_cast<const float *>(p.q) + ((int64_t)b * p.Hq + h0 + min(c, gb - 1)) * p.D;
    const bool q_aligned = (reinterpret_cast<uintptr_t>(p.q) & 15) == 0;
    auto query = [&](int d) {
        if (q_aligned) return *reinterpret_cast<const f32x4_t *>(q + d);
        return f32x4_t{q[d], q[d + 1], q[d + 2], q[d + 3]};
    };
    constexpr int US = CODES ? 2 : 1;        // a wave's 16-value pieces of the head dimension (D <= 128)
    f32x4_t qop[KS], q_raw[US], u_raw[US][KS];
    if constexpr (CODES) {                   // what the projection reads is requested ahead of everything
        const float *U = static_cast<const float *>(p.U_K) + ((int64_t)hk * W + c) * p.D;
#pragma unroll
        for (int n = 0; n < US; ++n) {
            const int d = min(16 * (wave + kWavesPerBlock * n), p.D - 16) + 4 * r;
            q_raw[n] = query(d);
#pragma unroll
            for (int s = 0; s < KS; ++s) u_raw[n][s] = __builtin_bit_cast(f32x4_t, load16(U + (int64_t)16 * s * p.D + d));
        }
    } else {
#pragma unroll
        for (int s = 0; s < KS; ++s) qop[s] = query(16 * s + 4 * r);
    }
    const ShardRef sh = resolve_shard(p, b, b, j, lane);
    int r0, r1;
    split_rows<TILE>(p, sh.n, split, &r0, &r1);

    __shared__ float sm_m[kWavesPerBlock][16];
    __shared__ float sm_l[kWavesPerBlock][16];
    // the waves' parts of the projected query; the raw scores of the block's rows, [head][chunk]; the waves'
    // outputs (gqa32_merge_bytes)
    extern __shared__ __attribute__((aligned(16))) float gqa32_lds[];

    const int64_t part_base = (((int64_t)b * p.Hq + h0) * p.k + j) * p.nsplit + split;
    const int64_t part_head_stride = (int64_t)p.k * p.nsplit;
    if (r0 >= r1) {
        for (int idx = tid; idx < gb * (W / 4); idx += blockDim.x) {
            const int g = idx / (W / 4), d = (idx - g * (W / 4)) * 4;
            const int64_t at = part_base + g * part_head_stride;
            *reinterpret_cast<float4 *>(p.part_acc + at * W + d) = make_float4(0.f, 0.f, 0.f, 0.f);
            if (d == 0) *reinterpret_cast<float2 *>(p.part_ml + at * 2) = make_float2(-INFINITY, 0.f);
        }
        return;
    }

    // Requests as in attn_partial_gqa: 32-bit byte offsets from the kv head's base, rows past the end
    // clamped onto the last one by a minimum, sums that saturate, each tile's offset hidden from the optimiser.
    const char *Kb = sh.K + (int64_t)hk * p.stride_h * 4;
    const char *Vb = sh.V + (int64_t)hk * p.stride_h * 4;
    const uint32_t rb = (uint32_t)(p.stride_s * 4);
    const uint32_t last = (uint32_t)(r1 - 1) * rb;
    auto opaque = [](uint32_t v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    const int row_most = p.S - 1;
    auto rows_bytes = [&](int rows) { return (uint32_t)min(rows, row_most) * rb; };
    auto sum = [](uint32_t a, uint32_t b) { return __builtin_elementwise_add_sat(a, b); };
    f32x4_t kr[SUBS][KS];
    uint32_t vr[SUBS][4][VL][VW];
    auto load_k = [&](int t0) {
        const uint32_t at = opaque(sum(rows_bytes(t0), rows_bytes(c)));
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub) {
            const char *row = Kb + (size_t)(min(sum(at, rows_bytes(16 * sub)), last) + 16 * r);
#pragma unroll
            for (int s = 0; s < KS; ++s) kr[sub][s] = __builtin_bit_cast(f32x4_t, load16_stream(row + 64 * s));
        }
    };
    auto load_v = [&](int t0) {
        const uint32_t at = opaque(sum(rows_bytes(t0), rows_bytes(4 * r)));
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const char *row = Vb + (size_t)(min(sum(at, rows_bytes(16 * sub + i)), last) + 4 * VW * c);
#pragma unroll
                for (int l = 0; l < VL; ++l) load_words_stream<VW>(vr[sub][i][l], row + 64 * VW * l);
            }
    };
    auto mfma = [](float a, float b, f32x4_t acc) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0); };
    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
    int t0 = r0 + __builtin_amdgcn_readfirstlane(wave) * TILE;
    load_k(t0);                              // (a wave without rows loads the last one)
    load_v(t0);

    constexpr int AP = W + 4;                // floats of a head's row in LDS (banks)
    if constexpr (CODES) {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            f32x4_t proj[4] = {zero, zero, zero, zero};
#pragma unroll
            for (int n = 0; n < US; ++n)
                if (16 * (wave + kWavesPerBlock * n) < p.D)
#pragma unroll
                    for (int i = 0; i < 4; ++i) proj[i] = mfma(u_raw[n][s][i], q_raw[n][i], proj[i]);
            *reinterpret_cast<f32x4_t *>(gqa32_lds + (wave * 16 + c) * AP + 16 * s + 4 * r) =
                (proj[0] + proj[1]) + (proj[2] + proj[3]);
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            f32x4_t of[kWavesPerBlock];
#pragma unroll
            for (int w = 0; w < kWavesPerBlock; ++w)
                of[w] = *reinterpret_cast<const f32x4_t *>(gqa32_lds + (w * 16 + c) * AP + 16 * s + 4 * r);
            qop[s] = (of[0] + of[1]) + (of[2] + of[3]);
        }
        if (SC == kScoresStaged) __syncthreads();            // the area becomes the score stage
    }
    // complete before the loop: a wait for it in there would be a wait for the tiles' loads
#pragma unroll
    for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(qop[s]));

    float m = -INFINITY, lsum = 0.0f;
    f32x4_t oacc[SETS];                      // oacc[4 l + i][x] = O[head c][16 VW l + VW (4 r + x) + i]
#pragma unroll
    for (int i = 0; i < SETS; ++i) oacc[i] = zero;

    if (t0 < r1) do {
        const int tnext = t0 + kWavesPerBlock * TILE;
        float sv[4 * SUBS];                  // sv[4 sub + x]: entry t0 + 16 sub + 4 r + x
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub) {
            f32x4_t of[4];                   // of[l]: sums of 2^l steps that wait for their partner
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                f32x4_t part[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) part[i] = mfma(kr[sub][s][i], qop[s][i], zero);
                f32x4_t t = (part[0] + part[1]) + (part[2] + part[3]);
#pragma unroll
                for (int l = 0; l < 3; ++l) {                // pairwise, like the carry of a counter
                    if (((s + 1) & ((2 << l) - 1)) == 0) t = of[l] + t;
                    else if (((s + 1) & ((1 << l) - 1)) == 0) of[l] = t;
                }
                of[3] = t;
                if (W == 128 && (s & 1)) __builtin_amdgcn_sched_barrier(0);      // (registers)
            }
#pragma unroll
            for (int x = 0; x < 4; ++x) sv[4 * sub + x] = t0 + 16 * sub + 4 * r + x < r1 ? of[3][x] * p.scale : -INFINITY;
        }
        load_k(tnext);

        if (SC == kScoresStaged && c < gb) {
            float *dst = gqa32_lds + c * p.chunk + (t0 - r0) + 4 * r;
#pragma unroll
            for (int sub = 0; sub < SUBS; ++sub)
                *reinterpret_cast<float4 *>(dst + 16 * sub) = make_float4(sv[4 * sub], sv[4 * sub + 1], sv[4 * sub + 2], sv[4 * sub + 3]);
        } else if (SC == kScoresDirect && c < gb) {
            float *dst = p.scores + (((int64_t)b * p.Hq + h0 + c) * p.k + j) * p.S;
#pragma unroll
            for (int sub = 0; sub < SUBS; ++sub) {
                const int row = t0 + 16 * sub + 4 * r;
                if (row + 4 <= r1 && (p.S & 3) == 0 && (reinterpret_cast<uintptr_t>(p.scores) & 15) == 0) {
                    *reinterpret_cast<float4 *>(dst + row) = make_float4(sv[4 * sub], sv[4 * sub + 1], sv[4 * sub + 2], sv[4 * sub + 3]);
                } else {
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        if (row + x < r1) dst[row + x] = sv[4 * sub + x];
                }
            }
        }

        // online softmax for head c (its entries are spread over the 4 lane groups)
        float tm = sv[0];
#pragma unroll
        for (int x = 1; x < 4 * SUBS; ++x) tm = fmaxf(tm, sv[x]);
        const float mn = fmaxf(m, group_max(tm));
        const float base = mn == -INFINITY ? 0.0f : mn;      // (nothing but -Inf so far: weights of zero, not NaN)
        if (__any(mn > m)) {                 // else the factor is 1 in every lane
            const float corr = __expf(m - base);
            m = mn;
            lsum *= corr;
#pragma unroll
            for (int i = 0; i < SETS; ++i) oacc[i] = oacc[i] * corr;
        }
#pragma unroll
        for (int x = 0; x < 4 * SUBS; ++x) {
            sv[x] = __expf(sv[x] - base);
            lsum += sv[x];
        }
        if (t0 + TILE > r1) {                // rows past the end repeat the last one: a weight of zero times Inf is NaN
#pragma unroll
            for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
                for (int x = 0; x < 4; ++x)
#pragma unroll
                    for (int l = 0; l < VL; ++l)
#pragma unroll
                        for (int i = 0; i < VW; ++i) vr[sub][x][l][i] = t0 + 16 * sub + 4 * r + x < r1 ? vr[sub][x][l][i] : 0u;
        }
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
            for (int l = 0; l < VL; ++l)
#pragma unroll
                for (int i = 0; i < VW; ++i) {
                    f32x4_t part[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) part[x] = mfma(__uint_as_float(vr[sub][x][l][i]), sv[4 * sub + x], zero);
                    oacc[VW * l + i] = oacc[VW * l + i] + ((part[0] + part[1]) + (part[2] + part[3]));
                }
        load_v(tnext);
        t0 = tnext;
    } while (t0 < r1);

    __syncthreads();
    if (SC == kScoresStaged) {               // the block's scores: one burst per head, a head per wave
        const int rows = r1 - r0, rows4 = rows & ~3;
        for (int g = wave; g < gb; g += kWavesPerBlock) {
            float *dst = p.scores + (((int64_t)b * p.Hq + h0 + g) * p.k + j) * p.S + r0;
            const float *src = gqa32_lds + g * p.chunk;
            if ((p.S & 3) == 0 && (reinterpret_cast<uintptr_t>(p.scores) & 15) == 0) {
                for (int i = lane * 4; i < rows4; i += kWave * 4)
                    *reinterpret_cast<float4 *>(dst + i) = *reinterpret_cast<const float4 *>(src + i);
                if (lane < rows - rows4) dst[rows4 + lane] = src[rows4 + lane];
            } else {
                for (int i = lane; i < rows; i += kWave) dst[i] = src[i];
            }
        }
        __syncthreads();                     // the stage becomes the merge area
    }

    // the waves' results -> LDS, then merge the waves and write the block's partial
    lsum += __shfl_xor(lsum, 16, kWave);
    lsum += __shfl_xor(lsum, 32, kWave);
    if (c < gb) {
        float *wacc = gqa32_lds + (wave * 16 + c) * AP;
#pragma unroll
        for (int l = 0; l < VL; ++l)
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int i = 0; i < VW; ++i) wacc[16 * VW * l + VW * (4 * r + x) + i] = oacc[VW * l + i][x];
    }
    if (r == 0) {
        sm_m[wave][c] = m;
        sm_l[wave][c] = lsum;
    }
    __syncthreads();
    // (four values per thread, like the bf16 groups: 8 heads x 128 values, 64 MiB, 22.8 -> 22.0 us, 16 heads x 64 17.4 -> 17.0)
    for (int idx = tid; idx < gb * (W / 4); idx += blockDim.x) {
        const int g = idx / (W / 4), d = (idx - g * (W / 4)) * 4;
        float M = sm_m[0][g];
#pragma unroll
        for (int w2 = 1; w2 < kWavesPerBlock; ++w2) M = fmaxf(M, sm_m[w2][g]);
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
        float L = 0.0f;
#pragma unroll
        for (int w2 = 0; w2 < kWavesPerBlock; ++w2) {
            const float f = sm_m[w2][g] == -INFINITY ? 0.0f : __expf(sm_m[w2][g] - M);
            const float4 o = *reinterpret_cast<const float4 *>(gqa32_lds + (w2 * 16 + g) * AP + d);
            a = make_float4(fmaf(o.x, f, a.x), fmaf(o.y, f, a.y), fmaf(o.z, f, a.z), fmaf(o.w, f, a.w));
            L = fmaf(sm_l[w2][g], f, L);
        }
        const int64_t at = part_base + g * part_head_stride;
        *reinterpret_cast<float4 *>(p.part_acc + at * W + d) = a;
        if (d == 0) *reinterpret_cast<float2 *>(p.part_ml + at * 2) = make_float2(M, L);
    }
}

template <typename T, int THREADS>
__global__ __launch_bounds__(THREADS) void attn_combine(CombineParams p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // combine_smem_bytes()
    combine_head<T, THREADS>(p, blockIdx.x, smem);
}

// The smallest calls of one head per block in one launch: where the plan gives every split one tile and a head has at most
// kSmallWaves of them, a block takes a whole head, a wave a split.  The partials stay in LDS and the same block merges
// them - same rows per split, same sums in the same order, same bits as attn_partial and attn_combine, whose blocks here
// hold one busy wave of four.  What bounds such a call are launches and trips to memory: the merge's launch and its
// trip go.  (Pass and merge in a graph: 4 heads x 2 shards of 256 fp32 rows of 64 values 7.9 -> 7.25 us, of 128 x 2 sequences 8.0 ->
// 6.2, 4 heads x 2 of 128 bf16 rows of 128 8.5 -> 6.7, 63 heads x 3 of 128 rows of 16 values 8.45 -> 6.05; a launch less of host
// time.)  More tiles than a block has waves would be a second trip: those calls stay with the two kernels.
constexpr int kSmallWaves = 16;
inline size_t small_lds_bytes(int W, int np) { return (size_t)np * (W + 2) * sizeof(float) + 16 + combine_smem_bytes(256, np, 0); }
template <typename T, int W>
__global__ __launch_bounds__(kSmallWaves *kWave) void attn_small(AttnParams p, CombineParams c) {
    constexpr int EPL = Pack16<T>::N;        // as in attn_partial
    constexpr int LPR = W / EPL;
    constexpr int RPL = kWave / LPR;
    constexpr int NL = plain_loads_per_tile(W * (int)sizeof(T), 1);
    constexpr int CB = ilog2(LPR);
    extern __shared__ __attribute__((aligned(16))) float small_lds[];       // np x W accumulators, np pairs, the merge's
    const int np = p.k * p.nsplit;
    float *parts = small_lds, *pairs = parts + np * W;
    unsigned char *merge = reinterpret_cast<unsigned char *>(pairs + (np * 2 + 3) / 4 * 4);

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & (LPR - 1), r = lane >> CB;
    int h, group_head, split;
    const int b = fast_divide(p.by_groups, blockIdx.x, &h);
    const int hk = fast_divide(p.by_G, h, &group_head);
    const float gate = combine_gate(c, blockIdx.x);      // ahead of the rows: the merge has no trip of its own
    if (wave < np) {
        const int j = fast_divide(p.by_nsplit, wave, &split);
        const T *qp = static_cast<const T *>(p.q) + ((int64_t)b * p.Hq + h) * W + col * EPL;
        float qf[EPL];
#pragma unroll
        for (int i = 0; i < EPL; ++i) qf[i] = load_scalar<T>(qp, i);
        const ShardRef sh = resolve_shard(p, b, b * p.rr + (p.rr == 1 ? 0 : h), j, lane);
        const int r0 = split * p.chunk, r1 = min(min(sh.n, p.S), r0 + p.chunk);
        float m = -INFINITY, l = 0.0f, acc[EPL];
#pragma unroll
        for (int i = 0; i < EPL; ++i) acc[i] = 0.0f;
        if (r0 < r1) {
            const T *Kb = reinterpret_cast<const T *>(sh.K) + (int64_t)hk * p.stride_h + col * EPL;
            const T *Vb = reinterpret_cast<const T *>(sh.V) + (int64_t)hk * p.stride_h + col * EPL;
            uint4 kr[NL], vr[NL];
#pragma unroll
            for (int t = 0; t < NL; ++t) kr[t] = load16_stream(Kb + (int64_t)min(r0 + t * RPL + r, r1 - 1) * p.stride_s);
#pragma unroll
            for (int t = 0; t < NL; ++t) vr[t] = load16_stream(Vb + (int64_t)min(r0 + t * RPL + r, r1 - 1) * p.stride_s);
#pragma unroll
            for (int i = 0; i < EPL; ++i) qf[i] = p.scale * qf[i];
            float s[NL];
#pragma unroll
            for (int t = 0; t < NL; ++t) {
                float kf[EPL];
                Pack16<T>::widen(kr[t], kf);
                float d = 0.0f;
#pragma unroll
                for (int i = 0; i < EPL; ++i) d = fmaf(qf[i], kf[i], d);
                d = bits_sum<0, CB>(d);
                s[t] = r0 + t * RPL + r < r1 ? d : -INFINITY;
            }
            if (p.scores != nullptr) {
                float *dst = p.scores + (((int64_t)b * p.Hq + h) * p.k + j) * p.S;
#pragma unroll
                for (int u = 0; u < NL; u += LPR) {
                    float v = s[u];
#pragma unroll
                    for (int t = 1; t < LPR && u + t < NL; ++t) v = (col == t) ? s[u + t] : v;
                    const int row = r0 + (u + col) * RPL + r;
                    if (u + col < NL && row < r1) dst[row] = v;
                }
            }
            float tm = s[0];
#pragma unroll
            for (int t = 1; t < NL; ++t) tm = fmaxf(tm, s[t]);
            tm = bits_max<CB, 6>(tm);
            const float mn = fmaxf(m, tm);
            const float corr = __expf(m - mn);
            m = mn;
            l *= corr;
#pragma unroll
            for (int i = 0; i < EPL; ++i) acc[i] *= corr;
#pragma unroll
            for (int t = 0; t < NL; ++t) {
                const float pt = __expf(s[t] - mn);
                s[t] = pt;
                l += pt;
            }
#pragma unroll
            for (int t = 0; t < NL; ++t) {
                float vf[EPL];
                Pack16<T>::widen(vr[t], vf);
#pragma unroll
                for (int i = 0; i < EPL; ++i) acc[i] = fmaf(s[t], vf[i], acc[i]);
            }
#pragma unroll
            for (int off = LPR; off < kWave; off <<= 1) {
                l += __shfl_xor(l, off, kWave);
#pragma unroll
                for (int i = 0; i < EPL; ++i) acc[i] += __shfl_xor(acc[i], off, kWave);
            }
            // as attn_partial joins this wave with three that have no rows
            const float M = fmaxf(m, -INFINITY), f = m == -INFINITY ? 0.0f : __expf(m - M);
            m = M;
            l = fmaf(l, f, 0.0f);
#pragma unroll
            for (int i = 0; i < EPL; ++i) acc[i] = fmaf(acc[i], f, 0.0f);
        }
        if (r == 0) {
#pragma unroll
            for (int i = 0; i < EPL; i += 4)
                *reinterpret_cast<float4 *>(parts + wave * W + col * EPL + i) = make_float4(acc[i], acc[i + 1], acc[i + 2], acc[i + 3]);
        }
        if (lane == 0) *reinterpret_cast<float2 *>(pairs + 2 * wave) = make_float2(m, l);
    }
    __syncthreads();
    if (wave >= 4) return;                   // (a barrier waits for the waves that are left)
    combine_head<T, 256>(c, blockIdx.x, merge, parts, pairs, [&] { return gate; });
}

template <typename T>
int launch_small(const AttnParams &p, const CombineParams &c, int heads, hipStream_t st) {
    const int np = p.k * p.nsplit;
    const dim3 grid(heads), block((np < 4 ? 4 : np) * kWave);
    const size_t lds = small_lds_bytes(c.W, np);
    switch (c.W) {
        case 16: hipLaunchKernelGGL((attn_small<T, 16>), grid, block, lds, st, p, c); break;
        case 32: hipLaunchKernelGGL((attn_small<T, 32>), grid, block, lds, st, p, c); break;
        case 64: hipLaunchKernelGGL((attn_small<T, 64>), grid, block, lds, st, p, c); break;
        case 128: hipLaunchKernelGGL((attn_small<T, 128>), grid, block, lds, st, p, c); break;
        default: return PIKV_ERR_UNSUPPORTED;
    }
    return launch_status();
}

template <typename T, int W>
int launch_partial_w(int gb, const AttnParams &p, int blocks, hipStream_t st) {
    const dim3 grid(blocks), block(kWavesPerBlock * kWave);
    const size_t lds = p.stage_scores ? (size_t)gb * p.chunk * sizeof(float) : 0;
    switch (gb) {
        case 1: hipLaunchKernelGGL((attn_partial<T, W, 1>), grid, block, lds, st, p); break;
        case 2: hipLaunchKernelGGL((attn_partial<T, W, 2>), grid, block, lds, st, p); break;
        case 4: hipLaunchKernelGGL((attn_partial<T, W, 4>), grid, block, lds, st, p); break;
        case 8: hipLaunchKernelGGL((attn_partial<T, W, 8>), grid, block, lds, st, p); break;
        default: return PIKV_ERR_UNSUPPORTED;
    }
    return launch_status();
}

template <int W, bool CODES>
void launch_gqa(int row_tiles, bool long_blocks, const AttnParams &p, int64_t blocks, size_t lds, hipStream_t st) {
    const dim3 grid((unsigned)blocks), block(kWavesPerBlock * kWave);
    auto launch = [&](auto rt, auto longs) {
        constexpr int RT = decltype(rt)::value;
        constexpr bool LONG = decltype(longs)::value;
        constexpr int kStaged = LONG ? kScoresDirect : kScoresStaged;      // (no long block of 128-value rows stages its scores)
        if (p.scores == nullptr)
            hipLaunchKernelGGL((attn_partial_gqa<W, RT, kScoresNone, CODES, LONG>), grid, block, lds, st, p);
        else if (p.stage_scores)
            hipLaunchKernelGGL((attn_partial_gqa<W, RT, kStaged, CODES, LONG>), grid, block, lds, st, p);
        else
            hipLaunchKernelGGL((attn_partial_gqa<W, RT, kScoresDirect, CODES, LONG>), grid, block, lds, st, p);
    };
    if (row_tiles == 2) launch(std::integral_constant<int, 2>{}, std::false_type{});
    else if (row_tiles == 4) launch(std::integral_constant<int, 4>{}, std::false_type{});
    else if (long_blocks) launch(std::integral_constant<int, 1>{}, std::bool_constant<W == 128>{});
    else launch(std::integral_constant<int, 1>{}, std::false_type{});
}

template <int W, bool CODES>
void launch_gqa32(int gb, const AttnParams &p, int64_t blocks, hipStream_t st) {
    const dim3 grid((unsigned)blocks), block(kWavesPerBlock * kWave);
    const size_t stage = p.stage_scores ? (size_t)gb * p.chunk * sizeof(float) : 0, merge = gqa32_merge_bytes(W);
    const size_t lds = stage > merge ? stage : merge;
    if (p.scores == nullptr)
        hipLaunchKernelGGL((attn_partial_gqa32<W, kScoresNone, CODES>), grid, block, lds, st, p, gb);
    else if (p.stage_scores)
        hipLaunchKernelGGL((attn_partial_gqa32<W, kScoresStaged, CODES>), grid, block, lds, st, p, gb);
    else
        hipLaunchKernelGGL((attn_partial_gqa32<W, kScoresDirect, CODES>), grid, block, lds, st, p, gb);
}

template <typename T>
int launch_partial(int width, int gb, const AttnParams &p, int blocks, hipStream_t st) {
    switch (width) {
        case 16: return launch_partial_w<T, 16>(gb, p, blocks, st);
        case 32: return launch_partial_w<T, 32>(gb, p, blocks, st);
        case 64: return launch_partial_w<T, 64>(gb, p, blocks, st);
        case 128: return launch_partial_w<T, 128>(gb, p, blocks, st);
        default: return PIKV_ERR_UNSUPPORTED;
    }
}

}  // namespace

static int g_split_override = 0;   // tuning hook, see pikv_set_attn_split
static hipEvent_t g_prof_start = nullptr, g_prof_stop = nullptr;   // see pikv_set_profile_events
void g_split_override_set(int v) { g_split_override = v > 0 ? v : 0; }

// Groups of narrow rows: does the plain kernel do better?  Measured on both sides over 2300 drawn calls
// (pass and merge; 16 - 64 values or codes, 2 - 64 heads, up to 1 GiB).
//   - 2 heads over 16 values: 14 of a tile's 16 rows are padding, and from 28 MB of K/V on that bounds the pass
//     (63 MB 22.8 against 25.6 us; below, the matrix cores are 5 - 15 % ahead).
//   - Groups of 2, 4 and 8 heads otherwise: never (4 heads 0.77, 8 heads 0.53 of the plain kernel's time).
//   - Other groups, which the plain kernel takes one head per block, re-reading K/V from the caches for each:
//     as long as whole groups make few blocks, which then are long (64 heads over 576 rows of rank 16 11
//     against 30 us), and the heads re-read little.  The lines: 96 blocks of rows of 16 values, 64 of 32, 48 of 64
//     (64 of one row tile); 64 MiB of re-reading at one row tile, 192 and 512 MiB at two and four, whose
//     blocks are longer (16 heads, 1664 rows of 64 values, 218 MB re-read 27.5 against 14.6 us).
// What counts is the capacity: the entry counts are on the device.
static bool plain_pays(const pikv_desc *d, int k, int row_tiles) {
    const int W = desc_width(d), G = d->Hq / d->Hkv;
    const int64_t units = (int64_t)d->B * d->Hkv * k, bytes = units * d->S * W * 4;
    if (G == 2 && W == 16) return bytes >= 28000000;
    if (W == 128 || G == 2 || G == 4 || G == 8 || units == 0) return false;
    int64_t splits = 256 * gqa_blocks_per_cu(W, row_tiles, d->rank > 0) / units;
    const int64_t most = d->S / (2 * kWavesPerBlock * gqa_tile(W, row_tiles));
    if (splits > most) splits = most;
    if (splits < 1) splits = 1;
    const int64_t few = W == 16 ? 96 : W == 32 || row_tiles == 1 ? 64 : 48;
    const int64_t mib = row_tiles == 1 ? 64 : row_tiles == 2 ? 192 : 512;
    if (W == 64 && d->rank > 0 && d->S <= 128 && units * G <= 768) return true;   // forming the query costs more than the rows
    return units * splits <= few && bytes * G <= mib << 20;
}

// The least heads per block for the fp32 matrix-core kernel: with two, 14 of a product's 16 rows are padding, and the plain
// kernel is ahead by 1 - 4 % (256 MiB 48.5 against 50.6 us, rank-32 codes 52.9 against 59).  Groups of four, which
// share one stream there too, are as fast or faster there, most of all in shards of uneven fill, its blocks being shorter
// (fused step, 16 x 8 kv heads x 2 shards of 2048 slots of 64 values: full 59.3 against 61.5 us, 10 - 100 % full 47.6
// against 51.8; 8 x 8 x 2 of 4096 rank-32 codes 43.2 against 45.3 and 36.9 against 40.6).
constexpr int kGqa32Heads = 3;

int make_attn_plan(const pikv_desc *d, int k, AttnPlan *plan, size_t scratch_limit) {
    const int rc = check_desc(d);
    if (rc != PIKV_OK) return rc;
    if (k < 1 || k > d->E) return PIKV_ERR_INVALID;
    const int W = desc_width(d);
    const int G = d->Hq / d->Hkv;
    int gb = 1;
    if (d->route_rows_per_seq == 1 && (G == 2 || G == 4 || G == 8)) gb = G;
    // The matrix-core kernel takes every group of bf16 rows that shares one routing decision and
    // addresses a kv head's rows in 32 bits - but for narrow ones where the plain kernel does better.
    const int group_tiles = G <= 16 ? 1 : (G <= 32 ? 2 : 4);
    const bool gqa_mfma = d->route_rows_per_seq == 1 && d->dtype == PIKV_BF16 && G >= 2 && G <= 64 &&
                          (int64_t)d->S * d->stride_s * 2 < ((int64_t)1 << 32) &&
                          !plain_pays(d, k, group_tiles);
    if (gqa_mfma) gb = G;
    // fp32 groups: as many heads per block as divide the group, up to the 16 of a product
    int gb32 = G < 16 ? G : 16;
    while (G % gb32 != 0) --gb32;
    const bool gqa_f32 = d->route_rows_per_seq == 1 && d->dtype == PIKV_F32 && gb32 >= kGqa32Heads &&
                         G != 4 && (int64_t)d->S * d->stride_s * 4 < ((int64_t)1 << 32);
    if (gqa_f32) gb = gb32;
    const int tq = d->tq > 1 ? d->tq : 1;
    // draft queries are folded into the query group of the matrix-core kernel's 128-value rows only
    if (tq > 1 && (!gqa_mfma || W != 128 || d->Hq % tq != 0 || G % tq != 0)) return PIKV_ERR_UNSUPPORTED;
    const int row_tiles = gqa_mfma ? group_tiles : 0;
    const int epl = 16 / elem_bytes(d->dtype);
    const int lpr = W / epl;
    if (lpr < 1 || lpr > 32) return PIKV_ERR_UNSUPPORTED;
    const int row_bytes = W * elem_bytes(d->dtype);
    const int tile = gqa_mfma ? gqa_tile(W, row_tiles) : gqa_f32 ? gqa32_tile(W) : (kWave / lpr) * plain_loads_per_tile(row_bytes, gb);
    const int64_t units = (int64_t)d->B * (d->Hq / gb) * k;
    // One round of resident blocks: 256 CUs times the 4-wave blocks a CU holds at this
    // kernel's register footprint.  Fewer, longer blocks keep the per-wave prefetch chain
    // busy and shrink the partials that the combine pass has to merge.
    int resident = gqa_mfma ? gqa_blocks_per_cu(W, row_tiles, d->rank > 0) : gqa_f32 ? kGqa32BlocksPerCu : plain_blocks_per_cu(row_bytes, gb);
    // More than 8 rows per kv head: every split writes and re-reads rows * 128 accumulators, and
    // two rounds' worth of longer blocks beat three (16 rows, 128 MiB: 36.0 against 40.0 us).
    if (gqa_mfma && W == 128 && gb > 8 && resident > 2) resident = 2;
    // Rank-64 codes: forming the query costs a block about as much as a tile (2 sequences x 8 kv heads
    // x 2 of 10112 rows 30.8 -> 27.5 us, 256 MiB over 256 units even).
    if (gqa_mfma && W == 64 && d->rank > 0 && resident > 2) resident = 2;
    int64_t nsplit = 1;
    int chunk = 0;
    // A block per CU, or nearly, for bf16 groups of one row tile: `least` splits of every unit (sequence, head group, shard),
    // instead of three or four blocks per CU.  Blocks beyond one per CU cost more - their
    // start, their merge, the partials that the merge reads - than they hide, and a shard that is not full still
    // makes whole, even blocks.  Where the line lies, from fused steps of 16 - 512 units x 1024 - 8192 slots, full / 55 % /
    // 10 - 100 % full, time against the other plan's:
    //   - at most 512 KiB of K and V (128 units x 64 values, 4096 slots 0.94 / 0.89 / 0.89, 8192 0.95 / 1.05 / 1.03; 80 units
    //     0.95 / 0.86 / 0.93 and 1.10 / 0.98 / 1.13), rows of 16 values 128 KiB (64 units, 6000 slots 0.88 / 0.89 / 0.89; 224
    //     units, 6000 slots 1.12 / 1.01 / 1.13): beyond, shards of uneven fill leave CUs waiting for the longest block;
    //   - at least 200 blocks (68 units x 3 0.90 / 0.89 / 0.96, 192 x 1 0.97 / 0.93 / 1.02, 96 x 2 of rank-32 codes 1.02 / 0.93 / 1.05),
    //     or 192 of at most 256 KiB (0.96 / 0.94 / 0.99 and 0.97 / 0.94 / 0.98);
    //   - at most 24 partials of a head (7 x 2 x 3 units, 18 partials 0.93 / 0.90 / 0.96, 10 x 5, 25 partials 1.07 / 1.02 / 1.09, 8 x 8,
    //     32 partials 1.09 / 1.04 / 1.10): the merge of up to 32 takes narrow blocks, where the other plan's many more
    //     take wide ones.  Narrow rows in blocks of up to two rounds of tiles have no more splits by the other plan:
    //     up to 32 (8 x 8 units of 1024 slots 0.98 / 0.95 / 0.96; 5 x 4, 48 partials, a tenth full 1.06);
    //   - rows of 128 values only beyond two rounds, where the other plan cuts alike (64 units of 1024 slots 1.02).
    // Fewer than 16 units are left to that plan, unmeasured.
    const int round = kWavesPerBlock * tile;
    const int64_t least = units > 0 ? 256 / units : 1;
    const int64_t block_rows = least > 0 ? (d->S + least - 1) / least : d->S;
    const bool two_rounds = block_rows <= 2 * round;
    const int64_t long_block = least * units >= 200 ? 128 * 1024 : least * units >= 192 ? 64 * 1024 : 0;     // values of K
    const bool by_unit = gqa_mfma && row_tiles == 1 && (W < 128 || (gb <= 8 && !two_rounds)) && units >= 16 &&
                         block_rows * W <= (W == 16 ? long_block / 4 : long_block) && k * least <= (W < 128 && two_rounds ? 32 : 24) &&
                         g_split_override == 0;
    // With few units a block takes fewer than two tiles per wave, down to one, and below 64 blocks to one in all (fp32
    // groups on the matrix cores take whole rounds): every kernel's chain of trips to memory is shorter then.  (7 units of 938 rows of 64 values x 8 heads, pass and
    // merge 15.1 -> 9.7 us, 6 of 256 rows of 128 9.7 -> 8.5, 16 of 768 rank-32 codes of one head 12.0 -> 9.9, 8 of 256
    // fp32 rows 9.9 -> 7.9, 4 of 1192 11.5 -> 9.5.)  Not past 128 partials of a head: 256 blocks of one unit 21.8 -> 24.8.  Groups
    // of narrow bf16 rows, whose tiles are long, only in shards below four rounds.
    const int64_t rounds = (d->S + round - 1) / round;
    const bool few = units > 0 && g_split_override == 0 && units * rounds <= 256 && k * rounds <= 128 &&
                     !(gqa_mfma && W < 128 && d->S >= 4 * round);
    int64_t finest = rounds;
    for (int part = round; few && !gqa_f32 && part > tile && units * finest * 2 <= 64; part /= 2)
        finest = (d->S + part / 2 - 1) / (part / 2);
    // Splits whose partials fit the fixed array of the call without a workspace: where a plan wants more of them than
    // the one that took these calls before, the call takes fewer and is not refused for it.
    const size_t split_bytes = (size_t)(d->B > 0 ? d->B : 1) * d->Hq * k * (W + 2) * sizeof(float);
    const bool capped = scratch_limit != SIZE_MAX &&
                        (few || gqa_f32 || (gqa_mfma && (W != 128 || (row_tiles == 1 && gb <= 8 && units <= 64))));
    const int64_t scratch_splits = capped ? (int64_t)((scratch_limit - 1024) / split_bytes) : INT32_MAX;
    auto split_for = [&](int res) {
        nsplit = units > 0 ? (int64_t)256 * res / units : 1;
        if (by_unit) nsplit = least;
        // No finer than two tiles per wave: with one, nothing is in flight while a wave computes,
        // and a block of uneven waves (2, 2, 1, 1 tiles) runs as long as one of twice the rows.
        // (Few units, short passes: 64 MiB over 16 units 14.0 -> 12.8 us, 32 MiB over 8 units
        // 8.6 -> 7.9 us, and fewer partials for the merge.)  A forced count is only held to one tile.
        int64_t max_split = d->S / (2 * kWavesPerBlock * tile);
        if (few) nsplit = max_split = finest;
        else if (by_unit) max_split = finest;
        if (g_split_override > 0) {
            nsplit = g_split_override;
            max_split = (d->S + tile - 1) / tile;
        }
        if (max_split < 1) max_split = 1;
        if (nsplit > max_split) nsplit = max_split;
        if (nsplit > kMaxPartialsPerHead / k) nsplit = kMaxPartialsPerHead / k;
        if (nsplit > scratch_splits) nsplit = scratch_splits;
        if (nsplit < 1) nsplit = 1;
        chunk = (int)((d->S + nsplit - 1) / nsplit);
        const int unit = gqa_f32 ? kWavesPerBlock * tile : tile;      // (fp32 groups: whole rounds, so that a split's scores start a line)
        chunk = (chunk + unit - 1) / unit * unit;
        nsplit = (d->S + chunk - 1) / chunk;
        // Matrix-core kernel: when that leaves the waves of a block uneven tile counts (c3: 11
        // tiles, 3 + 3 + 3 + 2) and blocks of exactly two tiles per wave are at most a third more
        // blocks, in whole multiples of the 256 CUs, take those.  The extra blocks form a short
        // last round, and a wave whose first tile is served late has one tile left instead of two
        // (c3: 24 -> 32 splits, pass 23.4 -> 23.1 us).  Longer even blocks in a partial round
        // measured slower (k = 16: 8 splits of 8 tiles per wave against 6 splits, +3.7 %).
        const int even = 2 * kWavesPerBlock * tile;
        const int64_t fine = d->S / even;
        if (gqa_mfma && !by_unit && g_split_override == 0 && chunk % (kWavesPerBlock * tile) != 0 &&
            d->S % even == 0 && fine > nsplit && fine * 3 <= nsplit * 4 && fine <= kMaxPartialsPerHead / k && fine <= scratch_splits &&
            (units * fine) % 256 == 0) {
            nsplit = fine;
            chunk = even;
        }
    };
    split_for(resident);
    size_t stage = (size_t)gb * chunk * sizeof(float);      // the block's raw scores, staged in LDS
    size_t stage_most = 64 * 1024 - 256;
    if (by_unit || few) {                                   // as many blocks as there are: a CU has LDS for larger stages
        const int64_t per_cu = (units * nsplit + 255) / 256;
        if (per_cu < resident) resident = per_cu > 0 ? (int)per_cu : 1;
        stage_most = 96 * 1024;
    }
    if (gqa_mfma && W == 128 && gb <= 8) {
        // few rows per kv head of long entries: writing whole lines from the loop measures faster
        // than staging them (8 rows, 128 MiB: 31.8 against 32.8 us with the merge, 4 rows even;
        // 16 rows 37.1 against 36.7, and rank-32 codes at 4 rows 39.5 against 38.0)
        stage = 0;
    } else if (gqa_mfma) {
        // The score stage must fit beside the matrix-core kernel's own LDS as often as a CU holds
        // blocks - three times with one row tile, or twice with longer blocks - or is left out.
        const size_t lds_cu = 160 * 1024;
        const size_t fixed = gqa_static_lds(W, tile, row_tiles);
        if ((size_t)resident * (fixed + stage) > lds_cu || stage > stage_most) {
            bool fits = false;
            if (resident > 2) {
                split_for(2);
                stage = (size_t)gb * chunk * sizeof(float);
                fits = 2 * (fixed + stage) <= lds_cu && stage <= 64 * 1024 - 256;
                if (fits) resident = 2;
            }
            if (!fits) split_for(resident);
            if (!fits && W < 128 && gb <= 4 && g_split_override == 0) {
                // Rounds of blocks over long shards of narrow rows: cut finer until the stage fits twice,
                // as long as a block keeps four rounds of tiles.  Scores written from the loop cost
                // these passes more than the partials of the extra splits (32 sequences x 64 heads over
                // 16 kv heads x 4 shards of 8832 rows of 32 values 545 -> 508 us, 16 x 16 over 8 x 4 of 8192 rank-32
                // codes 126 -> 111; without scores 355 -> 359, 92 -> 93).  Not from 5 rows on, where a store
                // from the loop fills more of its lines (7 rows of 64 values 434 against 441).
                const size_t room = lds_cu / 2 - fixed < 64 * 1024 - 256 ? lds_cu / 2 - fixed : 64 * 1024 - 256;
                const int round = kWavesPerBlock * tile, rows = (int)(room / (gb * sizeof(float)) / round * round);
                const int64_t splits = rows > 0 ? (d->S + rows - 1) / rows : INT32_MAX;
                if (rows >= 4 * round && splits <= kMaxPartialsPerHead / k && splits <= scratch_splits) {
                    chunk = (int)((d->S + splits - 1) / splits + round - 1) / round * round;
                    nsplit = (d->S + chunk - 1) / chunk;
                    stage = (size_t)gb * chunk * sizeof(float);
                    fits = true;
                    resident = 2;
                }
            }
            if (!fits) stage = 0;
        }
    } else if (gqa_f32) {
        // The stage shares its LDS with the merge of the waves; 512 bytes of statistics beside it.
        auto fits = [&](int res) {
            const size_t merge = gqa32_merge_bytes(W), lds = (stage > merge ? stage : merge) + 1024;
            return (size_t)res * lds <= 160 * 1024 && stage <= stage_most;
        };
        if (!fits(resident)) {
            split_for(2);
            stage = (size_t)gb * chunk * sizeof(float);
            bool fit = fits(2);
            if (!fit && g_split_override == 0) {
                // long shards: cut until the scores fit, as long as a block keeps four rounds of tiles (8 heads x
                // 8192 rows of 32 values, 512 MiB: 134.8 -> 126.7 us)
                const int round = kWavesPerBlock * tile, rows = (int)(52 * 1024 / (gb * sizeof(float)) / round * round);
                const int64_t splits = rows > 0 ? (d->S + rows - 1) / rows : INT32_MAX;
                if (rows >= 4 * round && splits <= kMaxPartialsPerHead / k && splits <= scratch_splits) {
                    chunk = (int)((d->S + splits - 1) / splits + round - 1) / round * round;
                    nsplit = (d->S + chunk - 1) / chunk;
                    stage = (size_t)gb * chunk * sizeof(float);
                    fit = fits(resident);
                }
            } else if (fit) {
                resident = 2;
            }
            if (!fit) {
                split_for(resident);
                stage = 0;
            }
        }
    } else if (stage > (size_t)kScoreStageBytes) {
        stage = 0;
    }
    const int64_t target_blocks = 256 * resident;
    plan->gqa_mfma = gqa_mfma;
    plan->gqa_f32 = gqa_f32;
    // one tile per split and a head's splits the waves of one block: attn_small
    plan->small = !gqa_mfma && !gqa_f32 && gb == 1 && d->rank == 0 && chunk == tile && k * nsplit <= kSmallWaves && g_split_override == 0;
    plan->long_blocks = W == 128 && by_unit && !few;
    plan->heads_per_block = gb;
    plan->row_tiles = row_tiles;
    plan->head_blocks = d->Hq / gb;
    plan->tile_rows = tile;
    plan->chunk = chunk;
    plan->nsplit = (int)nsplit;
    plan->resident_blocks = (int)target_blocks;
    plan->score_stage_bytes = stage;
    plan->acc_floats = (size_t)d->B * d->Hq * k * nsplit * W;
    plan->ml_floats = (size_t)d->B * d->Hq * k * nsplit * 2;
    return PIKV_OK;
}

}  // namespace pikv

using namespace pikv;

extern "C" void pikv_set_attn_split(int32_t nsplit) { pikv::g_split_override_set(nsplit); }

namespace pikv {
void g_profile_events_set(void *start, void *stop) {
    g_prof_start = static_cast<hipEvent_t>(start);
    g_prof_stop = static_cast<hipEvent_t>(stop);
}
}  // namespace pikv

extern "C" void pikv_set_profile_events(void *start, void *stop) {
    pikv::g_profile_events_set(start, stop);
}

static size_t workspace_bytes_of(const AttnPlan &plan) {
    const size_t acc = (plan.acc_floats * sizeof(float) + 255) / 256 * 256;
    const size_t ml = (plan.ml_floats * sizeof(float) + 255) / 256 * 256;
    return acc + ml + 256;
}
static size_t workspace_bytes_within(const pikv_desc *desc, int32_t k, size_t scratch_limit) {
    AttnPlan plan;
    return make_attn_plan(desc, k, &plan, scratch_limit) == PIKV_OK ? workspace_bytes_of(plan) : 0;
}

extern "C" size_t pikv_attn_workspace_bytes(const pikv_desc *desc, int32_t k) {
    return workspace_bytes_within(desc, k, SIZE_MAX);
}

namespace pikv {

// Every host-side check of the attention call and its split plan; launches nothing.
int check_attn_args(const pikv_desc *desc, const void *q, const void *const *K_shards,
                    const void *const *V_shards, const void *U_K, const void *U_V,
                    const int32_t *n_valid, const int32_t *topk_idx, int32_t k, int32_t combine,
                    float scale, const float *y, const void *workspace, size_t workspace_bytes,
                    AttnPlan *plan_out, size_t scratch_limit) {
    AttnPlan plan;
    const int rc = make_attn_plan(desc, k, &plan, scratch_limit);
    if (rc != PIKV_OK) return rc;
    if (!q || !K_shards || !V_shards || !n_valid || !topk_idx || !y) return PIKV_ERR_INVALID;
    if (desc->rank > 0 && (!U_K || !U_V)) return PIKV_ERR_INVALID;
    if (combine != PIKV_COMBINE_LSE && combine != PIKV_COMBINE_LOCAL) return PIKV_ERR_INVALID;
    if (!(scale == scale)) return PIKV_ERR_INVALID;
    *plan_out = plan;
    if (desc->B == 0) return PIKV_OK;
    if (!workspace || workspace_bytes < workspace_bytes_of(plan)) return PIKV_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return PIKV_ERR_INVALID;
    if ((int64_t)desc->B * plan.head_blocks * k * plan.nsplit > 0x7fffffff) return PIKV_ERR_UNSUPPORTED;
    return PIKV_OK;
}

bool profile_events_set() { return g_prof_start != nullptr || g_prof_stop != nullptr; }

// Validate and plan (unless the caller has), launch the split pass only and fill the parameters of the merge pass.
int launch_attn_partial(const pikv_desc *desc, const void *q, const void *const *K_shards,
                        const void *const *V_shards, const void *U_K, const void *U_V,
                        const int32_t *n_valid, const int32_t *topk_idx, const float *gates,
                        int32_t k, int32_t combine, float scale, float *y, float *row_max,
                        float *row_norm, float *scores, float *slot_coef, void *workspace,
                        size_t workspace_bytes, void *stream, const AttnPlan *checked, AttnPlan *plan_out,
                        CombineParams *c_out, size_t scratch_limit, bool *merged) {
    AttnPlan plan;
    if (checked != nullptr) {
        plan = *checked;
    } else {
        const int rc = check_attn_args(desc, q, K_shards, V_shards, U_K, U_V, n_valid, topk_idx, k, combine,
                                       scale, y, workspace, workspace_bytes, &plan, scratch_limit);
        if (rc != PIKV_OK) return rc;
    }
    *plan_out = plan;
    if (desc->B == 0) return PIKV_OK;

    const int W = desc_width(desc);
    float *part_acc = static_cast<float *>(workspace);
    float *part_ml = part_acc + (plan.acc_floats * sizeof(float) + 255) / 256 * 64;

    AttnParams p;
    p.q = q;
    p.K = K_shards;
    p.V = V_shards;
    p.U_K = U_K;
    p.n_valid = n_valid;
    p.topk = topk_idx;
    p.part_acc = part_acc;
    p.part_ml = part_ml;
    p.scores = scores;
    p.B = desc->B;
    p.Hq = desc->Hq;
    p.G = desc->Hq / desc->Hkv;
    p.D = desc->D;
    p.E = desc->E;
    p.S = desc->S;
    p.k = k;
    p.rr = desc->route_rows_per_seq;
    p.rank = desc->rank;
    p.tq = desc->tq > 1 ? desc->tq : 1;
    p.stride_h = desc->stride_h;
    p.stride_s = desc->stride_s;
    p.by_nsplit = fast_div(plan.nsplit);
    p.by_k = fast_div(k);
    p.by_groups = fast_div(plan.head_blocks);
    p.by_G = fast_div(p.G);
    p.by_draft = fast_div(p.G / p.tq);
    p.heads = desc->Hq / p.tq;
    p.nsplit = plan.nsplit;
    p.chunk = plan.chunk;
    p.nsplit_rcp = plan.nsplit > 1 ? (uint32_t)(((uint64_t)1 << 32) / plan.nsplit + 1) : 0u;
    p.stage_scores = scores != nullptr && plan.score_stage_bytes > 0;
    p.scale = scale > 0.0f ? scale : 1.0f / sqrtf((float)desc->D);

    const int64_t blocks64 = (int64_t)desc->B * plan.head_blocks * k * plan.nsplit;
    p.stream_scores = blocks64 > plan.resident_blocks;
    CombineParams c;
    c.part_acc = part_acc;
    c.part_ml = part_ml;
    c.gates = gates;
    c.U_V = U_V;
    c.y = y;
    c.row_max = row_max;
    c.row_norm = row_norm;
    c.slot_coef = slot_coef;
    c.Hq = desc->Hq;
    c.G = p.G;
    c.by_Hq = fast_div(c.Hq);
    c.by_G = fast_div(c.G);
    c.D = desc->D;
    c.W = W;
    c.k = k;
    c.rr = p.rr;
    c.rank = desc->rank;
    c.value_bias = (desc->flags & PIKV_DESC_VALUE_BIAS) ? 1 : 0;
    c.tq = p.tq;
    c.nsplit = plan.nsplit;
    c.combine = combine;
    c.decoder_bytes = reinterpret_cast<uintptr_t>(U_V) % 16 == 0 ? combine_decoder_bytes(c.rank, c.value_bias, c.D, elem_bytes(desc->dtype)) : 0;

    hipStream_t st = as_stream(stream);
    int lrc;
    if (g_prof_start) (void)hipEventRecord(g_prof_start, st);
    // (an event pair stands around the split pass alone: two launches then, of the same bits)
    const bool small = merged != nullptr && plan.small && !profile_events_set();
    if (merged != nullptr) *merged = small;
    if (small) {
        lrc = desc->dtype == PIKV_F32 ? launch_small<float>(p, c, desc->B * desc->Hq, st) : launch_small<bf16>(p, c, desc->B * desc->Hq, st);
    } else if (plan.gqa_mfma) {
        const size_t lds = p.stage_scores ? plan.score_stage_bytes : 0;
        const bool codes = desc->rank > 0;
        switch (W) {
            case 16: codes ? launch_gqa<16, true>(plan.row_tiles, plan.long_blocks, p, blocks64, lds, st) : launch_gqa<16, false>(plan.row_tiles, plan.long_blocks, p, blocks64, lds, st); break;
            case 32: codes ? launch_gqa<32, true>(plan.row_tiles, plan.long_blocks, p, blocks64, lds, st) : launch_gqa<32, false>(plan.row_tiles, plan.long_blocks, p, blocks64, lds, st); break;
            case 64: codes ? launch_gqa<64, true>(plan.row_tiles, plan.long_blocks, p, blocks64, lds, st) : launch_gqa<64, false>(plan.row_tiles, plan.long_blocks, p, blocks64, lds, st); break;
            default: launch_gqa<128, false>(plan.row_tiles, plan.long_blocks, p, blocks64, lds, st); break;
        }
        lrc = launch_status();
    } else if (plan.gqa_f32) {
        const bool codes = desc->rank > 0;
        const int gb = plan.heads_per_block;
        switch (W) {
            case 16: codes ? launch_gqa32<16, true>(gb, p, blocks64, st) : launch_gqa32<16, false>(gb, p, blocks64, st); break;
            case 32: codes ? launch_gqa32<32, true>(gb, p, blocks64, st) : launch_gqa32<32, false>(gb, p, blocks64, st); break;
            case 64: codes ? launch_gqa32<64, true>(gb, p, blocks64, st) : launch_gqa32<64, false>(gb, p, blocks64, st); break;
            default: launch_gqa32<128, false>(gb, p, blocks64, st); break;
        }
        lrc = launch_status();
    } else {
        lrc = desc->dtype == PIKV_F32
                  ? launch_partial<float>(W, plan.heads_per_block, p, (int)blocks64, st)
                  : launch_partial<bf16>(W, plan.heads_per_block, p, (int)blocks64, st);
    }
    if (g_prof_stop) (void)hipEventRecord(g_prof_stop, st);
    if (lrc != PIKV_OK) return lrc;

    *c_out = c;
    return PIKV_OK;
}

}  // namespace pikv

namespace pikv {
int pikv_sharded_attn_merge(const pikv_desc *desc, const CombineParams *c, void *stream) {
    const dim3 cgrid(desc->B * desc->Hq);
    hipStream_t st = as_stream(stream);
    const bool f32 = desc->dtype == PIKV_F32;
    const int np = c->k * c->nsplit;
    if (combine_threads(np) == 256) {
        const size_t lds = combine_smem_bytes(256, np, c->decoder_bytes);
        if (f32) hipLaunchKernelGGL((attn_combine<float, 256>), cgrid, dim3(256), lds, st, *c);
        else hipLaunchKernelGGL((attn_combine<bf16, 256>), cgrid, dim3(256), lds, st, *c);
    } else {
        const size_t lds = combine_smem_bytes(1024, np, c->decoder_bytes);
        if (f32) hipLaunchKernelGGL((attn_combine<float, 1024>), cgrid, dim3(1024), lds, st, *c);
        else hipLaunchKernelGGL((attn_combine<bf16, 1024>), cgrid, dim3(1024), lds, st, *c);
    }
    return launch_status();
}
}  // namespace pikv

static int sharded_attn(const pikv_desc *desc, const void *q, const void *const *K_shards,
                        const void *const *V_shards, const void *U_K, const void *U_V, const int32_t *n_valid,
                        const int32_t *topk_idx, const float *gates, int32_t k, int32_t combine, float scale,
                        float *y, float *row_max, float *row_norm, float *scores, float *slot_coef,
                        void *workspace, size_t workspace_bytes, void *stream, size_t scratch_limit) {
    AttnPlan plan;
    CombineParams c;
    bool merged = false;
    const int rc = launch_attn_partial(desc, q, K_shards, V_shards, U_K, U_V, n_valid, topk_idx, gates,
                                       k, combine, scale, y, row_max, row_norm, scores, slot_coef,
                                       workspace, workspace_bytes, stream, nullptr, &plan, &c, scratch_limit, &merged);
    if (rc != PIKV_OK || desc->B == 0 || merged) return rc;
    return pikv_sharded_attn_merge(desc, &c, stream);
}

extern "C" int pikv_sharded_attn(const pikv_desc *desc, const void *q, const void *const *K_shards,
                                 const void *const *V_shards, const void *U_K, const void *U_V,
                                 const int32_t *n_valid, const int32_t *topk_idx,
                                 const float *gates, int32_t k, int32_t combine, float scale,
                                 float *y, float *row_max, float *row_norm, float *scores,
                                 float *slot_coef, void *workspace, size_t workspace_bytes,
                                 void *stream) {
    return sharded_attn(desc, q, K_shards, V_shards, U_K, U_V, n_valid, topk_idx, gates, k, combine, scale, y,
                        row_max, row_norm, scores, slot_coef, workspace, workspace_bytes, stream, SIZE_MAX);
}

// ---------------------------------------------------------------------------------------
// The same call for callers that cannot allocate (code under HIP graph capture, tight serving
// loops): the split partials live in a file-scope device array instead of a caller workspace.
namespace {

constexpr size_t kStaticScratchBytes = PIKV_NOALLOC_SCRATCH_BYTES;   // per GPU, held until the process ends
constexpr int kMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Address of this GPU's copy of `scratch` (every device holds its own copy at its own address),
// looked up once per device with that device current.  In host code the array's name is only a
// handle for this lookup, never an address to pass to a kernel.
int static_scratch(void **out) {
    static void *ptr_of_device[kMaxDevices] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return PIKV_ERR_HIP;
    if (ptr_of_device[dev] == nullptr) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return PIKV_ERR_HIP;
        ptr_of_device[dev] = ptr;
    }
    *out = ptr_of_device[dev];
    return PIKV_OK;
}

}  // namespace

extern "C" int pikv_sharded_attn_noalloc(const pikv_desc *desc, const void *q, const void *const *K_shards,
                                         const void *const *V_shards, const void *U_K, const void *U_V,
                                         const int32_t *n_valid, const int32_t *topk_idx,
                                         const float *gates, int32_t k, int32_t combine, float scale,
                                         float *y, float *row_max, float *row_norm, float *scores,
                                         float *slot_coef, void *stream) {
    const size_t need = workspace_bytes_within(desc, k, kStaticScratchBytes);
    if (need > kStaticScratchBytes) return PIKV_ERR_WORKSPACE;   // geometry too large for the fixed array
    void *ws = nullptr;
    const int rc = static_scratch(&ws);
    if (rc != PIKV_OK) return rc;
    // Every partial the merge reads is written by the split pass of the same call (empty splits
    // write an empty partial), so nothing in the array has to start at zero.
    return sharded_attn(desc, q, K_shards, V_shards, U_K, U_V, n_valid, topk_idx, gates, k, combine, scale, y,
                        row_max, row_norm, scores, slot_coef, ws, kStaticScratchBytes, stream, kStaticScratchBytes);
}
