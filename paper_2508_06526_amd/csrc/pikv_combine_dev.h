// Merging the split partials of the attention pass (PiKV Algorithm 1, f_attn over C[g_t], with
// the router gates): device code shared by the stand-alone combine kernel and the fused
// post-attention kernel of the decode step.
#pragma once

#include "pikv_common.h"

#include <math.h>

namespace pikv {

struct CombineParams {
    const float *part_acc;
    const float *part_ml;
    const float *gates;
    const void *U_V;
    float *y;
    float *row_max;
    float *row_norm;
    float *slot_coef;
    int Hq, G, D, W, k, rr, rank, nsplit, combine;
    int value_bias;   // U_V holds rank + 1 rows per kv head, the last one the decoder's additive term
    int tq;           // draft queries per sequence: y and the row statistics are [B, tq, Hq / tq, ...]
    FastDiv by_Hq, by_G;
    int decoder_bytes;   // of a kv head's rows of U_V that the merge brings into LDS ahead of its sums; 0: it reads them where they are
};

constexpr int kCombinePrefetch = 4;         // partial rows each thread loads before the weights exist
constexpr int kMaxPartialsPerHead = 2048;   // k * nsplit

// (max, normaliser) of one selected shard from its nsplit partial (max, sum) pairs, computed by
// a group of 8 adjacent lanes: lane `sub` takes splits sub, sub+8, ... in ascending order, the
// 8 lane results are joined by an xor butterfly.  Every caller uses this one arrangement, so the
// stand-alone and the fused kernels produce identical bits.  `get(s)` returns split s's pair;
// all 8 lanes of a group must call together (pass nsplit = 0 for a padding group).
// The first kShardPairsHeld pairs of a lane are fetched once and kept (shard_pairs_load), so a
// caller can issue these loads ahead of other, slower ones; later pairs are fetched again in
// each of the two passes.
constexpr int kShardPairsHeld = 4;
struct ShardPairs {
    float2 v[kShardPairsHeld];
};
template <class F>
__device__ __forceinline__ ShardPairs shard_pairs_load(int nsplit, int sub, F get) {
    ShardPairs sp;
#pragma unroll
    for (int u = 0; u < kShardPairsHeld; ++u) {
        const int s = sub + 8 * u;
        sp.v[u] = s < nsplit ? get(s) : make_float2(-INFINITY, 0.0f);
    }
    return sp;
}
template <class F>
__device__ __forceinline__ void shard_stats8(const ShardPairs &sp, int nsplit, int sub, F get, float *M_out,
                                             float *Z_out) {
    float M = -INFINITY;
#pragma unroll
    for (int u = 0; u < kShardPairsHeld; ++u) M = sp.v[u].y > 0.0f ? fmaxf(M, sp.v[u].x) : M;
    for (int s = sub + 8 * kShardPairsHeld; s < nsplit; s += 8) {
        const float2 v = get(s);
        M = v.y > 0.0f ? fmaxf(M, v.x) : M;
    }
    M = bits_max<0, 3>(M);      // xor butterfly over the 8 lanes, inside a DPP row
    float Z = 0.0f;
#pragma unroll
    for (int u = 0; u < kShardPairsHeld; ++u) Z += sp.v[u].y > 0.0f ? sp.v[u].y * __expf(sp.v[u].x - M) : 0.0f;
    for (int s = sub + 8 * kShardPairsHeld; s < nsplit; s += 8) {
        const float2 v = get(s);
        Z += v.y > 0.0f ? v.y * __expf(v.x - M) : 0.0f;
    }
    Z = bits_sum<0, 3>(Z);
    *M_out = M;
    *Z_out = Z;
}
template <class F>
__device__ __forceinline__ void shard_stats8(int nsplit, int sub, F get, float *M_out, float *Z_out) {
    shard_stats8(shard_pairs_load(nsplit, sub, get), nsplit, sub, get, M_out, Z_out);
}

// The k shard weights of one query head in either combine mode, from the per-shard
// (max, normaliser), computed by an aligned group of `kp` lanes (kp = the power of two >= k, at
// most 64): lane j of the group holds shard j's values (Zj = 0 in lanes j >= k), the row max and
// the normaliser are joined by xor butterflies inside the group (fixed order).  Every lane of
// the group must call.  Outputs for the lane's own shard: weight w of its un-normalised
// accumulator and the (shift, coef) pair with p_i = coef * exp(s_i - shift); M and norm are the
// row max / normaliser (the same in every lane of the group).
struct HeadWeights {
    float w, shift, coef, M, norm;
};
__device__ __forceinline__ HeadWeights head_weights(int kp, float Mj, float Zj, float gj, int combine) {
    const bool live = Zj > 0.0f;
    float M = live ? Mj : -INFINITY;
    for (int off = 1; off < kp; off <<= 1) M = fmaxf(M, __shfl_xor(M, off, kWave));
    HeadWeights out;
    out.M = M;
    if (combine == PIKV_COMBINE_LSE) {
        float norm = live ? gj * Zj * __expf(Mj - M) : 0.0f;
        for (int off = 1; off < kp; off <<= 1) norm += __shfl_xor(norm, off, kWave);
        out.norm = norm;
        out.w = live ? gj * __expf(Mj - M) / norm : 0.0f;
        out.shift = live ? M : 0.0f;
        out.coef = live ? gj / norm : 0.0f;
    } else {
        float norm = live ? gj : 0.0f;
        for (int off = 1; off < kp; off <<= 1) norm += __shfl_xor(norm, off, kWave);
        out.norm = norm;
        out.w = live ? gj / (norm * Zj) : 0.0f;
        out.shift = live ? Mj : 0.0f;
        out.coef = out.w;
    }
    return out;
}
// The same from a wave whose 8-lane groups hold the statistics: lanes 8 g .. 8 g + 7 those of shard g % kp of a
// head, kp <= 8.  The joins run over the lane bits 3 .. 5, by moves inside the vector unit - no LDS, no
// barrier - and pair the same values in the same order as head_weights does.
constexpr int kWaveShards = 8;
template <class F>
__device__ __forceinline__ float groups_join(int kp, float x, F op) {
    if (kp > 1) x = op(x, lane_xchg<3>(x));      // (the same value in the 8 lanes of a group)
    if (kp > 2) {
        const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        x = op(__uint_as_float(q[0]), __uint_as_float(q[1]));
    }
    if (kp > 4) {
        const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        x = op(__uint_as_float(h[0]), __uint_as_float(h[1]));
    }
    return x;
}
__device__ __forceinline__ HeadWeights head_weights_of_groups(int kp, float Mj, float Zj, float gj, int combine) {
    const bool live = Zj > 0.0f;
    HeadWeights out;
    out.M = groups_join(kp, live ? Mj : -INFINITY, [](float a, float b) { return fmaxf(a, b); });
    auto add = [](float a, float b) { return a + b; };
    if (combine == PIKV_COMBINE_LSE) {
        const float e = __expf(Mj - out.M);
        out.norm = groups_join(kp, live ? gj * Zj * e : 0.0f, add);
        out.w = live ? gj * e / out.norm : 0.0f;
        out.shift = live ? out.M : 0.0f;
        out.coef = live ? gj / out.norm : 0.0f;
    } else {
        out.norm = groups_join(kp, live ? gj : 0.0f, add);
        out.w = live ? gj / (out.norm * Zj) : 0.0f;
        out.shift = live ? Mj : 0.0f;
        out.coef = out.w;
    }
    return out;
}
inline __host__ __device__ int pow2_at_least(int v) {
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

// One block (THREADS threads) merges the k * nsplit partials of head `bh`.  The partial
// accumulators do not depend on the weights, so their loads are issued first and overlap the
// whole weight computation:
//   phase 0: every thread = (slice of partials, float4 column group) issues its first
//            accumulator loads; the rows of the value decoder are requested as well.
//   phase 1: 8 lanes per selected shard reduce its splits to (max, normaliser), the shards' are joined to
//            the k gate-weighted shard weights in either combine mode, and every partial gets its
//            weight.  Up to kWaveShards shards that is one wave's work from end to end, without a
//            barrier: in blocks of four waves each does it for itself (a SIMD has one of them), in
//            larger ones the first for all.  More shards take the block and its barriers (combine_weights_block).
//   phase 2: weighted sum of the accumulators, slices reduced in a fixed order - across the waves by the
//            block's first wave, inside it lane to lane - then (rank > 0) the value decoder
//            y = ycode U_V[h'], by the same wave.
// The merge is bound by its chain of phases: with a barrier behind each of them (nine in all) the same sums took, as a kernel
// of its own, 4.0 us against 3.3 (4 heads x 16 partials of 64 values) and 5.4 against 4.8 (256 heads x 64 partials of 128).
// Bytes of LDS combine_head<., threads> carves from the buffer it is given (np = k * nsplit
// partials per head).  Sized by the real np, not by its maximum: the blocks are short and
// many, and the LDS they reserve decides how many of them a CU holds at once.
inline __host__ __device__ int combine_np_pad(int np) { return (np + 3) & ~3; }
// rows of [np] floats: a wave's own weights each, or the weights and the sums they come from
inline __host__ __device__ constexpr int combine_weight_copies(int threads) { return threads == 256 ? 4 : 2; }
// The value decoder's rows of a kv head go to LDS with the block's first requests where they are at most this many bytes -
// every bf16 decoder, the largest of which it is; fp32 ones of rank 32 over 128 values without the additive row, of rank 64 over 64
// with or without it; read column by column behind the sums the others are a trip of their own.
constexpr int kDecoderBytesMost = 65 * 128 * 2;
inline int combine_decoder_bytes(int rank, int value_bias, int D, int elem) {
    const int bytes = (rank + value_bias) * D * elem;
    return rank > 0 && bytes <= kDecoderBytesMost ? bytes : 0;
}
inline size_t combine_smem_bytes(int threads, int np, int decoder_bytes) {
    return (size_t)(combine_weight_copies(threads) * combine_np_pad(np) + 4 * 64 + 128 + 4) * 4 + (size_t)threads * 16 + decoder_bytes;
}

// Block size of the merge: one query head rarely has more than a few dozen partials; a small
// block then has the same latency and leaves the rest of the GPU to other work.  The fused
// and the stand-alone kernels use the same rule, which keeps their results bit-identical.
inline int combine_threads(int np) { return np <= 32 ? 256 : 1024; }

// Internal row bh = b * Hq + h (rows ordered kv head, draft query, head of the group) -> the row
// of the caller's [B, tq, Hq / tq] arrays (y, row_max, row_norm).
__device__ __forceinline__ int64_t caller_row(const CombineParams &p, int b, int h) {
    if (p.tq <= 1) return (int64_t)b * p.Hq + h;
    const int heads = p.Hq / p.tq, g = p.G / p.tq;
    const int hk = h / p.G, rem = h - hk * p.G;
    const int t = rem / g, gg = rem - t * g;
    return ((int64_t)b * p.tq + t) * heads + hk * g + gg;
}

// Weights of all partials of a head by the whole block: any k.
template <int THREADS>
__device__ __forceinline__ void combine_weights_block(const CombineParams &p, int bh, int64_t out, const float *ml, float gate,
                                                      float *wt, float *ls, float *scratch, float *live_s) {
    const int tid = threadIdx.x, np = p.k * p.nsplit;
    float *Mj = scratch, *Zj = Mj + 64, *shard_w = Zj + 64, *g_s = shard_w + 64;
    if (tid < p.k) g_s[tid] = gate;
    for (int i = tid; i < np; i += THREADS) {
        const float2 v = *reinterpret_cast<const float2 *>(ml + 2 * i);
        wt[i] = v.x;
        ls[i] = v.y;
    }
    __syncthreads();
    for (int j0 = 0; j0 < p.k; j0 += THREADS / 8) {   // 8 lanes per selected shard
        const int j = j0 + tid / 8;
        float M, Z;
        shard_stats8(j < p.k ? p.nsplit : 0, tid & 7,
                     [&](int sp) { return make_float2(wt[j * p.nsplit + sp], ls[j * p.nsplit + sp]); }, &M, &Z);
        if (j < p.k && (tid & 7) == 0) {
            Mj[j] = M;
            Zj[j] = Z;
        }
    }
    __syncthreads();
    if (tid < kWave) {   // lane j of the first wave owns selected shard j
        const bool mine = tid < p.k;
        const HeadWeights hw = head_weights(pow2_at_least(p.k), mine ? Mj[tid] : 0.0f, mine ? Zj[tid] : 0.0f,
                                            (mine && p.gates) ? g_s[tid] : 1.0f, p.combine);
        if (mine) {
            shard_w[tid] = hw.w;
            if (p.slot_coef)
                *reinterpret_cast<float2 *>(p.slot_coef + ((int64_t)bh * p.k + tid) * 2) =
                    make_float2(hw.shift, hw.coef);
        }
        if (tid == 0) {
            if (p.row_max) p.row_max[out] = hw.M;
            if (p.row_norm) p.row_norm[out] = hw.norm;
            *live_s = hw.M > -INFINITY ? 1.0f : 0.0f;
        }
    }
    __syncthreads();
    // weight of every partial: shard weight * exp(m_split - M_shard)
    for (int i = tid; i < np; i += THREADS) {
        const int j = i / p.nsplit;
        wt[i] = ls[i] > 0.0f ? shard_w[j] * __expf(wt[i] - Mj[j]) : 0.0f;
    }
    __syncthreads();
}

// The same by one wave, k <= kWaveShards: 8 lanes per shard.  `sp`: the pairs of the lane's first splits.
__device__ __forceinline__ void combine_weights_wave(const CombineParams &p, int bh, int64_t out, const float *ml, float gate,
                                                     const ShardPairs &sp, float *wt, bool writes, float *live_s) {
    const int lane = threadIdx.x & (kWave - 1), j = lane >> 3, sub = lane & 7;
    const int nsplit = j < p.k ? p.nsplit : 0;
    const float *mine = ml + 2 * (int64_t)j * p.nsplit;
    auto pair = [&](int s) { return *reinterpret_cast<const float2 *>(mine + 2 * s); };
    float M, Z;
    shard_stats8(sp, nsplit, sub, pair, &M, &Z);
    const HeadWeights hw = head_weights_of_groups(pow2_at_least(p.k), M, Z, gate, p.combine);
    auto weight = [&](float2 v) { return v.y > 0.0f ? hw.w * __expf(v.x - M) : 0.0f; };
#pragma unroll
    for (int u = 0; u < kShardPairsHeld; ++u)
        if (sub + 8 * u < nsplit) wt[j * p.nsplit + sub + 8 * u] = weight(sp.v[u]);
    for (int s = sub + 8 * kShardPairsHeld; s < nsplit; s += 8) wt[j * p.nsplit + s] = weight(pair(s));
    if (writes) {
        if (p.slot_coef && j < p.k && sub == 0)
            *reinterpret_cast<float2 *>(p.slot_coef + ((int64_t)bh * p.k + j) * 2) = make_float2(hw.shift, hw.coef);
        if (lane == 0) {
            if (p.row_max) p.row_max[out] = hw.M;
            if (p.row_norm) p.row_norm[out] = hw.norm;
            *live_s = hw.M > -INFINITY ? 1.0f : 0.0f;
        }
    }
}

__device__ __forceinline__ float4 add4(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }
// N values at a stride of kWave float4, joined as the fixed tree does: i with i + N / 2, down to one.
template <int N>
__device__ __forceinline__ float4 tree_of_waves(const float4 *red) {
    if constexpr (N == 1) return red[0];
    else {
        float4 v[N];
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = red[i * kWave];
#pragma unroll
        for (int half = N / 2; half >= 1; half /= 2)
#pragma unroll
            for (int i = 0; i < half; ++i) v[i] = add4(v[i], v[i + half]);
        return v[0];
    }
}

// The router gate a thread of the merge weighs with: its shard's.
__device__ __forceinline__ float combine_gate(const CombineParams &p, int bh) {
    int h;
    const int b = fast_divide(p.by_Hq, bh, &h);
    const int shard = p.k <= kWaveShards ? (threadIdx.x & (kWave - 1)) >> 3 : threadIdx.x;
    return p.gates != nullptr && shard < p.k ? p.gates[(int64_t)(b * p.rr + (p.rr == 1 ? 0 : h)) * p.k + shard] : 1.0f;
}

// `parts`, `pairs`: the head's k * nsplit accumulators and (max, sum) pairs; `gate()`: combine_gate, or what it gave before.
template <typename T, int THREADS, class F>
__device__ __forceinline__ void combine_head(const CombineParams &p, int bh, unsigned char *smem, const float *parts,
                                             const float *ml, F gate_of) {
    int h, group_head;
    const int b = fast_divide(p.by_Hq, bh, &h);
    const int hk = fast_divide(p.by_G, h, &group_head);
    const int64_t out = caller_row(p, b, h);
    const int tid = threadIdx.x;
    const int np = p.k * p.nsplit;
    constexpr int kWaves = THREADS / kWave;
    constexpr bool kEachWave = kWaves <= 4;      // every wave weighs for itself, a SIMD each

    float4 *red = reinterpret_cast<float4 *>(smem);                  // [THREADS]
    float *wts = reinterpret_cast<float *>(smem + THREADS * 16);    // weights of the partials
    float *scratch = wts + combine_weight_copies(THREADS) * combine_np_pad(np);      // [4 * 64]
    float *ycode = scratch + 4 * 64;                                 // [128]
    float *live_s = ycode + 128;                                     // [1] 1 if any selected shard holds entries
    T *decoder = reinterpret_cast<T *>(live_s + 4);                 // [decoder_bytes]

    const int cbits = __builtin_ctz(p.W) - 2;    // float4 column groups: 4..32, a power of two
    const int cgroups = 1 << cbits;
    const int slices = THREADS >> cbits;         // partial slices
    const int cg = tid & (cgroups - 1), sl = tid >> cbits;
    const float *acc = parts + cg * 4;
    const bool by_wave = p.k <= kWaveShards;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const int shard = by_wave ? lane >> 3 : tid;
    // the pairs and gates first: the weights hang off them, the sums off the weights
    ShardPairs sp;
    if (by_wave) {
        const float *mine = ml + 2 * (int64_t)min(shard, p.k - 1) * p.nsplit;
        sp = shard_pairs_load(shard < p.k ? p.nsplit : 0, lane & 7,
                              [&](int s) { return *reinterpret_cast<const float2 *>(mine + 2 * s); });
    }
    const float gate = gate_of();
    float4 pre[kCombinePrefetch];
#pragma unroll
    for (int u = 0; u < kCombinePrefetch; ++u) {
        const int i = sl + u * slices;
        pre[u] = i < np ? *reinterpret_cast<const float4 *>(acc + (int64_t)i * p.W)
                        : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    const T *U = static_cast<const T *>(p.U_V) + (int64_t)hk * (p.rank + p.value_bias) * p.D;
    if (p.decoder_bytes != 0) {
        const int chunks = (p.rank + p.value_bias) * p.D * (int)sizeof(T) / 16;
        for (int i = tid; i < chunks; i += THREADS)
            reinterpret_cast<uint4 *>(decoder)[i] = load16(reinterpret_cast<const uint4 *>(U) + i);
    }

    float *wt = wts;
    if (!by_wave) {
        combine_weights_block<THREADS>(p, bh, out, ml, gate, wts, wts + combine_np_pad(np), scratch, live_s);
    } else if constexpr (kEachWave) {
        wt = wts + wave * combine_np_pad(np);
        combine_weights_wave(p, bh, out, ml, gate, sp, wt, wave == 0, live_s);
        wave_lds_order();
    } else {
        if (wave == 0) combine_weights_wave(p, bh, out, ml, gate, sp, wt, true, live_s);
        __syncthreads();
    }

    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < kCombinePrefetch; ++u) {
        const int i = sl + u * slices;
        const float w = i < np ? wt[i] : 0.0f;
        a.x = fmaf(w, pre[u].x, a.x);
        a.y = fmaf(w, pre[u].y, a.y);
        a.z = fmaf(w, pre[u].z, a.z);
        a.w = fmaf(w, pre[u].w, a.w);
    }
    for (int i = sl + kCombinePrefetch * slices; i < np; i += slices) {
        const float w = wt[i];
        const float4 v = *reinterpret_cast<const float4 *>(acc + (int64_t)i * p.W);
        a.x = fmaf(w, v.x, a.x);
        a.y = fmaf(w, v.y, a.y);
        a.z = fmaf(w, v.z, a.z);
        a.w = fmaf(w, v.w, a.w);
    }
    red[tid] = a;
    __syncthreads();
    // Fixed-order tree over the slices (a power of two of them): slice s with s + half, half = slices / 2 .. 1.  A
    // wave holds 64 / cgroups slices, so the first steps join the waves and the last ones lanes of the first wave.
    if (wave != 0 && (p.rank == 0 || p.decoder_bytes != 0)) return;
    float4 t = a;
    if (wave == 0) {
        t = tree_of_waves<kWaves>(red + lane);
        auto other = [](float4 v, auto bit) {
            constexpr int BIT = decltype(bit)::value;
            return make_float4(lane_xor<BIT>(v.x), lane_xor<BIT>(v.y), lane_xor<BIT>(v.z), lane_xor<BIT>(v.w));
        };
        t = add4(t, other(t, std::integral_constant<int, 5>{}));
        if (cgroups <= 16) t = add4(t, other(t, std::integral_constant<int, 4>{}));
        if (cgroups <= 8) t = add4(t, other(t, std::integral_constant<int, 3>{}));
        if (cgroups <= 4) t = add4(t, other(t, std::integral_constant<int, 2>{}));
        if (p.rank == 0) {
            if (lane < cgroups) *reinterpret_cast<float4 *>(p.y + out * p.D + lane * 4) = t;
            return;
        }
        if (lane < cgroups) *reinterpret_cast<float4 *>(ycode + lane * 4) = t;
    }
    // value decoder: y = ycode U_V[h'] (+ b[h'], the weights of a row sum to one)
    if (p.decoder_bytes != 0) {
        wave_lds_order();
        for (int d = 2 * lane; d < p.D; d += 2 * kWave) {
            float y0 = 0.0f, y1 = 0.0f;
#pragma unroll 8
            for (int c = 0; c < p.rank; ++c) {
                y0 = fmaf(ycode[c], load_scalar<T>(decoder, c * p.D + d), y0);
                y1 = fmaf(ycode[c], load_scalar<T>(decoder, c * p.D + d + 1), y1);
            }
            if (p.value_bias && *live_s != 0.0f) {
                y0 += load_scalar<T>(decoder, p.rank * p.D + d);
                y1 += load_scalar<T>(decoder, p.rank * p.D + d + 1);
            }
            p.y[out * p.D + d] = y0;              // (y need not be 8-byte aligned)
            p.y[out * p.D + d + 1] = y1;
        }
        return;
    }
    __syncthreads();
    for (int d = tid; d < p.D; d += THREADS) {
        float a2 = 0.0f;
        for (int cidx = 0; cidx < p.rank; ++cidx)
            a2 = fmaf(ycode[cidx], load_scalar<T>(U, (int64_t)cidx * p.D + d), a2);
        if (p.value_bias && *live_s != 0.0f) a2 += load_scalar<T>(U, (int64_t)p.rank * p.D + d);
        p.y[out * p.D + d] = a2;
    }
}

template <typename T, int THREADS>
__device__ __forceinline__ void combine_head(const CombineParams &p, int bh, unsigned char *smem) {
    const int64_t first = (int64_t)bh * p.k * p.nsplit;
    combine_head<T, THREADS>(p, bh, smem, p.part_acc + first * p.W, p.part_ml + first * 2, [&] { return combine_gate(p, bh); });
}

// Host side (pikv_attn.hip).  check_attn_args: every host-side check of the attention call and
// its split plan, nothing launched - a caller with earlier launches of its own (the step's
// routing / insert kernel) rejects bad arguments before anything is enqueued.
int check_attn_args(const pikv_desc *desc, const void *q, const void *const *K_shards,
                    const void *const *V_shards, const void *U_K, const void *U_V,
                    const int32_t *n_valid, const int32_t *topk_idx, int32_t k, int32_t combine,
                    float scale, const float *y, const void *workspace, size_t workspace_bytes,
                    AttnPlan *plan_out, size_t scratch_limit = SIZE_MAX);
// True while a profiling event pair is installed (pikv_set_profile_events).
bool profile_events_set();

// launch_attn_partial: validate and plan - or take the plan that check_attn_args made for the same arguments -, launch the
// split pass only, and fill the parameters of the merge pass.  With `merged` it may launch a kernel that merges as well, and says so.
int launch_attn_partial(const pikv_desc *desc, const void *q, const void *const *K_shards,
                        const void *const *V_shards, const void *U_K, const void *U_V,
                        const int32_t *n_valid, const int32_t *topk_idx, const float *gates,
                        int32_t k, int32_t combine, float scale, float *y, float *row_max,
                        float *row_norm, float *scores, float *slot_coef, void *workspace,
                        size_t workspace_bytes, void *stream, const AttnPlan *checked, AttnPlan *plan_out,
                        CombineParams *c_out, size_t scratch_limit = SIZE_MAX, bool *merged = nullptr);

int pikv_sharded_attn_merge(const pikv_desc *desc, const CombineParams *c, void *stream);

}  // namespace pikv
