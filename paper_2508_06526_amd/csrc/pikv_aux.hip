// Two small stages around the hot path:
//
//   router_penalty : the additive per-expert term of PiKV's penalised routers (Section 3.2,
//                    Table 1, column "Penalty Term", rows LB, P and E), one wavefront
//                    (pikv_penalty_dev.h): absorbs this step's selections into the load counter
//                    and writes the bias that the next pikv_route / pikv_decode_step call adds
//                    to the logits.
//   compress_rows  : Algorithm 1, (K^, V^) <- C_cmp(K_t, V_t) for the rank-r linear compressor of
//                    Section 3.3 (Table 2, LoRA rows): code = W_enc x, rounded once to the storage
//                    type.  One block per (sequence, kv head, K or V); 8 lanes per code element read the
//                    encoder row and the vector with 16-byte loads and join by an xor butterfly.
#include "pikv_common.h"
#include "pikv_penalty_dev.h"

#include <math.h>

namespace pikv {
namespace {

__global__ __launch_bounds__(kWave) void router_penalty(PenaltyParams p) { penalty_wave(p, threadIdx.x); }

// Table 1 row B: the score-free round-robin router.  One thread per (routed row, position).
__global__ __launch_bounds__(256) void route_round_robin(int n, int E, int k, long long step, int32_t *topk,
                                                         float *gates) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int r = i / k, j = i - r * k;
    topk[i] = (int32_t)(((step + r) * k + j) % E);
    gates[i] = 1.0f / (float)k;
}

// Measurement kernel: reads `parts` spans of each of n buffers once, the way the attention pass
// reads K/V rows (4 waves per block, a wave load = 1 KiB of consecutive bytes, non-temporal,
// 16 loads of a wave in flight), folds the words (xor) and writes one per block.  No arithmetic
// besides the fold: what it reaches is the most any pass that has to read these bytes can.
__global__ __launch_bounds__(256) void stream_read_probe(const char *const *bufs, size_t bytes_each, size_t span,
                                                         int parts, uint32_t *out) {
    const int buf = blockIdx.x / parts, part = blockIdx.x - buf * parts;
    const char *base = bufs[buf];
    const size_t lo = (size_t)part * span, hi = lo + span < bytes_each ? lo + span : bytes_each;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint4 acc = make_uint4(0, 0, 0, 0);
    constexpr size_t kWaveBytes = 16 * 1024;           // per wave and iteration: 16 loads of 1 KiB
    for (size_t at = lo + (size_t)wave * kWaveBytes; at < hi; at += 4 * kWaveBytes) {
        uint4 v[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const size_t a = at + (size_t)t * 1024 + (size_t)lane * 16;
            const bool in = a + 16 <= hi;
            v[t] = load16_stream(base + (in ? a : hi - 16));   // clamped onto the span's last 16 bytes,
            if (!in) v[t] = make_uint4(0, 0, 0, 0);            // which then do not count
        }
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            acc.x ^= v[t].x;
            acc.y ^= v[t].y;
            acc.z ^= v[t].z;
            acc.w ^= v[t].w;
        }
    }
    uint32_t w = acc.x ^ acc.y ^ acc.z ^ acc.w;
    for (int off = 1; off < 64; off <<= 1) w ^= __shfl_xor(w, off, 64);
    __shared__ uint32_t ws[4];
    if (lane == 0) ws[wave] = w;
    __syncthreads();
    if (threadIdx.x == 0) out[blockIdx.x] = ws[0] ^ ws[1] ^ ws[2] ^ ws[3];
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

template <typename T>
__device__ __forceinline__ void store_elem(T *p, int64_t i, float v);
template <>
__device__ __forceinline__ void store_elem<float>(float *p, int64_t i, float v) {
    p[i] = v;
}
template <>
__device__ __forceinline__ void store_elem<bf16>(bf16 *p, int64_t i, float v) {
    const f32x2_t pair = {v, 0.0f};
    const bf16x2_t r = __builtin_convertvector(pair, bf16x2_t);     // round to nearest even
    p[i].bits = (uint16_t)(__builtin_bit_cast(uint32_t, r) & 0xffffu);
}

// A block's 256 threads take 32 code elements a pass, at most two passes; what both read is requested before either is
// summed (no request under a lane's condition), so that a block is one trip to memory: with a trip per 64 values of
// the head dimension and pass it was two (bf16, rank 32) to eight (kernel trace: 15 x 4 kv heads, rank 64, 3.3 -> 2.6 us, 5 x 2 in
// fp32, rank 16, 2.85 -> 2.5; right behind another kernel's writes 4.6 either way).  Chunks per lane and passes are those of the
// shape, and waves past the rank leave: with the most of both in every shape, clamped, a block of short rows requested up to
// eight times what it needed (in a graph, 84 x 32 kv heads of 16 fp32 values, rank 32, 4.4 us with a trip each, 8.8, now 3.7).
template <typename T, int CHUNKS, int PASSES>
__global__ __launch_bounds__(256) void compress_rows(const T *xK, const T *WK, T *codesK, const T *xV,
                                                     const T *WV, T *codesV, FastDiv by_Hkv, int D, int rank) {
    constexpr int EPL = Pack16<T>::N;
    const T *x = blockIdx.y == 0 ? xK : xV;    // grid.y: 0 = keys, 1 = values
    const T *W_enc = blockIdx.y == 0 ? WK : WV;
    T *codes = blockIdx.y == 0 ? codesK : codesV;
    const int bh = blockIdx.x;                 // b * Hkv + h
    int h;
    fast_divide(by_Hkv, bh, &h);
    const int tid = threadIdx.x, sub = tid & 7;
    if (PASSES == 1 && (tid & ~(kWave - 1)) >= 8 * rank) return;      // wave-uniform
    const int chunks = D / EPL;
    const T *xv = x + (int64_t)bh * D;
    const T *W = W_enc + (int64_t)h * rank * D;
    uint4 xr[CHUNKS], wr[PASSES][CHUNKS];
#pragma unroll
    for (int u = 0; u < CHUNKS; ++u) xr[u] = load16(xv + min(sub + 8 * u, chunks - 1) * EPL);
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass)
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u)
            wr[pass][u] = load16(W + min(32 * pass + (tid >> 3), rank - 1) * D + min(sub + 8 * u, chunks - 1) * EPL);
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
        const int c = 32 * pass + (tid >> 3);
        float a = 0.0f;
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u) {
            float wf[EPL], xf[EPL], with = a;
            Pack16<T>::widen(wr[pass][u], wf);
            Pack16<T>::widen(xr[u], xf);
#pragma unroll
            for (int i = 0; i < EPL; ++i) with = fmaf(wf[i], xf[i], with);
            a = sub + 8 * u < chunks ? with : a;
        }
        a += lane_xor<0>(a);
        a += lane_xor<1>(a);
        a += lane_xor<2>(a);
        if (c < rank && sub == 0) store_elem<T>(codes, (int64_t)bh * rank + c, a);
    }
}

}  // namespace
}  // namespace pikv

using namespace pikv;

extern "C" int pikv_router_penalty(int32_t mode, const int32_t *topk_idx, int32_t rows, int32_t k,
                                   int32_t E, int32_t *load, const int32_t *miss, float coef,
                                   float *bias, void *stream) {
    const int rc = check_penalty(mode, load, miss, coef, bias, E);
    if (rc != PIKV_OK) return rc;
    if (rows < 0 || k < 0) return PIKV_ERR_INVALID;
    if ((int64_t)rows * k > 0 && !topk_idx) return PIKV_ERR_INVALID;
    if ((int64_t)rows * k > 0x7fffffff) return PIKV_ERR_UNSUPPORTED;
    PenaltyParams p;
    p.mode = mode;
    p.topk = topk_idx;
    p.n_sel = rows * k;
    p.E = E;
    p.load = load;
    p.miss = miss;
    p.coef = coef;
    p.bias = bias;
    hipLaunchKernelGGL(router_penalty, dim3(1), dim3(kWave), 0, as_stream(stream), p);
    return launch_status();
}

extern "C" int pikv_compress(const pikv_desc *desc, const void *K_full, const void *Wenc_K,
                             void *K_codes, const void *V_full, const void *Wenc_V, void *V_codes,
                             void *stream) {
    const int rc = check_desc(desc);
    if (rc != PIKV_OK) return rc;
    if (desc->rank == 0 || !K_full || !Wenc_K || !K_codes) return PIKV_ERR_INVALID;
    const bool both = V_full || Wenc_V || V_codes;
    if (both && (!V_full || !Wenc_V || !V_codes)) return PIKV_ERR_INVALID;
    if (desc->B == 0) return PIKV_OK;
    const dim3 grid(desc->B * desc->Hkv, both ? 2 : 1), block(256);
    hipStream_t st = as_stream(stream);
    auto launch = [&](auto type, auto chunks, auto passes) {
        typedef decltype(type) T;
        hipLaunchKernelGGL((compress_rows<T, decltype(chunks)::value, decltype(passes)::value>), grid, block, 0, st,
                           static_cast<const T *>(K_full), static_cast<const T *>(Wenc_K), static_cast<T *>(K_codes),
                           static_cast<const T *>(V_full), static_cast<const T *>(Wenc_V), static_cast<T *>(V_codes),
                           fast_div(desc->Hkv), desc->D, desc->rank);
    };
    const std::integral_constant<int, 1> one{};
    const std::integral_constant<int, 2> two{};
    const std::integral_constant<int, 4> four{};
    auto launch_passes = [&](auto type, auto chunks) {
        if (desc->rank > 32) launch(type, chunks, two);
        else launch(type, chunks, one);
    };
    const int lane_chunks = (desc->D * elem_bytes(desc->dtype) / 16 + 7) / 8;      // 1, 2 or (fp32) 4
    if (desc->dtype == PIKV_F32) {
        if (lane_chunks == 1) launch_passes(float{}, one);
        else if (lane_chunks == 2) launch_passes(float{}, two);
        else launch_passes(float{}, four);
    } else {
        if (lane_chunks == 1) launch_passes(bf16{}, one);
        else launch_passes(bf16{}, two);
    }
    return launch_status();
}

extern "C" int pikv_route_round_robin(int32_t rows, int32_t E, int32_t k, int64_t step,
                                      int32_t *topk_idx, float *gates, void *stream) {
    if (rows < 0 || E < 1 || E > 64 || k < 1 || k > E || step < 0) return PIKV_ERR_INVALID;
    if (!topk_idx || !gates) return PIKV_ERR_INVALID;
    if ((int64_t)rows * k > 0x7fffffff) return PIKV_ERR_UNSUPPORTED;
    if (rows == 0) return PIKV_OK;
    const int n = rows * k;
    hipLaunchKernelGGL(route_round_robin, dim3((n + 255) / 256), dim3(256), 0, as_stream(stream), n, E, k,
                       (long long)step, topk_idx, gates);
    return launch_status();
}


extern "C" int pikv_stream_read_probe(const void *const *bufs, int32_t n, size_t bytes_each, int32_t parts,
                                      uint32_t *out, void *stream) {
    if (!bufs || !out || n < 1 || parts < 1 || bytes_each < 16 || bytes_each % 16 != 0) return PIKV_ERR_INVALID;
    if ((int64_t)n * parts > 0x7fffffff) return PIKV_ERR_INVALID;
    size_t span = (bytes_each + parts - 1) / parts;
    span = (span + 4095) / 4096 * 4096;
    if (span * (size_t)(parts - 1) >= bytes_each) return PIKV_ERR_INVALID;      // a part would be empty
    hipLaunchKernelGGL(stream_read_probe, dim3((unsigned)(n * parts)), dim3(256), 0, as_stream(stream),
                       reinterpret_cast<const char *const *>(bufs), bytes_each, span, parts, out);
    return launch_status();
}
