// PiKV routing (Section 3.2, Table 1 "TopK softmax" with the optional additive penalty):
// one 1024-thread block computes the E logits of x W_r (+ bias), the softmax over all experts
// and the k-hot mask of R routed rows, in a single launch.  R = 1 up to 256 rows (one block per
// CU: a decode step); the rows of a prompt share a block's pass over W_r.
// Every sum of a row is formed in the same order whatever R, so its bits do not depend on it
// (nor do they differ from the decode step's, whose kernel uses the one-row form).
//
//   route_mfma_kernel,
//   route_mfma_few_kernel,
//   route_mfma_rows_kernel : bf16, one row, a few or up to 16, on the matrix cores.
//   route_vec_kernel,
//   route_rows_kernel : fp32, W_r rows that are a power-of-two number of 16-byte chunks.
//   route_single_kernel : fp32, any other E and alignment, few elements.
//   route_flat_kernel,
//   route_flat_rows_kernel : the rest of fp32.
// The sums are described in pikv_route_dev.h.  Selection
// is by rank counting: expert e's rank is the number of experts that beat it under (logit
// descending, index ascending), so the output order and the tie-break need no sorting network.
#include "pikv_common.h"
#include "pikv_route_dev.h"

#include <math.h>

namespace pikv {
namespace {

// bf16, one row.
template <int MOST>
__global__ __launch_bounds__(kRouteThreads) void route_mfma_kernel(const bf16 *x, const bf16 *W_r, const float *bias,
                                                                   int d_r, int E, bool words, int k, int32_t *topk_idx,
                                                                   float *gates, float *probs) {
    __shared__ RouteShared<MOST, 1> sh;
    const int lane = threadIdx.x & (kWave - 1), row = blockIdx.x;
    const float bias_e = route_bias_of_lane(bias, E, lane);
    const float logit = route_logit_mfma<MOST>(x + (int64_t)row * d_r, W_r, d_r, E, words, bias_e, sh);
    if (threadIdx.x < kWave) select_topk(logit, lane, row, E, k, topk_idx, gates, probs);
}

// bf16, several rows, a column of the product for every row and set (route_mfma_few).
template <int MOST>
__global__ __launch_bounds__(kRouteThreads) void route_mfma_few_kernel(const bf16 *x, const bf16 *W_r, const float *bias,
                                                                       int rows, int R, int d_r, int E, int k,
                                                                       int32_t *topk_idx, float *gates, float *probs) {
    constexpr int ROWS = 16 / RouteTiles<MOST>::kSets;
    __shared__ RouteShared<MOST, ROWS> sh;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int row0 = blockIdx.x * R, here = min(R, rows - row0);
    const float bias_e = route_bias_of_lane(bias, E, lane);
    const float logit = route_logits_few<MOST, ROWS>(x + (int64_t)row0 * d_r, here, d_r, W_r, d_r, E, bias_e, sh);
    if (wave < here) select_topk(logit, lane, row0 + wave, E, k, topk_idx, gates, probs);
}

// bf16, up to 16 rows: the rows are one side of the matrix-core product, the experts the other.
// Bound by the bytes: a block of 16 rows of 4096 values reads 128 KiB of x and as much of W_r, which every
// block of an XCD reads from its L2.
template <int MOST, bool WORDS>
__global__ __launch_bounds__(kRouteThreads) void route_mfma_rows_kernel(const bf16 *x, const bf16 *W_r, const float *bias,
                                                                        int rows, int R, int d_r, int E, int k,
                                                                        int32_t *topk_idx, float *gates, float *probs) {
    constexpr int ET = RouteTiles<MOST>::kTiles;
    constexpr int kPitch = 16 * ET + 1;                      // (odd: the rows' sums fall in different banks)
    extern __shared__ float route_sums[];                    // [wave][R][kPitch]
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int c = lane & 15, r = lane >> 4;
    const int row0 = blockIdx.x * R;
    const float bias_e = route_bias_of_lane(bias, E, lane);
    f32x4_t acc[ET];
    route_mfma_rows<MOST, WORDS>(x + (int64_t)min(row0 + min(c, R - 1), rows - 1) * d_r, W_r, d_r, E, acc);
    if (c < R) {
#pragma unroll
        for (int et = 0; et < ET; ++et)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                route_sums[(wave * R + c) * kPitch + route_tile_expert<MOST, WORDS>(et, 4 * r + i)] = acc[et][i];
    }
    __syncthreads();
    if (wave < R && row0 + wave < rows)      // a row per wave
        select_topk(route_logit_joined<MOST, kRouteThreads / kWave>(route_sums + wave * kPitch, R * kPitch, bias_e, E, lane),
                    lane, row0 + wave, E, k, topk_idx, gates, probs);
}

// fp32, one row: a row of W_r is a whole number (1, 2, 4, 8 or 16) of 16-byte chunks; see
// route_logits_vec for the thread layout.
__global__ __launch_bounds__(kRouteThreads) void route_vec_kernel(const float *x, const float *W_r,
                                                                  const float *bias, int d_r,
                                                                  int E, int cpr, int k,
                                                                  int32_t *topk_idx, float *gates,
                                                                  float *probs) {
    __shared__ float red[kRouteThreads / kWave][64];
    const int row = blockIdx.x;
    const float bias_e = route_bias_of_lane(bias, E, threadIdx.x & (kWave - 1));
    route_logits_vec(x + (int64_t)row * d_r, W_r, d_r, cpr, red);
    if (threadIdx.x < 64)
        select_topk(route_logit_of_lane(red[0], 64, bias_e, E, threadIdx.x), threadIdx.x, row, E, k, topk_idx, gates,
                    probs);
}

// fp32, few elements, R rows.
template <int R>
__global__ __launch_bounds__(kRouteThreads) void route_single_kernel(const float *x, const float *W_r, const float *bias,
                                                                     int rows, int d_r, int E, int EP, int k, int32_t *topk_idx,
                                                                     float *gates, float *probs) {
    __shared__ float red[R * kRouteThreads];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6, row0 = blockIdx.x * R;
    const float bias_e = route_bias_of_lane(bias, E, lane);
    const float *xr[R];
#pragma unroll
    for (int q = 0; q < R; ++q) xr[q] = x + (int64_t)min(row0 + q, rows - 1) * d_r;
    route_logits_single<R>(xr, W_r, d_r, E, EP, red);
    if (wave < R && row0 + wave < rows)      // a row per wave
        select_topk(route_logit_single_of_lane(red + wave * kRouteThreads, bias_e, E, lane), lane, row0 + wave, E, k, topk_idx, gates, probs);
}

// fp32, any E and alignment, one row (4096 values x 12 experts, against single elements 9.2 -> 5.1 us, x 24 16.3 -> 7.3;
// several rows, below: 1024 rows 22 -> 9.2 and 40 -> 12.6, 4096 rows 51 -> 29 and 87 -> 43).
__global__ __launch_bounds__(kRouteThreads) void route_flat_kernel(const float *x, const float *W_r, const float *bias,
                                                                   int d_r, int E, int T, bool aligned, int k,
                                                                   int32_t *topk_idx, float *gates, float *probs) {
    __shared__ __attribute__((aligned(16))) float buf[kFlatFloats];
    __shared__ float red[kRouteThreads / kWave][64];
    const int lane = threadIdx.x & (kWave - 1), row = blockIdx.x;
    const float bias_e = route_bias_of_lane(bias, E, lane);
    route_logits_flat(x + (int64_t)row * d_r, W_r, d_r, E, T, aligned, buf, red);
    if (threadIdx.x < kWave) select_topk(route_logit_of_lane(red[0], 64, bias_e, E, lane), lane, row, E, k, topk_idx, gates, probs);
}

// ... several rows: a set of T threads takes RT rows, a block up to 4 sets.  Held to 64 registers, a CU takes two blocks,
// and one's loads cover the other's sums (4096 rows: 2048 values x 6 17.6 -> 13.2 us, 4096 x 24 49.8 -> 43.0).
template <int RT>
__global__ __launch_bounds__(kRouteThreads, RT == 1 ? 4 : 8) void route_flat_rows_kernel(const float *x, const float *W_r, const float *bias,
                                                                        int rows, int sets, int d_r, int E, int EP, int T,
                                                                        bool aligned, int k, int32_t *topk_idx, float *gates,
                                                                        float *probs) {
    constexpr int kWaves = kRouteThreads / kWave;
    extern __shared__ __attribute__((aligned(16))) float flat_sums[];     // [row of the block][4 T], [row][wave][EP]
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int row0 = blockIdx.x * sets * RT;
    const int set = tid / T, t = tid - set * T;
    if (set < sets) {
        const float *xr[RT];
#pragma unroll
        for (int q = 0; q < RT; ++q) xr[q] = x + (int64_t)min(row0 + set * RT + q, rows - 1) * d_r;
        float acc[RT][4];
        route_flat_sums<RT>(t, xr, W_r, d_r, E, T, aligned, acc);
#pragma unroll
        for (int q = 0; q < RT; ++q)
            *reinterpret_cast<float4 *>(flat_sums + (set * RT + q) * 4 * T + 4 * t) = make_float4(acc[q][0], acc[q][1], acc[q][2], acc[q][3]);
    }
    const float bias_e = route_bias_of_lane(bias, E, lane);   // (not across the sums: registers)
    __syncthreads();
    float *red = flat_sums + sets * RT * 4 * T;
    for (int q = 0; q < sets * RT; ++q) {
        const float share = route_flat_share(flat_sums + q * 4 * T, E, EP, T, wave, lane);
        if (lane < EP) red[(q * kWaves + wave) * EP + lane] = share;
    }
    __syncthreads();
    if (wave < sets * RT && row0 + wave < rows)               // a row per wave
        select_topk(route_logit_of_lane(red + wave * kWaves * EP, EP, bias_e, E, lane), lane, row0 + wave, E, k, topk_idx, gates,
                    probs);
}

// Sums of N per-lane values over the lane bits [BIT, 6), each lane ending with N >> (6 - BIT) of
// them (at least one): a lane passes on the half it does not keep, so the whole costs about N
// exchanges instead of N per bit.  The sum of two lanes is the same from either side, hence the
// same bits as the xor butterfly over the same bits in the same order.  `first` becomes the
// index of the lane's first value.
template <int BIT, int N>
__device__ __forceinline__ void scatter_sums(float *v, int lane, int &first) {
    if constexpr (BIT < 6 && N == 1) {
        v[0] += lane_xor<BIT>(v[0]);
        scatter_sums<BIT + 1, 1>(v, lane, first);
    } else if constexpr (BIT < 6) {
        const bool upper = (lane >> BIT) & 1;
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
            if constexpr (BIT >= 4) {        // rows or halves trade places in one instruction
                const uint32_t lo = __float_as_uint(v[i]), hi = __float_as_uint(v[i + N / 2]);
                if constexpr (BIT == 4) {
                    const auto s = __builtin_amdgcn_permlane16_swap(lo, hi, false, false);
                    v[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
                } else {
                    const auto s = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
                    v[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
                }
            } else {
                const float keep = upper ? v[i + N / 2] : v[i], pass = upper ? v[i] : v[i + N / 2];
                v[i] = keep + lane_xor<BIT>(pass);
            }
        }
        if (upper) first += N / 2;
        scatter_sums<BIT + 1, N / 2>(v, lane, first);
    }
}

// The same for R rows: thread layout, order of the multiply-adds, of the lane sums and of the wave
// sums as in route_logits_vec.  What bounds the one-row form over a prompt is W_r itself, read
// from L2 once per row, and the lane exchanges per wave and row; with
// R rows a chunk of W_r meets R values of x in registers.
template <int R, int CSHIFT>
__global__ __launch_bounds__(kRouteThreads) void route_rows_kernel(const float *x, const float *W_r, const float *bias,
                                                                   int rows, int d_r, int E, int k,
                                                                   int32_t *topk_idx, float *gates, float *probs) {
    constexpr int EPL = 4, WAVES = kRouteThreads / kWave;
    constexpr int NB = 2;      // chunks in flight per thread (1024 rows: 2 12.2 us, 1 15.4)
    __shared__ float red[R][WAVES][64];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int row0 = blockIdx.x * R;
    const float bias_e = route_bias_of_lane(bias, E, lane);
    float acc[R * EPL];
#pragma unroll
    for (int i = 0; i < R * EPL; ++i) acc[i] = 0.0f;
    const float *xr[R];
#pragma unroll
    for (int r = 0; r < R; ++r) xr[r] = x + (int64_t)min(row0 + r, rows - 1) * d_r;
    auto batch = [&](int c, auto nload) {
        constexpr int N = decltype(nload)::value;
        uint4 w[N];
        float xj[N][R];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int cu = c + u * kRouteThreads;
            w[u] = load16(W_r + (int64_t)cu * EPL);
#pragma unroll
            for (int r = 0; r < R; ++r) xj[u][r] = xr[r][cu >> CSHIFT];
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            float wf[EPL];
            Pack16<float>::widen(w[u], wf);
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int i = 0; i < EPL; ++i) acc[r * EPL + i] = fmaf(xj[u][r], wf[i], acc[r * EPL + i]);
        }
    };
    const int total = d_r << CSHIFT;
    int c = tid;
    for (; c + (NB - 1) * kRouteThreads < total; c += NB * kRouteThreads) batch(c, std::integral_constant<int, NB>{});
    for (; c < total; c += kRouteThreads) batch(c, std::integral_constant<int, 1>{});
    int first = 0;
    scatter_sums<CSHIFT, R * EPL>(acc, lane, first);
    constexpr int LEFT = R * EPL >> (6 - CSHIFT) > 0 ? R * EPL >> (6 - CSHIFT) : 1;
#pragma unroll
    for (int i = 0; i < LEFT; ++i) {
        const int at = first + i;
        red[at / EPL][wave][(lane & ((1 << CSHIFT) - 1)) * EPL + at % EPL] = acc[i];
    }
    __syncthreads();
    if (wave < R && row0 + wave < rows)      // a row per wave
        select_topk(route_logit_of_lane(red[wave][0], 64, bias_e, E, lane), lane, row0 + wave, E, k, topk_idx, gates, probs);
}

template <int R>
void launch_rows(int cpr, int rows, const float *x, const float *W_r, const float *bias, int d_r, int E, int k,
                 int32_t *topk_idx, float *gates, float *probs, hipStream_t st) {
    const dim3 grid((rows + R - 1) / R), block(kRouteThreads);
    auto go = [&](auto cshift) {
        hipLaunchKernelGGL((route_rows_kernel<R, decltype(cshift)::value>), grid, block, 0, st, x, W_r, bias, rows, d_r,
                           E, k, topk_idx, gates, probs);
    };
    switch (cpr) {
        case 1: go(std::integral_constant<int, 0>{}); break;
        case 2: go(std::integral_constant<int, 1>{}); break;
        case 4: go(std::integral_constant<int, 2>{}); break;
        case 8: go(std::integral_constant<int, 3>{}); break;
        default: go(std::integral_constant<int, 4>{}); break;     // rows of 64 experts
    }
}

// Rows per block, fp32: one block per CU as long as that takes the rows, then 2 and 4 of them.
inline int rows_per_block(int rows) { return rows <= 256 ? 1 : rows <= 512 ? 2 : 4; }

int route_f32(const float *x, const float *W_r, const float *bias, int rows, int d_r, int E, int k, int32_t *topk_idx,
              float *gates, float *probs, hipStream_t st) {
    const dim3 block(kRouteThreads);
    int cpr = 0;
    if (route_vec_ok(W_r, E, &cpr)) {
        switch (rows_per_block(rows)) {
            case 1: hipLaunchKernelGGL(route_vec_kernel, dim3(rows), block, 0, st, x, W_r, bias, d_r, E, cpr, k, topk_idx, gates, probs); break;
            case 2: launch_rows<2>(cpr, rows, x, W_r, bias, d_r, E, k, topk_idx, gates, probs, st); break;
            default: launch_rows<4>(cpr, rows, x, W_r, bias, d_r, E, k, topk_idx, gates, probs, st); break;
        }
        return launch_status();
    }
    if (route_single_ok(d_r, E)) {           // a block per CU as long as that takes the rows, then 2, 4 and 8 of them
        auto go = [&](auto r) {
            constexpr int R = decltype(r)::value;
            hipLaunchKernelGGL((route_single_kernel<R>), dim3((rows + R - 1) / R), block, 0, st, x, W_r, bias, rows, d_r, E,
                               route_flat_pow2(E), k, topk_idx, gates, probs);
        };
        if (rows <= 256) go(std::integral_constant<int, 1>{});
        else if (rows <= 512) go(std::integral_constant<int, 2>{});
        else if (rows <= 1024) go(std::integral_constant<int, 4>{});
        else go(std::integral_constant<int, 8>{});
        return launch_status();
    }
    const int T = route_flat_threads(d_r, E);
    const bool aligned = reinterpret_cast<uintptr_t>(W_r) % 16 == 0;
    if (rows <= 256) {
        hipLaunchKernelGGL(route_flat_kernel, dim3(rows), block, 0, st, x, W_r, bias, d_r, E, T, aligned, k, topk_idx, gates, probs);
        return launch_status();
    }
    // One block per CU as long as a block can take the rows: sets of threads first, then rows of a thread - no more sets than
    // those need, and not three where they cannot take the rows: at 12 rows a block 4096 leave some CUs two blocks and
    // others one (4096 rows x 1024 values x 10 experts 20.0 -> 16.2 us, 1024 rows in blocks of 6 7.4 -> 6.2).
    const int EP = route_flat_pow2(E), want = rows < 16 * 256 ? (rows + 255) / 256 : 16;
    int sets = kRouteThreads / T < 4 ? kRouteThreads / T : 4;
    if (EP == 64 && sets > 2) sets = 2;                       // LDS: at most 96 KiB
    const int RT = sets >= want ? 1 : 2 * sets >= want ? 2 : 4;
    if (sets > (want + RT - 1) / RT) sets = (want + RT - 1) / RT;
    if (sets == 3 && 3 * RT < want) sets = 2;
    auto go = [&](auto rt) {
        constexpr int R = decltype(rt)::value;
        const int per_block = sets * R;
        hipLaunchKernelGGL((route_flat_rows_kernel<R>), dim3((rows + per_block - 1) / per_block), block,
                           (size_t)per_block * (4 * T + kRouteThreads / kWave * EP) * sizeof(float), st, x, W_r, bias, rows, sets,
                           d_r, E, EP, T, aligned, k, topk_idx, gates, probs);
    };
    if (RT == 1) go(std::integral_constant<int, 1>{});
    else if (RT == 2) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 4>{});
    return launch_status();
}

int route_bf16(const bf16 *x, const bf16 *W_r, const float *bias, int rows, int d_r, int E, int k, int32_t *topk_idx,
               float *gates, float *probs, hipStream_t st) {
    const bool words = route_words_ok(x, d_r, W_r, d_r, E);
    // Rows per block: one block per CU as long as a block can take the rows, at most the 16 of a tile.  Rows of 4096
    // values x 16 experts, against the vector form before: 1 row 4.4 -> 3.7 us, 256 6.2 -> 4.5, 512 6.3 -> 5.3, 1024 7.1 ->
    // 5.5, 2048 9.9 -> 7.2, 4096 17.0 -> 10.3; x 12 experts, before element by element: 1 row 9.5 -> 3.7, 4096 41.6 -> 10.2.
    const int R = rows <= 256 ? 1 : rows >= 16 * 256 ? 16 : (rows + 255) / 256;
    auto go = [&](auto most) {
        constexpr int MOST = decltype(most)::value;
        const dim3 grid((rows + R - 1) / R), block(kRouteThreads);
        const size_t lds = (size_t)kRouteThreads / kWave * R * (16 * RouteTiles<MOST>::kTiles + 1) * sizeof(float);
        if (R == 1)
            hipLaunchKernelGGL((route_mfma_kernel<MOST>), grid, block, 0, st, x, W_r, bias, d_r, E, words, k, topk_idx, gates, probs);
        else if (words && MOST <= 16 && R <= 16 / RouteTiles<MOST>::kSets)
            hipLaunchKernelGGL((route_mfma_few_kernel<MOST <= 16 ? MOST : 16>), grid, block, 0, st, x, W_r, bias, rows, R, d_r, E, k, topk_idx, gates, probs);
        else if (words)
            hipLaunchKernelGGL((route_mfma_rows_kernel<MOST, true>), grid, block, lds, st, x, W_r, bias, rows, R, d_r, E, k, topk_idx, gates, probs);
        else
            hipLaunchKernelGGL((route_mfma_rows_kernel<MOST, false>), grid, block, lds, st, x, W_r, bias, rows, R, d_r, E, k, topk_idx, gates, probs);
    };
    switch (route_experts_most(E)) {
        case 8: go(std::integral_constant<int, 8>{}); break;
        case 16: go(std::integral_constant<int, 16>{}); break;
        case 32: go(std::integral_constant<int, 32>{}); break;
        default: go(std::integral_constant<int, 64>{}); break;
    }
    return launch_status();
}

}  // namespace
}  // namespace pikv

using namespace pikv;

extern "C" int pikv_route(const void *x, const void *W_r, const float *bias, int32_t rows,
                          int32_t d_r, int32_t E, int32_t k, int32_t dtype, int32_t *topk_idx,
                          float *gates, float *probs, void *stream) {
    if (!x || !W_r || !topk_idx || !gates) return PIKV_ERR_INVALID;
    if (rows < 0 || d_r < 1 || E < 1 || E > 64 || k < 1 || k > E) return PIKV_ERR_INVALID;
    if (dtype != PIKV_F32 && dtype != PIKV_BF16) return PIKV_ERR_INVALID;
    if (rows == 0) return PIKV_OK;
    hipStream_t st = as_stream(stream);
    if (dtype == PIKV_F32)
        return route_f32(static_cast<const float *>(x), static_cast<const float *>(W_r), bias, rows, d_r, E, k,
                         topk_idx, gates, probs, st);
    return route_bf16(static_cast<const bf16 *>(x), static_cast<const bf16 *>(W_r), bias, rows, d_r, E, k, topk_idx,
                      gates, probs, st);
}
