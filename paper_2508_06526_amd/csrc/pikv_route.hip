// PiKV routing (Section 3.2, Table 1 "TopK softmax" with the optional additive penalty):
// one 1024-thread block computes the E logits of x W_r (+ bias), the softmax over all experts
// and the k-hot mask of R routed rows, in a single launch.  R = 1 up to 256 rows (one block per
// CU: a decode step); the rows of a prompt share a block's pass over W_r, up to 4 or 8 at a time.
// Every sum of a row is formed in the same order whatever R, so its bits do not depend on it
// (nor do they differ from the decode step's, whose kernel uses the one-row form).
//
//   route_vec_kernel : W_r rows that are a power-of-two number of 16-byte chunks (E = 8..64
//                      in bf16, 4..64 in fp32): 16-byte loads, see pikv_route_dev.h.
//   route_kernel     : any E <= 64: threads laid out as (row slice, expert) with scalar
//                      element loads (consecutive lanes read consecutive elements of W_r),
//                      slices summed by a fixed-order LDS tree.
// Both make the logits (and therefore the selection) independent of scheduling.  Selection
// is by rank counting: expert e's rank is the number of experts that beat it under (logit
// descending, index ascending), so the output order and the tie-break need no sorting network.
#include "pikv_common.h"
#include "pikv_route_dev.h"

#include <math.h>

namespace pikv {
namespace {

// Generic path (any E <= 64): scalar element loads, LDS tree over the row slices.  The thread
// layout and the tree are route_logits_generic's; a W_r element is read once for the R rows.
template <typename T, int R>
__global__ __launch_bounds__(kRouteThreads) void route_kernel(const T *x, const T *W_r,
                                                              const float *bias, int rows, int d_r, int E,
                                                              int EP, int k, int32_t *topk_idx,
                                                              float *gates, float *probs) {
    const int row0 = blockIdx.x * R;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    __shared__ float red[R][kRouteThreads];
    const float bias_e = route_bias_of_lane(bias, E, lane);
    const int e = tid % EP, js = tid / EP, JS = kRouteThreads / EP;
    float acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.0f;
    if (e < E) {
        for (int j = js; j < d_r; j += JS) {
            const float w = load_scalar<T>(W_r, (int64_t)j * E + e);
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] = fmaf(load_scalar<T>(x, (int64_t)min(row0 + r, rows - 1) * d_r + j), w, acc[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) red[r][tid] = acc[r];
    __syncthreads();
    for (int half = JS >> 1; half >= 1; half >>= 1) {
        if (js < half)
#pragma unroll
            for (int r = 0; r < R; ++r) red[r][tid] += red[r][tid + half * EP];
        __syncthreads();
    }
    if (wave < R && row0 + wave < rows)      // a row per wave
        select_topk(route_logit_generic_of_lane(red[wave], bias_e, E, lane), lane, row0 + wave, E, k, topk_idx, gates, probs);
}

// Fast path for one row: a row of W_r is a whole number (1, 2, 4, 8 or 16) of 16-byte chunks; see
// route_logits_vec for the thread layout.
template <typename T>
__global__ __launch_bounds__(kRouteThreads) void route_vec_kernel(const T *x, const T *W_r,
                                                                  const float *bias, int d_r,
                                                                  int E, int cpr, int k,
                                                                  int32_t *topk_idx, float *gates,
                                                                  float *probs) {
    __shared__ float red[kRouteThreads / kWave][64];
    const int row = blockIdx.x;
    const float bias_e = route_bias_of_lane(bias, E, threadIdx.x & (kWave - 1));
    route_logits_vec<T>(x + (int64_t)row * d_r, W_r, bias, d_r, E, cpr, red);
    if (threadIdx.x < 64)
        select_topk(route_logit_of_lane(red, bias_e, E, threadIdx.x), threadIdx.x, row, E, k, topk_idx, gates,
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

// Fast path for R rows: thread layout, order of the multiply-adds, of the lane sums and of the wave
// sums as in route_logits_vec.  What bounds the one-row form over a prompt is W_r itself, read
// from L2 once per row (4096 rows x 128 KiB: 41.6 us), and 40 lane exchanges per wave and row; with
// R rows a chunk of W_r meets R values of x in registers.
template <typename T, int R, int CSHIFT>
__global__ __launch_bounds__(kRouteThreads) void route_rows_kernel(const T *x, const T *W_r, const float *bias,
                                                                   int rows, int d_r, int E, int k,
                                                                   int32_t *topk_idx, float *gates, float *probs) {
    constexpr int EPL = Pack16<T>::N, WAVES = kRouteThreads / kWave;
    // Chunks in flight per thread: the fewer, the more blocks a CU holds, and other blocks hide the
    // trips to L2 (bf16, 4096 rows: 1 chunk 16.4 us, 2 19.2, 4 20.3; fp32, 1024 rows: 2 12.2, 1 15.4)
    constexpr int NB = EPL == 8 ? 1 : 2;
    __shared__ float red[R][WAVES][64];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int row0 = blockIdx.x * R;
    const float bias_e = route_bias_of_lane(bias, E, lane);
    float acc[R * EPL];
#pragma unroll
    for (int i = 0; i < R * EPL; ++i) acc[i] = 0.0f;
    const T *xr[R];
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
            for (int r = 0; r < R; ++r) xj[u][r] = load_scalar<T>(xr[r], cu >> CSHIFT);
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            float wf[EPL];
            Pack16<T>::widen(w[u], wf);
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
        select_topk(route_logit_of_lane(red[wave], bias_e, E, lane), lane, row0 + wave, E, k, topk_idx, gates, probs);
}

template <typename T, int R>
void launch_rows(int cpr, int rows, const T *x, const T *W_r, const float *bias, int d_r, int E, int k,
                 int32_t *topk_idx, float *gates, float *probs, hipStream_t st) {
    const dim3 grid((rows + R - 1) / R), block(kRouteThreads);
    auto go = [&](auto cshift) {
        hipLaunchKernelGGL((route_rows_kernel<T, R, decltype(cshift)::value>), grid, block, 0, st, x, W_r, bias, rows, d_r,
                           E, k, topk_idx, gates, probs);
    };
    switch (cpr) {
        case 1: go(std::integral_constant<int, 0>{}); break;
        case 2: go(std::integral_constant<int, 1>{}); break;
        case 4: go(std::integral_constant<int, 2>{}); break;
        case 8: go(std::integral_constant<int, 3>{}); break;
        default: go(std::integral_constant<int, 4>{}); break;     // 16: fp32 rows of 64 experts
    }
}

// Rows per block: one block per CU as long as that takes the rows, then 2 and 4 of them - and 8 in
// the generic form, whose scalar reads of W_r weigh more than its longer blocks (12 experts, 4096
// rows: 41.0 against 50.1 us with 4; the fast form with 8 takes 27.9 us against 20.3: 128 registers).
// Measured, rows of 4096 values x 16 experts in bf16, one row per block -> this rule: 512 rows 6.4 ->
// 4.7 us, 1024 10.1 -> 6.3, 2048 23.1 -> 9.7, 4096 41.6 -> 16.4; 12 experts, 4096 rows 157 -> 41.
inline int rows_per_block(int rows, int most) {
    int R = 1;
    while (R < most && rows > 256 * R) R *= 2;
    return R;
}

template <typename T>
int route(const T *x, const T *W_r, const float *bias, int rows, int d_r, int E, int k, int32_t *topk_idx,
          float *gates, float *probs, int dtype, hipStream_t st) {
    const dim3 block(kRouteThreads);
    int cpr = 0;
    if (route_vec_ok(W_r, E, dtype, &cpr)) {
        switch (rows_per_block(rows, 4)) {
            case 1: hipLaunchKernelGGL(route_vec_kernel<T>, dim3(rows), block, 0, st, x, W_r, bias, d_r, E, cpr, k, topk_idx, gates, probs); break;
            case 2: launch_rows<T, 2>(cpr, rows, x, W_r, bias, d_r, E, k, topk_idx, gates, probs, st); break;
            default: launch_rows<T, 4>(cpr, rows, x, W_r, bias, d_r, E, k, topk_idx, gates, probs, st); break;
        }
        return launch_status();
    }
    int EP = 1;
    while (EP < E) EP <<= 1;
    auto go = [&](auto r) {
        constexpr int R = decltype(r)::value;
        hipLaunchKernelGGL((route_kernel<T, R>), dim3((rows + R - 1) / R), block, 0, st, x, W_r, bias, rows, d_r, E, EP, k,
                           topk_idx, gates, probs);
    };
    switch (rows_per_block(rows, 8)) {
        case 1: go(std::integral_constant<int, 1>{}); break;
        case 2: go(std::integral_constant<int, 2>{}); break;
        case 4: go(std::integral_constant<int, 4>{}); break;
        default: go(std::integral_constant<int, 8>{}); break;
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
        return route<float>(static_cast<const float *>(x), static_cast<const float *>(W_r), bias, rows, d_r, E, k,
                            topk_idx, gates, probs, dtype, st);
    return route<bf16>(static_cast<const bf16 *>(x), static_cast<const bf16 *>(W_r), bias, rows, d_r, E, k, topk_idx,
                       gates, probs, dtype, st);
}
