// Device-side pieces of the router shared by the stand-alone routing kernel and the fused
// step kernel (PiKV Section 3.2, Table 1 "TopK softmax").
#pragma once

#include <type_traits>

#include "pikv_common.h"

#include <math.h>

namespace pikv {

constexpr int kRouteThreads = 1024;

// Softmax over the E logits, rank-count selection and gate renormalisation by one wavefront,
// from registers: lane e holds expert e's logit (-inf in lanes >= E).  Returns the lane's rank
// under (logit descending, index ascending); lanes with rank < k are the selection.  Every
// wavefront that calls it with the same logits gets the same result, so a block may let all
// its waves call it instead of broadcasting one wave's result through a barrier.
// Lane i receives the value of lane (i - R) & 15 of its row of 16 lanes (DPP row rotate right).
template <int R>
__device__ __forceinline__ float row_rotate(float x) {
    static_assert(R >= 1 && R <= 15, "rotation inside a row of 16 lanes");
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + R, 0xf, 0xf, true));
}

// rank += [expert (lane - R) & 15 beats this lane's expert], R = 1 .. 15: with E <= 16 all experts
// sit in the first row of 16 lanes, and every pair meets in one rotation without the scalar unit.
template <int R>
__device__ __forceinline__ void rank_by_rotation(float mine, int lane, int &rank) {
    if constexpr (R <= 15) {
        const float other = row_rotate<R>(mine);
        const int o = (lane - R) & 15;
        rank += (other > mine) || (other == mine && o < lane);
        rank_by_rotation<R + 1>(mine, lane, rank);
    }
}

// The selection in two parts, so that a caller can start what depends on the selected experts
// alone (their ranks) before the gates exist: the rank needs the logits only, the gates need the
// softmax as well.
//   route_rank : the lane's rank under (logit descending, index ascending), 64 in lanes >= E.
//   route_gates: softmax over the E logits, the gates of the k selected experts renormalised
//                over the selection; writes topk_idx / gates (and probs) when given.
__device__ __forceinline__ int route_rank(float mine, int lane, int E) {
    int rank = 0;
    if (E <= 16) {
        rank_by_rotation<1>(mine, lane, rank);
    } else {
        for (int o = 0; o < E; ++o) {      // every lane's logit passes through the scalar unit
            const float other = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), o));
            rank += (other > mine) || (other == mine && o < lane);
        }
    }
    return lane < E ? rank : 64;
}
__device__ __forceinline__ void route_gates(float mine, int rank, int lane, int row, int E, int k,
                                            int32_t *topk_idx, float *gates, float *probs) {
    // Lanes >= E hold the identities (-inf, 0), and only lanes < E use the results: with E <= 16
    // the butterflies stay inside the first row of 16 lanes (same operands, same bits).
    const bool one_row = E <= 16;
    const float mx = one_row ? bits_max<0, 4>(mine) : bits_max<0, 6>(mine);
    const float pe = lane < E ? __expf(mine - mx) : 0.0f;
    const float den = one_row ? bits_sum<0, 4>(pe) : bits_sum<0, 6>(pe);
    if (probs && lane < E) probs[(int64_t)row * E + lane] = pe / den;
    const bool chosen = lane < E && rank < k;
    const float picked = chosen ? pe : 0.0f;
    const float sel = one_row ? bits_sum<0, 4>(picked) : bits_sum<0, 6>(picked);
    if (chosen && topk_idx) {
        topk_idx[(int64_t)row * k + rank] = lane;
        gates[(int64_t)row * k + rank] = pe / sel;
    }
}
__device__ __forceinline__ int select_topk(float mine, int lane, int row, int E, int k,
                                           int32_t *topk_idx, float *gates, float *probs) {
    const int rank = route_rank(mine, lane, E);
    route_gates(mine, rank, lane, row, E, k, topk_idx, gates, probs);
    return rank;
}

// The logits, four forms.  Each ends with partial sums in LDS that route_logit_of_lane joins, and none depends on scheduling or on how many rows share a block: a row's
// logits are the same bits in a decode step, in a call of a few rows and in a prompt.
//
// (1) bf16 on the matrix cores, any E and d_r.  The block's 16 waves cut the contraction into units of
// 128 values, unit s to wave s % 16; a unit is four steps of 32 indices, each with a running sum of its
// own over the wave's units (kChains; short chains, and independent products).
// The operand of W_r wants 8 rows of one expert in a lane, and memory holds a row's experts side by
// side: lanes read 32-bit words of two experts and make operands of the words' low and high halves.  16 lanes
// cover kSets = S rows of W_r (4 rows of up to 8 experts, 2 of up to 16, else 1); S steps are taken as a
// group, in which set s of lane group r has, as slot t of its step, index 4 S t + S r + s: one load
// instruction then reads 256 consecutive bytes of W_r.  (With 8 consecutive rows in a lane it touched 8 - 16
// cache lines instead of 2: one row of 4096 values took 4.2 us at any number of experts up to 16.)
//
// With few routed rows there are columns of the product to spare.  Rather than trade words among the
// lanes until all 16 hold the same indices, each set keeps its rows of W_r, a routed row's x stands in a column
// per set, and of the product only the places where set and column agree are used: up to 16 / S rows
// (route_mfma_few).  x is read once per wave, 8 bytes a lane, and comes back from LDS as operands.
// With up to 16 rows (a long prompt) every column is a row, and the lanes do trade (route_mfma_rows; 1024 rows of
// 4096 values over 8 experts 6.4 us that way and 4.6 with a column per set).  The sums are the same.
constexpr int kRouteUnit = 128;

template <int MOST>                      // experts at most: 8, 16, 32, 64
struct RouteTiles {
    static constexpr int kLanes = MOST == 8 ? 4 : MOST == 16 ? 8 : 16;   // that cover a row of W_r
    static constexpr int kSets = 16 / kLanes;
    static constexpr int kWords = MOST == 64 ? 2 : 1;                    // of a lane, a load each: word c and 16 + c
    static constexpr int kGroups = 4 / kSets;                            // of kSets steps in a unit
    static constexpr int kChains = MOST == 64 ? 2 : 4;                   // (64: registers)
    static constexpr int kTiles = MOST <= 16 ? 1 : MOST / 16;            // of 16 experts
    static constexpr int kSums = (kRouteThreads / kWave) * kSets;        // partial sums of one row in LDS
    static constexpr int kUnits = MOST == 8 ? 4 : MOST == 16 ? 2 : 1;    // units in flight, one row
    static constexpr int kRowUnits = MOST <= 16 ? 2 : 1;                 // ... several
};
// Units in flight of route_mfma_few: with several rows two, x takes its share of the registers.
template <int MOST, int ROWS>
constexpr int route_few_units() {
    return ROWS == 1 || RouteTiles<MOST>::kUnits < 2 ? RouteTiles<MOST>::kUnits : 2;
}
inline int route_experts_most(int E) { return E <= 8 ? 8 : E <= 16 ? 16 : E <= 32 ? 32 : 64; }
// Are x (rows `x_stride` elements apart) and W_r fit for words, and W_r for 32-bit offsets?
inline bool route_words_ok(const void *x, int64_t x_stride, const void *W_r, int d_r, int E) {
    return E % 2 == 0 && (int64_t)d_r * E < ((int64_t)1 << 30) && x_stride % 8 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0 &&
           reinterpret_cast<uintptr_t>(W_r) % 4 == 0;
}
__device__ __forceinline__ uint32_t route_halves(uint32_t first, uint32_t second, bool high) {
    return __builtin_amdgcn_perm(second, first, high ? 0x07060302u : 0x05040100u);
}

// A wave-uniform address, hidden from the optimiser: it would otherwise carry one running address per load
// through the loops (a vector register pair each, set up ahead of the first request) instead of a scalar
// base and the lane's 32-bit offsets.
typedef const char __attribute__((address_space(1))) *global_bytes;
__device__ __forceinline__ global_bytes route_base(const bf16 *p) {
    uint64_t a = reinterpret_cast<uint64_t>(p);
    asm volatile("" : "+s"(a));
    return (global_bytes)a;
}
// The same for a unit's number: the sums that lead to its addresses stay in the loop, a few scalar
// instructions, rather than in front of it, where the first requests wait for them.
__device__ __forceinline__ uint32_t route_unit(int unit) {
    asm volatile("" : "+s"(unit));
    return (uint32_t)unit;
}
// (... and widen the offsets outside of the loop, which the addressing mode does by itself.)
__device__ __forceinline__ uint32_t route_offset(uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ uint32_t route_word(global_bytes from) {
    return *(const uint32_t __attribute__((address_space(1))) *)from;
}
// The whole units of a contraction.  (Where up to 64 experts take two words of a lane, the second may lie past
// the row's end, in the next row: the unit of the last row then counts as not whole.)
template <int MOST>
__device__ __forceinline__ int route_whole_units(int d_r, int E) {
    return (int)((uint32_t)(MOST == 64 && E < 64 ? d_r - 1 : d_r) / kRouteUnit);
}

// Element `at` of `left` (the others are zero), `stride` elements apart.
__device__ __forceinline__ uint32_t route_end_element(global_bytes from, int at, int left, int stride) {
    const uint32_t bits = *(const uint16_t __attribute__((address_space(1))) *)(from + 2 * (uint32_t)(min(at, left - 1) * stride));
    return at < left ? bits : 0u;
}

// The words of the lane's 8 slots, 4 S rows apart from row `first` on, of `left` rows (the others are zero).
template <int MOST>
__device__ __forceinline__ void route_end_words(uint32_t (&w)[8][RouteTiles<MOST>::kWords], global_bytes rows, int first,
                                                int left, int E, int w_col) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const int at = first + 4 * RouteTiles<MOST>::kSets * t;
#pragma unroll
        for (int i = 0; i < RouteTiles<MOST>::kWords; ++i) {
            const uint32_t word = route_word(rows + 2 * (uint32_t)(min(at, left - 1) * E + min(w_col + 32 * i, E - 2)));
            w[t][i] = at < left ? word : 0u;
        }
    }
}
// The same of x.
template <int S>
__device__ __forceinline__ uint4 route_end_x(global_bytes xs, int first, int left) {
    uint32_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        v[u] = route_end_element(xs, first + 4 * S * (2 * u), left, 1) | route_end_element(xs, first + 4 * S * (2 * u + 1), left, 1) << 16;
    return make_uint4(v[0], v[1], v[2], v[3]);
}

// Up to ROWS routed rows (1 or 16 / S), R of them, x_stride elements apart: row q's set s in column S q + s.
// sums[q][wave * S + set][expert]; block_x: 256 * kUnits * ROWS bytes of LDS per wave (route_few_units).
// Every wave of the block calls; a block barrier has to follow.
template <int MOST, int ROWS>
__device__ __forceinline__ void route_mfma_few(const bf16 *x, int R, int x_stride, const bf16 *W_r, int d_r, int E,
                                               unsigned char *block_x, float (*sums)[RouteTiles<MOST>::kSums][MOST]) {
    using Tiles = RouteTiles<MOST>;
    constexpr int S = Tiles::kSets, GROUPS = Tiles::kGroups, CH = Tiles::kChains / S, NW = Tiles::kWords;
    constexpr int kWaves = kRouteThreads / kWave, kMost = route_few_units<MOST, ROWS>();
    static_assert(ROWS == 1 || (ROWS == 16 / S && S > 1), "a column per row and set");
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, r = lane >> 4;
    const int set = c / Tiles::kLanes, column = c & (S - 1), row = ROWS == 1 ? 0 : c / S;
    const int w_col = min(2 * (c % Tiles::kLanes), E - 2);    // (past the last expert: the last two)
    constexpr int kUnitBytes = 2 * kRouteUnit * ROWS;         // of x
    unsigned char *wave_x = block_x + wave * (kUnitBytes * kMost);
    f32x4_t acc[CH][2 * NW];                                  // [chain of the set][half of a word]
#pragma unroll
    for (int ch = 0; ch < CH; ++ch)
#pragma unroll
        for (int i = 0; i < 2 * NW; ++i) acc[ch][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // offsets of the lane's 8 rows from the first row of a group, the same for every group: a load is then
    // a scalar base and one of these
    uint32_t w_at[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) w_at[t] = 2 * ((uint32_t)((4 * S * t + S * r + set) * E) + w_col);
    struct Unit {
        uint32_t w[GROUPS][8][NW];
    };
    auto multiply = [&](const Unit &u, int g, uint4 xg) {
#pragma unroll
        for (int i = 0; i < 2 * NW; ++i) {
            const auto &w = u.w[g];
            const uint4 rows = make_uint4(route_halves(w[0][i >> 1], w[1][i >> 1], i & 1), route_halves(w[2][i >> 1], w[3][i >> 1], i & 1),
                                          route_halves(w[4][i >> 1], w[5][i >> 1], i & 1), route_halves(w[6][i >> 1], w[7][i >> 1], i & 1));
            acc[g % CH][i] = mfma_rows(rows, xg, acc[g % CH][i]);
        }
    };
    // x in LDS, by unit and row: operand (column, group r) of a group of steps is the 16 bytes at
    // 16 (S r + column); the lane brings indices 4 j .. 4 j + 3 of a row and unit, j = lane % 32, which are slot t of
    // four neighbouring operands.  A load covers two rows of a unit, or one row's part of two units.
    const int xj = 4 * (lane & 31);
    const uint32_t x_to = 64 * S * (xj / (32 * S)) + 16 * (xj % (4 * S)) + 2 * (xj % (32 * S) / (4 * S));
    auto units = [&](int unit, auto count) {                  // units unit, unit + 16, ...
        constexpr int N = decltype(count)::value, PARTS = N * ROWS, XL = PARTS > 1 ? PARTS / 2 : 1;
        const uint4 *x_of_lane = reinterpret_cast<const uint4 *>(wave_x + 2 * kRouteUnit * row + 16 * (S * r + column));
        Unit op[N];
        const uint32_t k0 = route_unit(unit) * kRouteUnit;
        uint32_t at[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) at[t] = route_offset(w_at[t]);
        auto part = [&](int h) { return PARTS > 1 ? 2 * h + (lane >> 5) : 0; };   // (one part: twice)
        uint2 xv[XL];
#pragma unroll
        for (int h = 0; h < XL; ++h) {
            typedef uint32_t words_t __attribute__((ext_vector_type(2)));
            const int q = min(part(h) % ROWS, R - 1);
            const words_t v = *(const words_t __attribute__((address_space(1))) *)(
                route_base(x + k0) + route_offset(2 * (part(h) / ROWS * kWaves * kRouteUnit + q * x_stride + xj)));
            xv[h] = make_uint2(v[0], v[1]);
        }
#pragma unroll
        for (int n = 0; n < N; ++n) {
#pragma unroll
            for (int g = 0; g < GROUPS; ++g) {
                const global_bytes rows = route_base(W_r + (k0 + n * kWaves * kRouteUnit + 32 * S * g) * (uint32_t)E);
#pragma unroll
                for (int t = 0; t < 8; ++t)
#pragma unroll
                    for (int i = 0; i < NW; ++i) op[n].w[g][t][i] = route_word(rows + 64 * i + at[t]);
            }
        }
#pragma unroll
        for (int h = 0; h < XL; ++h) {
            unsigned char *to = wave_x + 2 * kRouteUnit * part(h) + x_to;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<uint16_t *>(to + 16 * i) = (uint16_t)((i < 2 ? xv[h].x : xv[h].y) >> (16 * (i & 1)));
        }
        wave_lds_order();
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int g = 0; g < GROUPS; ++g) multiply(op[n], g, x_of_lane[kUnitBytes / 16 * n + 4 * S * g]);
        wave_lds_order();
    };
    const int whole = route_whole_units<MOST>(d_r, E);
    int unit = wave;
    for (; unit + (kMost - 1) * kWaves < whole; unit += kMost * kWaves) units(unit, std::integral_constant<int, kMost>{});
    if constexpr (kMost > 2)
        for (; unit + kWaves < whole; unit += 2 * kWaves) units(unit, std::integral_constant<int, 2>{});
    if constexpr (kMost > 1)
        for (; unit < whole; unit += kWaves) units(unit, std::integral_constant<int, 1>{});
    const int left = d_r - whole * kRouteUnit;
    if (unit == whole && left > 0) {                          // what is left, in the wave whose turn it is: zeros from d_r on
        const global_bytes rows = route_base(W_r + (uint32_t)whole * kRouteUnit * (uint32_t)E);
        const global_bytes xs = route_base(x + (int64_t)whole * kRouteUnit) + 2 * (uint32_t)(min(row, R - 1) * x_stride);
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            Unit op;
            route_end_words<MOST>(op.w[g], rows, 32 * S * g + S * r + set, left, E, w_col);
            multiply(op, g, route_end_x<S>(xs, 32 * S * g + S * r + column, left));
            __builtin_amdgcn_sched_barrier(0);               // (a group's loads at a time: registers)
        }
    }
    // the places where set and column agree: rows 4r .. 4r + 3 of the product are lanes 4r .. of a load
    if ((S == 1 || column == 4 * r / Tiles::kLanes) && (ROWS > 1 ? row < R : c < S)) {
#pragma unroll
        for (int i = 0; i < 2 * NW; ++i) {
            f32x4_t total = acc[0][i];
            if constexpr (CH == 2) total = acc[0][i] + acc[1][i];
            if constexpr (CH == 4) total = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
#pragma unroll
            for (int y = 0; y < 4; ++y)
                sums[row][wave * S + column][32 * (i >> 1) + 2 * ((4 * r + y) % Tiles::kLanes) + (i & 1)] = total[y];
        }
    }
}

// Transpose of 4 registers over the 4 rows of 16 lanes: v[u] of row r becomes v[r] of row u.
__device__ __forceinline__ void route_transpose(uint32_t (&v)[4]) {
    auto swap32 = [](uint32_t &a, uint32_t &b) {             // a's upper half for b's lower one
        const auto o = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = o[0], b = o[1];
    };
    auto swap16 = [](uint32_t &a, uint32_t &b) {             // a's odd rows for b's even ones
        const auto o = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = o[0], b = o[1];
    };
    swap32(v[0], v[2]);
    swap32(v[1], v[3]);
    swap16(v[0], v[1]);
    swap16(v[2], v[3]);
}

// Set s's word of what 16 lanes loaded, in the lanes that use it: of two sets in all (lanes c and c + 8), of four in
// lanes 0 - 7 (banks 0 and 1 of the row's four).
template <int S>
__device__ __forceinline__ int route_set_word(int s, int mine) {
    if constexpr (S == 2) {
        if (s == 0) return __builtin_amdgcn_update_dpp(mine, mine, 0x128, 0xf, 0xc, false);     // lanes 8 - 15: from 8 below
        return __builtin_amdgcn_update_dpp(mine, mine, 0x128, 0xf, 0x3, false);                 // lanes 0 - 7: from 8 above
    } else if constexpr (S == 4) {
        int w;
        switch (s) {
            case 0: return __builtin_amdgcn_update_dpp(mine, mine, 0x124, 0xf, 0x2, false);     // bank 1 from 4 below
            case 1: return __builtin_amdgcn_update_dpp(mine, mine, 0x12c, 0xf, 0x1, false);     // bank 0 from 4 above
            case 2:
                w = __builtin_amdgcn_update_dpp(mine, mine, 0x128, 0xf, 0x1, false);            // bank 0 from 8 above
                return __builtin_amdgcn_update_dpp(w, mine, 0x12c, 0xf, 0x2, false);            // bank 1 from 4 above
            default:
                w = __builtin_amdgcn_update_dpp(mine, mine, 0x124, 0xf, 0x1, false);            // bank 0 from 12 above
                return __builtin_amdgcn_update_dpp(w, mine, 0x128, 0xf, 0x2, false);            // bank 1 from 8 above
        }
    } else {
        return mine;
    }
}

// The expert of row mm (0 .. 15) of tile et in route_mfma_rows.
template <int MOST, bool WORDS>
__device__ __forceinline__ int route_tile_expert(int et, int mm) {
    if (!WORDS) return 16 * et + mm;
    if (MOST == 8) return mm < 8 ? 2 * (mm & 3) + (mm >> 2) : mm;      // (rows 8 .. 15 are no experts)
    if (MOST == 16) return 2 * (mm & 7) + (mm >> 3);
    return 32 * (et >> 1) + 2 * mm + (et & 1);
}
// Up to 16 rows: x is the lane's row (row c of the block's); acc: the wave's sums, experts
// route_tile_expert(et, 4r + i) of row c.  Without WORDS (odd E, x or W_r not aligned) element by element.
template <int MOST, bool WORDS>
__device__ __forceinline__ void route_mfma_rows(const bf16 *x, const bf16 *W_r, int d_r, int E,
                                                f32x4_t (&acc)[RouteTiles<MOST>::kTiles]) {
    using Tiles = RouteTiles<MOST>;
    constexpr int ET = Tiles::kTiles, S = Tiles::kSets, GROUPS = Tiles::kGroups, NW = Tiles::kWords, CH = Tiles::kChains;
    constexpr int kWaves = kRouteThreads / kWave, kMost = Tiles::kRowUnits;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, r = lane >> 4;
    f32x4_t chain[CH][ET];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch)
#pragma unroll
        for (int et = 0; et < ET; ++et) chain[ch][et] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int whole = route_whole_units<MOST>(d_r, E);
    int unit = wave;
    if constexpr (WORDS) {
        const int set = c / Tiles::kLanes;
        const int w_col = min(2 * (c % Tiles::kLanes), E - 2);
        uint32_t w_at[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) w_at[t] = 2 * ((uint32_t)((4 * S * t + S * r + set) * E) + w_col);
        struct Group {
            uint32_t w[8][NW];
            uint32_t x[S][4];                                // a load each
        };
        // the operand of tile et of step s: word u holds the lane's expert in slots 2u (low half) and 2u + 1
        auto w_operand = [&](const Group &op, int s, int et) {
            uint32_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                uint32_t of[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    of[i] = (uint32_t)route_set_word<S>(s, (int)op.w[2 * u + i][et >> 1]);
                }
                if constexpr (S > 1) v[u] = __builtin_amdgcn_perm(of[1], of[0], c >= Tiles::kLanes ? 0x07060302u : 0x05040100u);
                else v[u] = route_halves(of[0], of[1], et & 1);
            }
            return make_uint4(v[0], v[1], v[2], v[3]);
        };
        auto multiply = [&](const Group &op, int g, int s, uint4 xs) {
#pragma unroll
            for (int et = 0; et < ET; ++et)
                chain[(g * S + s) % CH][et] = mfma_rows(w_operand(op, s, et), xs, chain[(g * S + s) % CH][et]);
        };
        auto units = [&](int unit, auto count) {
            constexpr int N = decltype(count)::value;
            Group op[N * GROUPS];
            const uint32_t k0 = route_unit(unit) * kRouteUnit;
            uint32_t at[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) at[t] = route_offset(w_at[t]);
#pragma unroll
            for (int q = 0; q < N * GROUPS; ++q) {
                const uint32_t k = k0 + q / GROUPS * kWaves * kRouteUnit + 32 * S * (q % GROUPS);
#pragma unroll
                for (int h = 0; h < S; ++h) {
                    const uint4 v = load16(x + k + 32 * h + 8 * r);
                    op[q].x[h][0] = v.x, op[q].x[h][1] = v.y, op[q].x[h][2] = v.z, op[q].x[h][3] = v.w;
                }
                const global_bytes rows = route_base(W_r + k * (uint32_t)E);
#pragma unroll
                for (int t = 0; t < 8; ++t)
#pragma unroll
                    for (int i = 0; i < NW; ++i) op[q].w[t][i] = route_word(rows + 64 * i + at[t]);
            }
#pragma unroll
            for (int q = 0; q < N * GROUPS; ++q) {
                auto &v = op[q].x;
                if constexpr (S == 1) {                      // lane u's indices 8u + r and 8u + 4 + r to lane group r, word u
                    uint32_t w[4] = {route_halves(v[0][0], v[0][2], false), route_halves(v[0][0], v[0][2], true),
                                     route_halves(v[0][1], v[0][3], false), route_halves(v[0][1], v[0][3], true)};
                    route_transpose(w);
                    multiply(op[q], q % GROUPS, 0, make_uint4(w[0], w[1], w[2], w[3]));
                } else if constexpr (S == 2) {               // lane t's word r (indices 8t + 2r, + 1) to lane group r
                    route_transpose(v[0]);
                    route_transpose(v[1]);
#pragma unroll
                    for (int s = 0; s < 2; ++s)
                        multiply(op[q], q % GROUPS, s, make_uint4(route_halves(v[0][0], v[0][1], s), route_halves(v[0][2], v[0][3], s),
                                                                  route_halves(v[1][0], v[1][1], s), route_halves(v[1][2], v[1][3], s)));
                } else {                                     // indices 16t + 4r .. + 3 to lane group r, words [t][0], [t][1]
                    uint32_t w[8][2];
#pragma unroll
                    for (int h = 0; h < 4; ++h)
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            const auto y = __builtin_amdgcn_permlane16_swap(v[h][i], v[h][2 + i], false, false);
                            const auto z = __builtin_amdgcn_permlane32_swap(y[0], y[1], false, false);
                            w[2 * h][i] = z[0], w[2 * h + 1][i] = z[1];
                        }
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const int i = s >> 1;
                        multiply(op[q], q % GROUPS, s, make_uint4(route_halves(w[0][i], w[1][i], s & 1), route_halves(w[2][i], w[3][i], s & 1),
                                                                  route_halves(w[4][i], w[5][i], s & 1), route_halves(w[6][i], w[7][i], s & 1)));
                    }
                }
            }
        };
        for (; unit + (kMost - 1) * kWaves < whole; unit += kMost * kWaves) units(unit, std::integral_constant<int, kMost>{});
        if constexpr (kMost > 1)
            for (; unit < whole; unit += kWaves) units(unit, std::integral_constant<int, 1>{});
        const int left = d_r - whole * kRouteUnit;
        if (unit == whole && left > 0) {                     // what is left: zeros from d_r on
            const global_bytes rows = route_base(W_r + (uint32_t)whole * kRouteUnit * (uint32_t)E);
            const global_bytes xs = (global_bytes) reinterpret_cast<uint64_t>(x + (int64_t)whole * kRouteUnit);
#pragma unroll
            for (int g = 0; g < GROUPS; ++g) {
                Group op;
                route_end_words<MOST>(op.w, rows, 32 * S * g + S * r + set, left, E, w_col);
#pragma unroll
                for (int s = 0; s < S; ++s) multiply(op, g, s, route_end_x<S>(xs, 32 * S * g + S * r + s, left));
                __builtin_amdgcn_sched_barrier(0);           // (a group's loads at a time: registers)
            }
        }
    } else {
        for (; unit * kRouteUnit < d_r; unit += kWaves) {
            const int left = min(d_r - unit * kRouteUnit, kRouteUnit);
            const global_bytes rows = route_base(W_r + (int64_t)unit * kRouteUnit * E);
            const global_bytes xs = (global_bytes) reinterpret_cast<uint64_t>(x + (int64_t)unit * kRouteUnit);
#pragma unroll
            for (int step = 0; step < 4; ++step) {
                const int first = 32 * S * (step / S) + S * r + step % S;
                const uint4 xg = route_end_x<S>(xs, first, left);
#pragma unroll
                for (int et = 0; et < ET; ++et) {
                    const global_bytes column = rows + 2 * (uint32_t)min(16 * et + c, E - 1);
                    uint32_t v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        v[u] = route_end_element(column, first + 4 * S * (2 * u), left, E) |
                               route_end_element(column, first + 4 * S * (2 * u + 1), left, E) << 16;
                    chain[step % CH][et] = mfma_rows(make_uint4(v[0], v[1], v[2], v[3]), xg, chain[step % CH][et]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // joined as in the one-row form: a set's steps first, then the sets
#pragma unroll
    for (int et = 0; et < ET; ++et) {
        if constexpr (CH == 2) acc[et] = chain[0][et] + chain[1][et];
        else if constexpr (S == 2) acc[et] = (chain[0][et] + chain[2][et]) + (chain[1][et] + chain[3][et]);
        else acc[et] = (chain[0][et] + chain[1][et]) + (chain[2][et] + chain[3][et]);
    }
}

// Plus lane ^ 16's, plus lane ^ 32's value.
__device__ __forceinline__ float route_sum_rows(float v) {
    const auto o = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(o[0]) + __uint_as_float(o[1]);
}
__device__ __forceinline__ float route_sum_halves(float v) {
    const auto o = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(o[0]) + __uint_as_float(o[1]);
}

// Expert `lane`'s logit (lanes >= E: -inf; a NaN logit ranks last) from N partial sums, `pitch` floats apart, joined
// pairwise: 64 / MOST groups of lanes take a part each.  Any whole wavefront may call it.
template <int MOST, int N>
__device__ __forceinline__ float route_logit_joined(const float *sums, int pitch, float bias_of_lane, int E, int lane) {
    constexpr int kParts = kWave / MOST, kEach = N / kParts;
    static_assert(kEach >= 1 && kEach * kParts == N, "whole parts");
    float v[kEach];
#pragma unroll
    for (int i = 0; i < kEach; ++i) v[i] = sums[((lane / MOST) * kEach + i) * pitch + (lane & (MOST - 1))];
#pragma unroll
    for (int step = 1; step < kEach; step *= 2)
#pragma unroll
        for (int i = 0; i < kEach; i += 2 * step) v[i] += v[i + step];
    float sum = v[0];
    if constexpr (MOST <= 8) sum += lane_xor<3>(sum);
    if constexpr (MOST <= 16) sum = route_sum_rows(sum);
    if constexpr (MOST <= 32) sum = route_sum_halves(sum);
    sum += bias_of_lane;
    return lane < E ? (sum != sum ? -INFINITY : sum) : -INFINITY;
}

// The logits of the block's R routed rows (at most ROWS), with the block's barrier: in wave q, lane e, row q's of expert e.
template <int MOST, int ROWS>
struct RouteShared {
    __attribute__((aligned(16))) unsigned char x[(kRouteThreads / kWave) * 2 * kRouteUnit * route_few_units<MOST, ROWS>() * ROWS];
    float sums[ROWS][RouteTiles<MOST>::kSums][MOST];
};
template <int MOST, int ROWS>
__device__ __forceinline__ float route_logits_few(const bf16 *x, int R, int x_stride, const bf16 *W_r, int d_r, int E,
                                                  float bias_of_lane, RouteShared<MOST, ROWS> &sh) {
    const int wave = threadIdx.x >> 6;
    route_mfma_few<MOST, ROWS>(x, R, x_stride, W_r, d_r, E, sh.x, sh.sums);
    __syncthreads();
    if (wave >= R) return 0.0f;
    return route_logit_joined<MOST, RouteTiles<MOST>::kSums>(sh.sums[wave][0], MOST, bias_of_lane, E, threadIdx.x & (kWave - 1));
}
// One row, in the first wave, of any alignment.
template <int MOST>
__device__ __forceinline__ float route_logit_mfma(const bf16 *x, const bf16 *W_r, int d_r, int E, bool words,
                                                  float bias_of_lane, RouteShared<MOST, 1> &sh) {
    constexpr int kWaves = kRouteThreads / kWave, ET = RouteTiles<MOST>::kTiles;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    if (words) return route_logits_few<MOST, 1>(x, 1, 0, W_r, d_r, E, bias_of_lane, sh);
    f32x4_t acc[ET];
    route_mfma_rows<MOST, false>(x, W_r, d_r, E, acc);       // (every column is the one row)
    if ((lane & 15) == 0) {
#pragma unroll
        for (int et = 0; et < ET; ++et)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = 16 * et + 4 * (lane >> 4) + i;
                if (e < MOST) sh.sums[0][wave][e] = acc[et][i];
            }
    }
    __syncthreads();
    return wave == 0 ? route_logit_joined<MOST, kWaves>(sh.sums[0][0], MOST, bias_of_lane, E, lane) : 0.0f;
}

// (2) fp32, rows of W_r that are a power of two (1 .. 16) of aligned 16-byte chunks.  Thread t
// streams chunks t, t+1024, ... (a wave reads 1 KiB of consecutive bytes per load; all loads of
// a thread are independent); its chunk-in-row index never changes, so it accumulates the same 4
// experts throughout.  Lanes with equal chunk index are summed by xor-shuffles; the 16 waves'
// sums go to `red`.
__device__ __forceinline__ void route_logits_vec(const float *xr, const float *W_r, int d_r, int cpr, float (*red)[64]) {
    constexpr int EPL = 4;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = tid >> 6;
    const int cir = tid & (cpr - 1);
    const int cshift = ilog2(cpr);
    const int total = d_r * cpr;

    float acc[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) acc[i] = 0.0f;
    // batches of 8, then 4, then single chunks: all loads of a batch are in flight together,
    // the multiply-adds stay in ascending chunk order whatever the batching
    auto batch = [&](int c, auto nload) {
        constexpr int NB = decltype(nload)::value;
        uint4 w[NB];
        float xj[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            w[u] = load16(W_r + (int64_t)(c + u * kRouteThreads) * EPL);
            xj[u] = xr[(c + u * kRouteThreads) >> cshift];
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            float wf[EPL];
            Pack16<float>::widen(w[u], wf);
#pragma unroll
            for (int i = 0; i < EPL; ++i) acc[i] = fmaf(xj[u], wf[i], acc[i]);
        }
    };
    int c = tid;
    for (; c + 7 * kRouteThreads < total; c += 8 * kRouteThreads) batch(c, std::integral_constant<int, 8>{});
    for (; c + 3 * kRouteThreads < total; c += 4 * kRouteThreads) batch(c, std::integral_constant<int, 4>{});
    for (; c < total; c += kRouteThreads) batch(c, std::integral_constant<int, 1>{});
    // lanes with the same chunk-in-row index: xor butterfly over the lane bits from log2(cpr) up
    auto join = [&](auto bit) {
        constexpr int BIT = decltype(bit)::value;
        if ((1 << BIT) >= cpr) {
#pragma unroll
            for (int i = 0; i < EPL; ++i) acc[i] += lane_xor<BIT>(acc[i]);
        }
    };
    join(std::integral_constant<int, 0>{});
    join(std::integral_constant<int, 1>{});
    join(std::integral_constant<int, 2>{});
    join(std::integral_constant<int, 3>{});
    join(std::integral_constant<int, 4>{});
    join(std::integral_constant<int, 5>{});
    if (lane < cpr) {
#pragma unroll
        for (int i = 0; i < EPL; ++i) red[wave][cir * EPL + i] = acc[i];
    }
    __syncthreads();
}

// (3) fp32, any other E and any alignment, few elements: threads as (row slice, expert), an element of W_r each, and a
// pairwise tree over the slices.  A thread has less to set up than in the next form, which pays from 6 to 8
// elements a thread on, and sooner where its chunks are of one row of W_r (E a multiple of 4); with up to 3 experts a
// chunk of that form spans rows, and it never pays.  This form against the next, us, 1 row, 500 and 4096 rows: 600 values x 6
// experts 3.38, 4.19, 8.7 and 3.60, 4.93, 10.3, 768 x 6 3.59, 4.39, 9.7 and 3.36, 4.81, 10.1; 512 x 13 3.6, 4.5, 10.3 and
// 3.7, 5.0, 11.2; 512 x 12 3.6, 4.5, 10.3 and 3.3, 4.6, 9.9; 3 experts, 1 row x 8192 6.2 and 6.7, 4096 x 4096 22 and 44.
// (Row counts do not enter: a row's bits are the same whatever their number.)
inline bool route_single_ok(int d_r, int E) {
    int EP = 1;
    while (EP < E) EP <<= 1;
    return E <= 3 || (int64_t)d_r * EP <= (E % 4 == 0 ? 4096 : EP <= 8 ? 6000 : 8192);
}
// The logits of R rows: row q's are the first E floats of red + 1024 q, of R * 1024.
template <int R>
__device__ __forceinline__ void route_logits_single(const float *const (&xr)[R], const float *W_r, int d_r, int E, int EP, float *red) {
    const int tid = threadIdx.x, e = tid & (EP - 1), slice = tid / EP, slices = kRouteThreads / EP;
    float acc[R];
#pragma unroll
    for (int q = 0; q < R; ++q) acc[q] = 0.0f;
    if (e < E) {
        for (int j = slice; j < d_r; j += slices) {
            const float w = W_r[(int64_t)j * E + e];
#pragma unroll
            for (int q = 0; q < R; ++q) acc[q] = fmaf(xr[q][j], w, acc[q]);
        }
    }
#pragma unroll
    for (int q = 0; q < R; ++q) red[q * kRouteThreads + tid] = acc[q];
    __syncthreads();
    for (int half = slices >> 1; half >= 1; half >>= 1) {
        if (slice < half)
#pragma unroll
            for (int q = 0; q < R; ++q) red[q * kRouteThreads + tid] += red[q * kRouteThreads + tid + half * EP];
        __syncthreads();
    }
}
// Expert `lane`'s logit of a row (experts >= E: -inf; a NaN logit ranks last).
__device__ __forceinline__ float route_logit_single_of_lane(const float *red, float bias_of_lane, int E, int lane) {
    if (lane >= E) return -INFINITY;
    const float v = red[lane] + bias_of_lane;
    return v != v ? -INFINITY : v;
}

// (4) fp32, the rest: W_r as one flat array, cut into chunks of 4 elements.
// A row of E elements repeats its place in the chunks every E / gcd(E, 4) of them, so with the
// block's threads cut down to a multiple of that, T, thread t's chunks t, t + T, ... hold the same
// 4 experts each, and it sums them in registers; the 4 T sums (element g belongs to expert g % E)
// meet in LDS.
// Several rows: route_flat_rows_kernel, R rows to a thread, and as many sets of T threads as a block holds.
constexpr int kFlatFloats = 4 * kRouteThreads;
// T: as many threads as have about 8 chunks each - the sums that meet in LDS are few then, and 8 loads
// are one trip (the same for every number of rows, like all that decides the order of a sum).
inline int route_flat_threads(int d_r, int E) {
    const int period = E / (E % 4 == 0 ? 4 : E % 2 == 0 ? 2 : 1);
    const int64_t eighth = (int64_t)d_r * E / 32;
    const int T = eighth < kRouteThreads ? (int)eighth : kRouteThreads;
    return T < period ? period : T / period * period;
}
// XJ: values of x that a chunk meets - 1 (E a multiple of 4) or 2 (at most two rows of W_r: E > 4).
template <int R, int XJ>
__device__ __forceinline__ void route_flat_sums(int tid, const float *const (&xr)[R], const float *W_r, int d_r, int E, int T,
                                                bool aligned, float (&acc)[R][4]) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[r][i] = 0.0f;
    if (tid >= T) return;
    int j[XJ];                              // rows of W_r (past the last one: the last)
    j[0] = 4 * tid / E;
    const int second = (j[0] + 1) * E - 4 * tid;              // XJ == 2: the chunk's first element of the second row
    if (XJ == 2) j[XJ - 1] = j[0] + 1;
    const int dj = 4 * T / E;               // rows from one chunk of the thread to the next
    const int64_t whole = (int64_t)d_r * E / 4;
    auto batch = [&](int64_t c, auto count) {
        constexpr int N = decltype(count)::value;
        float w[N][4], x[N][R][XJ];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const float *at = W_r + (c + u * T) * 4;
            if (aligned) {
                Pack16<float>::widen(load16(at), w[u]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) w[u][i] = at[i];
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int i = 0; i < XJ; ++i) x[u][r][i] = xr[r][i == 1 ? min(j[i] + u * dj, d_r - 1) : j[0] + u * dj];
        }
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float xi = XJ == 1 || i < second ? x[u][r][0] : x[u][r][XJ - 1];
                    acc[r][i] = fmaf(xi, w[u][i], acc[r][i]);
                }
#pragma unroll
        for (int i = 0; i < XJ; ++i) j[i] += N * dj;
    };
    constexpr int MOST = R > 1 ? 2 : 8;
    int64_t c = tid;
    for (; c + (MOST - 1) * T < whole; c += MOST * T) batch(c, std::integral_constant<int, MOST>{});
    for (; c < whole; c += T) batch(c, std::integral_constant<int, 1>{});
    if (XJ > 1 && c == whole) {              // the elements left over, fewer than a chunk
        const int left = (int)((int64_t)d_r * E & 3);
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (i < left)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    acc[r][i] = fmaf(xr[r][i < second ? j[0] : j[XJ - 1]], W_r[whole * 4 + i], acc[r][i]);
    }
}
template <int R>
__device__ __forceinline__ void route_flat_sums(int tid, const float *const (&xr)[R], const float *W_r, int d_r, int E, int T,
                                                bool aligned, float (&acc)[R][4]) {
    if (E % 4 == 0) route_flat_sums<R, 1>(tid, xr, W_r, d_r, E, T, aligned, acc);
    else route_flat_sums<R, 2>(tid, xr, W_r, d_r, E, T, aligned, acc);
}
// A wave's share of the 4 T sums of expert lane % EP: every (1024 / EP)-th from wave * (64 / EP) + lane / EP on.
__device__ __forceinline__ float route_flat_share(const float *buf, int E, int EP, int T, int wave, int lane) {
    const int e = lane & (EP - 1), sums = 4 * T / E;
    float s = 0.0f;
    if (e < E)
        for (int m = wave * (kWave / EP) + lane / EP; m < sums; m += kRouteThreads / EP) s += buf[m * E + e];
    if (EP <= 4) s += lane_xor<2>(s);
    if (EP <= 8) s += lane_xor<3>(s);
    if (EP <= 16) s = route_sum_rows(s);
    if (EP <= 32) s = route_sum_halves(s);
    return s;
}
inline __host__ __device__ int route_flat_pow2(int E) {
    int EP = 1;
    while (EP < E) EP <<= 1;
    return EP;
}
// buf: 4096 floats
__device__ __forceinline__ void route_logits_flat(const float *xr, const float *W_r, int d_r, int E, int T, bool aligned,
                                                  float *buf, float (*red)[64]) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    float acc[1][4];
    route_flat_sums<1>(tid, {xr}, W_r, d_r, E, T, aligned, acc);
    if (tid < T) *reinterpret_cast<float4 *>(buf + 4 * tid) = make_float4(acc[0][0], acc[0][1], acc[0][2], acc[0][3]);
    __syncthreads();
    const int EP = route_flat_pow2(E);
    const float share = route_flat_share(buf, E, EP, T, wave, lane);
    if (lane < EP) red[wave][lane] = share;
    __syncthreads();
}

// The additive term of expert `lane` (0 without a bias or past the last expert).  Callers read
// it before the weights: it depends on nothing, and a load issued after the block barrier
// would put a whole trip to memory between the logits and the selection.
__device__ __forceinline__ float route_bias_of_lane(const float *bias, int E, int lane) {
    return (bias != nullptr && lane < E) ? bias[lane] : 0.0f;
}

template <int N>
__device__ __forceinline__ float route_pairwise(float (&v)[N]) {
#pragma unroll
    for (int step = 1; step < N; step *= 2)
#pragma unroll
        for (int i = 0; i < N; i += 2 * step) v[i] += v[i + step];
    return v[0];
}

// Expert `lane`'s logit from the per-wave sums, `pitch` floats apart (waves joined pairwise;
// experts >= E hold -inf; a NaN logit is replaced by -inf).  Any wavefront may call it after the barrier.
__device__ __forceinline__ float route_logit_of_lane(const float *red, int pitch, float bias_of_lane, int E,
                                                     int lane) {
    constexpr int kWaves = kRouteThreads / kWave;
    float v = -INFINITY;
    if (lane < E) {
        float sums[kWaves];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sums[w] = red[w * pitch + lane];
        v = route_pairwise(sums);
        v += bias_of_lane;
        if (v != v) v = -INFINITY;
    }
    return v;
}

// True when route_logits_vec applies: fp32 rows of W_r that are a power-of-two number of aligned
// 16-byte chunks.
inline bool route_vec_ok(const void *W_r, int E, int *cpr) {
    *cpr = E / 4;
    return E % 4 == 0 && (*cpr & (*cpr - 1)) == 0 && reinterpret_cast<uintptr_t>(W_r) % 16 == 0;
}

}  // namespace pikv
