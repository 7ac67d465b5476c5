// recur.h -- shared pieces of the chunked vector recursions (recur_max.hip, recur_log.hip):
// tile layouts, row-broadcasts and the loads of an edge's potentials.
//
// A recursion walks the edges of a chain with one vector of C entries: C^2 work per edge
// instead of the C^3 of a matrix product.  To use the whole chip, a chain is cut into chunks
// of S edges; every chunk is walked at once, the first from its true start vector, the others
// from a guess.  Products of such matrices forget their start: after some edges the vector
// walked from the guess equals, up to one common factor (an offset in the max semiring), the
// vector walked from the true start, and from there on everything that follows is the same.
// So in further rounds a chunk is walked again from its predecessor's end vector, but only
// until its vector agrees with the stored one.  A round that reaches its chunk's end without
// agreeing changes the end vector, and the next chunk is walked again in the next round.
// After kRecRounds such rounds what is still pending is walked in order, or, where that is more than
// a few chunks and the tree is faster, left to it (Plan::gate), as the tree needs no such property.
// A sequence of one chunk is exact at once.
#pragma once
#include <hip/hip_runtime.h>

#include "device.h"
#include "internal.h"

namespace tsc {

// Layout of one edge's C x C potentials over a workgroup of kNW waves.  A row takes kLPR lanes
// (kVec consecutive columns each, kCP such blocks per lane), so a wave holds kG = 64 / kLPR
// rows side by side; each of these row groups walks kRG consecutive rows, group g of the
// workgroup (g = wave * kG + group in the wave) rows g * kRG .. g * kRG + kRG - 1.  A wave owns
// kRPW = kG * kRG <= 16 consecutive rows, and as columns the same 16 labels: it merges the
// groups' partial results of those columns itself, so a step needs one barrier.
template <int VEC, int LPR, int CP, int RG, int NW>
struct RecCfg {
    static constexpr int kVec = VEC, kLPR = LPR, kCP = CP, kRG = RG, kNW = NW;
    static constexpr int kG = 64 / LPR, kNG = NW * kG, kRPW = kG * RG, kT = NW * 64;
    static constexpr int kCols = LPR * VEC * CP;   // columns the lanes cover (>= C)
    static constexpr int kCB = CP * VEC;           // columns per lane
    // whether log-semiring walks can take exponentials formed beforehand (recur_log.hip)
    static constexpr bool kPre = RG * CP * VEC >= 12 && NW >= 8;
    // edges in flight: up to 64 registers' worth in the layouts of fewer than 16 waves.  The max
    // semiring's walks also have room for two of the 16-wave layouts' smaller tiles (odd label
    // counts from 65 to 128; Viterbi of B = 32, N = 500, C = 75: 277 us with one, 217 with two;
    // B = 7, N = 777, C = 101: 356 and 293; B = 4, N = 8192, C = 127: 664 and 630); the log
    // semiring's would spill registers for 2 to 4%.
    static constexpr int kDepth = NW == 16 ? 1 : RG * CP * VEC <= 16 ? 4 : 2;
    static constexpr int kDepthMax = NW == 16 && RG * CP * VEC <= 16 ? 2 : kDepth;
    static_assert(kRPW <= 16 && kNG % 4 == 0 && kNW <= 16, "a wave's labels fit 16 lanes");
};

// A value that every lane holds, in a scalar register
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ bool uniform(bool x) { return __builtin_amdgcn_readfirstlane((int)x) != 0; }
__device__ __forceinline__ const float* uniform(const float* p) {
    const uint64_t u = (uint64_t)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)u);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(u >> 32));
    return (const float*)(((uint64_t)hi << 32) | lo);
}

// The value of lane `r` of each row of 16 lanes, in every lane of that row (r is a constant
// once the caller's loop is unrolled)
__device__ __forceinline__ int row_bcast_i(int x, int r) {
#define TSC_BC(n) case n: return __builtin_amdgcn_update_dpp(0, x, 0x150 + n, 0xF, 0xF, false);
    switch (r) {
        TSC_BC(0) TSC_BC(1) TSC_BC(2) TSC_BC(3) TSC_BC(4) TSC_BC(5) TSC_BC(6) TSC_BC(7)
        TSC_BC(8) TSC_BC(9) TSC_BC(10) TSC_BC(11) TSC_BC(12) TSC_BC(13) TSC_BC(14)
        default: return __builtin_amdgcn_update_dpp(0, x, 0x15F, 0xF, 0xF, false);
    }
#undef TSC_BC
}
__device__ __forceinline__ float row_bcast(float x, int r) {
    return __int_as_float(row_bcast_i(__float_as_int(x), r));
}
__device__ __forceinline__ double row_bcast(double x, int r) {
    const unsigned long long u = __double_as_longlong(x);
    const unsigned lo = (unsigned)row_bcast_i((int)(unsigned)u, r);
    const unsigned hi = (unsigned)row_bcast_i((int)(unsigned)(u >> 32), r);
    return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}

// The values of lanes (l & ~16) and (l | 16), and of lanes (l & 31) and (l | 32), in every lane
struct Pair { unsigned a, b; };
__device__ __forceinline__ Pair pair16(unsigned x) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return {r[0], r[1]};
}
__device__ __forceinline__ Pair pair32(unsigned x) {
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return {r[0], r[1]};
}
struct PairD { double a, b; };
__device__ __forceinline__ double join_d(unsigned lo, unsigned hi) {
    return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ PairD pair16_d(double x) {
    const unsigned long long u = __double_as_longlong(x);
    const Pair l = pair16((unsigned)u), h = pair16((unsigned)(u >> 32));
    return {join_d(l.a, h.a), join_d(l.b, h.b)};
}
__device__ __forceinline__ PairD pair32_d(double x) {
    const unsigned long long u = __double_as_longlong(x);
    const Pair l = pair32((unsigned)u), h = pair32((unsigned)(u >> 32));
    return {join_d(l.a, h.a), join_d(l.b, h.b)};
}

// Maximum over each row of 16 lanes, in every lane of the row
__device__ __forceinline__ double dpp_d(double x, int ctrl) {
    const unsigned long long u = __double_as_longlong(x);
    const float lo = dpp_f(__int_as_float((int)(unsigned)u), ctrl);
    const float hi = dpp_f(__int_as_float((int)(unsigned)(u >> 32)), ctrl);
    return join_d(__float_as_uint(lo), __float_as_uint(hi));
}
__device__ __forceinline__ double row_max_d(double x) {
    x = fmax(x, dpp_d(x, 0xB1));
    x = fmax(x, dpp_d(x, 0x4E));
    x = fmax(x, dpp_d(x, 0x141));
    return fmax(x, dpp_d(x, 0x140));
}
__device__ __forceinline__ double row_sum_d(double x) {   // (the sum over each row of 16 lanes)
    x += dpp_d(x, 0xB1);
    x += dpp_d(x, 0x4E);
    x += dpp_d(x, 0x141);
    return x + dpp_d(x, 0x140);
}
__device__ __forceinline__ float row_max(float x) {
    x = fmaxf(x, dpp_f(x, 0xB1));
    x = fmaxf(x, dpp_f(x, 0x4E));
    x = fmaxf(x, dpp_f(x, 0x141));
    return fmaxf(x, dpp_f(x, 0x140));
}

// The range of the linear log-semiring walks: |l| <= 24 gives E within 2^+-34.7; with 256 labels a step grows
// the largest entry by less than 2^43, and vectors are scaled by the exponent of the one
// before, so entries that are not 0 lie within [kRecLow 2^-43, 2^43] of what a step reads and
// its smallest product stays above 2^-46 - 43 - 35 = 2^-124.
constexpr float kRecLow = 0x1p-46f;
constexpr unsigned kRecPotBits = 0x84800000u;   // fin_bits(24)

// Order-preserving magnitude of a finite x; 0 for -inf (one shift-add)
__device__ __forceinline__ unsigned fin_bits(float x) { return (__float_as_uint(x) << 1) + 0x01000000u; }

// exp(l) to about one rounding for any l of the range: exp2 of the rounded product, corrected
// by what the rounding dropped.  (-inf is read as a number large enough to give exactly 0.)
__device__ __forceinline__ float edge_exp(float l) {
    l = fmaxf(l, -3e37f);
    const float x = l * 1.4426950408889634f;
    const float e = __builtin_amdgcn_exp2f(x);
    return fmaf(e, fmaf(-x, 0.6931471805599453f, l), e);
}

// floor(log2 x) of a positive normal x; 0 for 0
__device__ __forceinline__ int exponent_of(float x) {
    return x > 0.f ? (int)(__float_as_uint(x) >> 23) - 127 : 0;
}

// Per-lane offsets of a tile's loads: row r of the lane's group, column block cp.  Rows and
// columns past C read whatever the descriptor's bound leaves (a later row's entries, or 0
// past the edge): callers give such rows no weight and never use such columns.
template <class F>
struct Tile {
    float x[F::kRG][F::kCB];
};
template <class F>
__device__ __forceinline__ unsigned tile_offset(int C) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int g = w * F::kG + lane / F::kLPR;
    return 4u * (unsigned)(g * F::kRG * C + (lane % F::kLPR) * F::kVec);
}
template <class F>
__device__ __forceinline__ void tile_load_row(float (&x)[F::kCB], __amdgpu_buffer_rsrc_t rs,
                                              unsigned voff, int r, int C) {
#pragma unroll
    for (int cp = 0; cp < F::kCP; ++cp) {
        const int soff = 4 * (r * C + cp * F::kLPR * F::kVec);
        if constexpr (F::kVec == 4) {
            const float4 v = buffer_load4(rs, voff, soff);
            x[cp * 4] = v.x; x[cp * 4 + 1] = v.y; x[cp * 4 + 2] = v.z; x[cp * 4 + 3] = v.w;
        } else {
            x[cp] = buffer_load1(rs, voff, soff);
        }
    }
}

// Chunk k of sequence b of a recursion: its edges [s, e), and the versions of end vectors.
// Round r's walks write version r; chg[r][b][k] (r >= 1) says that they did.
__device__ __forceinline__ int latest_version(const int32_t* chg, int64_t nbk, int64_t bk, int r) {
    int v = 0;   // (all at once: a walk usually has changed nothing since version 0)
#pragma unroll
    for (int q = 1; q <= kRecRounds + 1; ++q)
        if (q <= r && chg[(size_t)(q - 1) * nbk + bk]) v = q;
    return v;
}

// Calls fn(cfg) with the layout for C labels: 16-byte loads when rows are 16-byte aligned
// (C a multiple of 4), one entry per load otherwise.  Sixteen row groups (eight or four for the
// narrow one-entry layouts) give each wave up to 16 rows and each lane 4 to 64 entries; the
// layouts between the powers of two (6 and 12 rows per group) keep idle rows below a third.
// Up to 16 labels one wave walks alone: its step has no other wave to wait for (marginals of B
// = 21, N = 525, C = 9: 73 us with four waves, 50 with one; B = 64, N = 2000, C = 16: 259 with
// two, 162 with one).  From 17 to 32 one or two waves with longer rows are slower (B = 16, N =
// 2000, C = 32: 137 against 123).
template <class Fn>
hipError_t with_rec_cfg(int64_t C, Fn&& fn) {
    if (C <= 16) return fn(RecCfg<1, 16, 1, 4, 1>{});
    if (C % 4 == 0) {
        if (C <= 32) return fn(RecCfg<4, 8, 1, 2, 2>{});
        if (C <= 64) return fn(RecCfg<4, 16, 1, 4, 4>{});
        if (C <= 96) return fn(RecCfg<4, 32, 1, 6, 8>{});
        if (C <= 128) return fn(RecCfg<4, 32, 1, 8, 8>{});
        if (C <= 192) return fn(RecCfg<4, 64, 1, 12, 16>{});
        return fn(RecCfg<4, 64, 1, 16, 16>{});
    }
    if (C <= 32) return fn(RecCfg<1, 32, 1, 4, 4>{});
    if (C <= 64) return fn(RecCfg<1, 64, 1, 8, 8>{});
    if (C <= 96) return fn(RecCfg<1, 64, 2, 6, 16>{});
    if (C <= 128) return fn(RecCfg<1, 64, 2, 8, 16>{});
    if (C <= 192) return fn(RecCfg<1, 64, 3, 12, 16>{});
    return fn(RecCfg<1, 64, 4, 16, 16>{});
}

}  // namespace tsc
