// Device helpers for kernels in which one workgroup holds one vocabulary row (float4 x ITEMS
// per thread, VT threads).  Shared by the verification and the draft-sampling kernels: the wavefront reductions, sums
// and scans.  The sampler's alone: the row load, the totals by pieces and the inverse-CDF search among them, with a row in order
// across the workgroup; verification has a load that deals a row to the wavefronts in consecutive shares, and searches by the
// totals of the wavefronts.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "mcsd.h"

namespace mcsd {
namespace vocab {

// Wavefront reductions on the DPP cross-lane paths (no LDS round trip).  The result is
// complete in lane 63 only: quad swaps, half-row and row mirrors give every lane its row's
// total, then row_bcast15 / row_bcast31 fold the four rows of 16 lanes into the last one.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_f(float old, float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_d(double old, double v)
{
    const long long o = __double_as_longlong(old), x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp((int)o, (int)x, CTRL, ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(x >> 32), CTRL, ROW_MASK, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

constexpr int DPP_QUAD_1032 = 0xB1, DPP_QUAD_2301 = 0x4E, DPP_ROW_HALF_MIRROR = 0x141, DPP_ROW_MIRROR = 0x140,
              DPP_ROW_BCAST15 = 0x142, DPP_ROW_BCAST31 = 0x143,
              DPP_ROW_SHR1 = 0x111, DPP_ROW_SHR2 = 0x112, DPP_ROW_SHR4 = 0x114, DPP_ROW_SHR8 = 0x118;

__device__ __forceinline__ float wave_max(float v)      // valid in lane 63
{
    v = fmaxf(v, dpp_f<DPP_QUAD_1032, 0xf>(v, v));
    v = fmaxf(v, dpp_f<DPP_QUAD_2301, 0xf>(v, v));
    v = fmaxf(v, dpp_f<DPP_ROW_HALF_MIRROR, 0xf>(v, v));
    v = fmaxf(v, dpp_f<DPP_ROW_MIRROR, 0xf>(v, v));
    v = fmaxf(v, dpp_f<DPP_ROW_BCAST15, 0xa>(v, v));
    v = fmaxf(v, dpp_f<DPP_ROW_BCAST31, 0xc>(v, v));
    return v;
}

__device__ __forceinline__ int wave_min(int v)           // valid in lane 63
{
    v = min(v, __builtin_amdgcn_update_dpp(v, v, DPP_QUAD_1032, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, DPP_QUAD_2301, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, DPP_ROW_HALF_MIRROR, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, DPP_ROW_MIRROR, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, DPP_ROW_BCAST15, 0xa, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(v, v, DPP_ROW_BCAST31, 0xc, 0xf, false));
    return v;
}

// Largest value of the wavefront and the lowest index among the lanes that hold it, in every
// lane: two DPP reductions and two lane reads instead of six rounds of cross-lane shuffles.
__device__ __forceinline__ void wave_argmax(float &bv, int &bi)
{
    const float m = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_max(bv)), 63));
    const int i = wave_min(bv == m ? bi : 0x7fffffff);
    bv = m;
    bi = __builtin_amdgcn_readlane(i, 63);
}

__device__ __forceinline__ double wave_sum(double v)    // valid in lane 63
{
    v += dpp_d<DPP_QUAD_1032, 0xf>(0.0, v);
    v += dpp_d<DPP_QUAD_2301, 0xf>(0.0, v);
    v += dpp_d<DPP_ROW_HALF_MIRROR, 0xf>(0.0, v);
    v += dpp_d<DPP_ROW_MIRROR, 0xf>(0.0, v);
    v += dpp_d<DPP_ROW_BCAST15, 0xa>(0.0, v);
    v += dpp_d<DPP_ROW_BCAST31, 0xc>(0.0, v);
    return v;
}

// The same sum in every lane.  The last two steps exchange whole rows of 16 lanes and the two halves of the
// wavefront (v_permlane16_swap, v_permlane32_swap on two copies leave one side in the first, the other in
// the second): one instruction per word, and both partners add the same two numbers.
__device__ __forceinline__ double add_rows(double v)
{
    const long long x = __double_as_longlong(v);
    const unsigned lo = (unsigned)x, hi = (unsigned)(x >> 32);
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false), h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __longlong_as_double(((long long)h[0] << 32) | l[0]) + __longlong_as_double(((long long)h[1] << 32) | l[1]);
}

__device__ __forceinline__ double add_halves(double v)
{
    const long long x = __double_as_longlong(v);
    const unsigned lo = (unsigned)x, hi = (unsigned)(x >> 32);
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false), h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __longlong_as_double(((long long)h[0] << 32) | l[0]) + __longlong_as_double(((long long)h[1] << 32) | l[1]);
}

template <int CTRL>
__device__ __forceinline__ double mov_dpp_d(double v)    // (every lane has a source)
{
    const long long x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)x, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(x >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ double wave_sum_all(double v)
{
    v += mov_dpp_d<DPP_QUAD_1032>(v);
    v += mov_dpp_d<DPP_QUAD_2301>(v);
    v += mov_dpp_d<DPP_ROW_HALF_MIRROR>(v);
    v += mov_dpp_d<DPP_ROW_MIRROR>(v);
    return add_halves(add_rows(v));
}

// Inclusive running sum over the lanes of the wavefront: shifts inside the rows of 16 lanes
// (a lane without a source adds zero), then the totals of the rows before it.
__device__ __forceinline__ double wave_scan_inclusive(double v)
{
    v += dpp_d<DPP_ROW_SHR1, 0xf>(0.0, v);
    v += dpp_d<DPP_ROW_SHR2, 0xf>(0.0, v);
    v += dpp_d<DPP_ROW_SHR4, 0xf>(0.0, v);
    v += dpp_d<DPP_ROW_SHR8, 0xf>(0.0, v);
    v += dpp_d<DPP_ROW_BCAST15, 0xa>(0.0, v);
    v += dpp_d<DPP_ROW_BCAST31, 0xc>(0.0, v);
    return v;
}

// ITEMS values per lane -> for every row of 16 lanes, the 16-lane total of each of the ITEMS
// values, spread over the lanes of that row: lane l ends up with the total of value number
// `which`.  Each of the first log2(ITEMS) steps halves the values a lane carries: the partner
// (whose lane number differs in the step's bit) gets the half this lane gives up, and this lane
// adds the partner's copy of the half it keeps.  15 exchanges for 16 values instead of 16 x 4.
template <int ITEMS>
__device__ __forceinline__ double row_totals_scattered(double (&x)[ITEMS], int lane, int &which)
{
    static_assert(ITEMS == 1 || ITEMS == 2 || ITEMS == 4 || ITEMS == 8 || ITEMS == 16, "power of two up to 16");
    which = 0;
    auto step = [&](auto ctrl_c, auto n_c, int bit) __attribute__((always_inline)) {
        constexpr int CTRL = decltype(ctrl_c)::value;
        constexpr int N = decltype(n_c)::value;          // values carried before this step
        if constexpr (N > 1) {
            const bool keep_hi = (lane >> bit) & 1;
#pragma unroll
            for (int j = 0; j < N / 2; ++j) {
                const double mine = keep_hi ? x[j + N / 2] : x[j];
                const double give = keep_hi ? x[j] : x[j + N / 2];
                x[j] = mine + mov_dpp_d<CTRL>(give);
            }
            if (keep_hi) which += N / 2;
        } else {
            x[0] += mov_dpp_d<CTRL>(x[0]);
        }
    };
    // Widest exchange first: the row mirror (lane i <-> 15 - i) flips bit 3, and every later
    // exchange (mirror inside 8 lanes, lanes 2 apart, neighbours) leaves the bits of the earlier
    // steps alone, so the two partners of a step always carry the same subset of the values.
    step(std::integral_constant<int, DPP_ROW_MIRROR>(), std::integral_constant<int, ITEMS>(), 3);
    step(std::integral_constant<int, DPP_ROW_HALF_MIRROR>(), std::integral_constant<int, (ITEMS > 1 ? ITEMS / 2 : 1)>(), 2);
    step(std::integral_constant<int, DPP_QUAD_2301>(), std::integral_constant<int, (ITEMS > 2 ? ITEMS / 4 : 1)>(), 1);
    step(std::integral_constant<int, DPP_QUAD_1032>(), std::integral_constant<int, (ITEMS > 4 ? ITEMS / 8 : 1)>(), 0);
    return x[0];
}

// Sum of the four lanes of a float4, exact in fp64: the normalisers A and Z_q enter the accept
// ratios divided by the rejection probabilities, so their rounding must stay far below 1e-6.
__device__ __forceinline__ double sum4(const float4 &v)
{
    return ((double)v.x + (double)v.y) + ((double)v.z + (double)v.w);
}

// A logit row is read through a buffer resource whose extent is the row: the address of float4
// number t + VT i is one per-thread offset plus a scalar, reads past the end return zero instead
// of leaving the array, and no per-load address registers or bounds branches are needed.
// Elements past V are then set to -inf by settle_pieces().
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_resource(const float *row, int V)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(row), 0, V * 4, 0x00020000);
}

// max(a, b, c) as the one hardware instruction.  fmaxf() has to quiet signalling NaNs, and for
// values the compiler knows nothing about (loaded from memory) it does so with an extra
// v_max_f32 x, x per operand: three instructions per element instead of half of one.  The
// instruction itself returns the largest non-NaN operand, which is what the row maximum wants.
__device__ __forceinline__ float max3_raw(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

template <int ITEMS>
__device__ __forceinline__ float row_max(const float4 (&r)[ITEMS])
{
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) m = max3_raw(max3_raw(m, r[i].x, r[i].y), r[i].z, r[i].w);
    return m;
}

// ------------------------------------------------------------------ rows in pieces
// A piece is what one wavefront holds of one item:
// 256 consecutive tokens; piece number j = item * waves + wave is their order in the row.  Every
// wavefront keeps all piece totals itself (PPL = pieces per lane, in order), so that it finds the
// piece of a crossing with one scan over its lanes; the wavefront that owns that piece then finds
// the token with a second scan and publishes it: one workgroup barrier per search.

// Loads of a logit row, four tokens per thread and item, -inf past V.  The first FULL items lie
// inside every row of this configuration.  A row whose length is no multiple of four starts at any
// 4-byte address, which 128-bit buffer loads allow; its last tokens (fewer than four) come by
// single loads, so that no load straddles the end of the resource.
template <int ITEMS, int VT, int FULL, bool ALIGNED>
__device__ __forceinline__ void load_pieces(const float *row, int V, int tid, float4 (&r)[ITEMS])
{
    constexpr int NT = 2;                   // non-temporal: a logit row is read once
    const float ninf = -INFINITY;
    const int V4 = V & ~3;
    const __amdgpu_buffer_rsrc_t rs = row_resource(row, ALIGNED ? V : V4);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, tid * 16, i * (VT * 16), NT);
        r[i] = make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3]));
    }
    float4 tail;
    if (!ALIGNED) {
        const __amdgpu_buffer_rsrc_t rt = row_resource(row, V);
        tail.x = (V4 < V) ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rt, 0, V4 * 4, NT)) : ninf;
        tail.y = (V4 + 1 < V) ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rt, 4, V4 * 4, NT)) : ninf;
        tail.z = (V4 + 2 < V) ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rt, 8, V4 * 4, NT)) : ninf;
    }
#pragma unroll
    for (int i = FULL; i < ITEMS; ++i) {
        if (4 * VT * (i + 1) > V4) {        // uniform
            const int e = 4 * (tid + VT * i);
            const bool past = e > V4 || (ALIGNED && e == V4), at = !ALIGNED && e == V4;
            r[i] = make_float4(past ? ninf : (at ? tail.x : r[i].x), past ? ninf : (at ? tail.y : r[i].y),
                               past ? ninf : (at ? tail.z : r[i].z), past ? ninf : (at ? ninf : r[i].w));
        }
    }
}

template <int ITEMS, int VT>
struct Pieces {
    static constexpr int NW = VT / 64, NP = ITEMS * NW, PPL = NP <= 64 ? 1 : NP / 64;
    double tot[PPL], least[PPL];            // totals of pieces lane * PPL ...; for remove()

    // s_piece holds 4 NP doubles: the totals per row of 16 lanes
    static __device__ __forceinline__ void store4(const double (&x)[4], int i0, int lane, int wave, double *s_piece)
    {
        double y[4] = {x[0], x[1], x[2], x[3]};
        int which;
        const double w = row_totals_scattered<4>(y, lane, which);
        s_piece[((i0 + which) * NW + wave) * 4 + (lane >> 4)] = w;
    }
    static __device__ __forceinline__ void store(const float4 (&a)[ITEMS], int lane, int wave, double *s_piece)
    {
#pragma unroll
        for (int i0 = 0; i0 < ITEMS; i0 += 4) {
            double x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = (i0 + i < ITEMS) ? sum4(a[i0 + i < ITEMS ? i0 + i : 0]) : 0.0;
            store4(x, i0, lane, wave, s_piece);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __device__ __forceinline__ void read(const double *s_piece, int lane)
    {
#pragma unroll
        for (int q = 0; q < PPL; ++q) {
            const int j = lane * PPL + q;
            const double *s = s_piece + 4 * (j < NP ? j : 0);
            const double t = (s[0] + s[1]) + (s[2] + s[3]);
            tot[q] = j < NP ? t : 0.0;
            least[q] = tot[q] * 0x1p-20;
        }
    }
    __device__ __forceinline__ double scan() const      // inclusive, over the lanes
    {
        double v = tot[0];
#pragma unroll
        for (int q = 1; q < PPL; ++q) v += tot[q];
        return wave_scan_inclusive(v);
    }
    // The token's weight leaves its piece.  true (in every lane): the difference may be little but rounding
    // and the piece has to be summed anew (set).  That is where less than 2^-20 is left of what
    // the piece had at first (`least`); above, the rounding is below 2^-33 of what is left.
    __device__ __forceinline__ bool remove(int token, float weight, int lane)
    {
        const int j = token >> 8;
        bool little = false;
#pragma unroll
        for (int q = 0; q < PPL; ++q)
            if (j == lane * PPL + q) {
                tot[q] -= (double)weight;
                little = tot[q] < least[q];
            }
        return __ballot(little) != 0ull;
    }
    __device__ __forceinline__ void set(int j, double total, int lane)
    {
#pragma unroll
        for (int q = 0; q < PPL; ++q)
            if (j == lane * PPL + q) tot[q] = total;
    }
};

__device__ __forceinline__ double readlane_d(double v, int lane)
{
    const long long x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)x, lane), hi = __builtin_amdgcn_readlane((int)(x >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

struct Drawn {
    int token;
    float weight;
    int near;
};

// This lane's weights of piece j, which the calling wavefront holds.  The tokens of taken[0 .. n_taken)
// have left the row: their weights count as zero.
template <int ITEMS, int VT>
__device__ __forceinline__ float4 piece_values(const float4 (&a)[ITEMS], int j, int lane, const Drawn *taken, int n_taken)
{
    const int is = j / Pieces<ITEMS, VT>::NW;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (i == is) v = a[i];
    for (int n0 = 0; n0 < n_taken; n0 += 64) {
        const int x_lane = n0 + lane < n_taken ? taken[n0 + lane].token : -1;
        for (unsigned long long m = __ballot((x_lane >> 8) == j); m; m &= m - 1) {      // those of this piece
            const int x = __builtin_amdgcn_readlane(x_lane, __ffsll((long long)m) - 1);
            if ((x >> 2) == 64 * j + lane) {
                if ((x & 3) == 0) v.x = 0.f;
                if ((x & 3) == 1) v.y = 0.f;
                if ((x & 3) == 2) v.z = 0.f;
                if ((x & 3) == 3) v.w = 0.f;
            }
        }
    }
    return v;
}

// The smallest token whose cumulative weight exceeds tau = u A, or the last one that carries weight
// where rounding leaves none.  `incl` = P.scan().  Every wavefront calls it; the one that owns the
// token writes it, its weight and whether tau lies within tol of an edge of its interval to *out
// (-1 if nothing carries weight: then wavefront 0 does); the caller publishes with one barrier.
// taken, n_taken: as above.  (The rule among the 256 tokens of the piece is that of verification's search_piece, near ties among
// them, and has to stay that.  One function for both cost the sampler 0.05 us per draw: 16 from a row of 4000 14.0 -> 14.8 us.)
template <int ITEMS, int VT>
__device__ __forceinline__ void draw_token(const float4 (&a)[ITEMS], const Pieces<ITEMS, VT> &P, double incl, double tau, double tol,
                                           int lane, int wave, Drawn *out, const Drawn *taken = nullptr, int n_taken = 0)
{
    constexpr int PPL = Pieces<ITEMS, VT>::PPL, NW = Pieces<ITEMS, VT>::NW;
    // piece of the crossing; without one, the last piece that carries weight
    double mine_tot = P.tot[0];
#pragma unroll
    for (int q = 1; q < PPL; ++q) mine_tot += P.tot[q];
    const unsigned long long cross = __ballot(incl > tau), weight = __ballot(mine_tot > 0.0);
    if (!cross && !weight) {
        if (wave == 0 && lane == 0) *out = {-1, 0.f, 1};
        return;
    }
    const int ls = cross ? __ffsll((long long)cross) - 1 : 63 - __clzll((long long)weight);
    double base = readlane_d(incl, ls > 0 ? ls - 1 : 0);
    if (ls == 0) base = 0.0;
    int qs = -1, q_last = 0;
    double run = base, run_last = base;
#pragma unroll
    for (int q = 0; q < PPL; ++q) {
        const double tq = readlane_d(P.tot[q], ls);
        if (qs < 0) {
            if (tq > 0.0) { q_last = q; run_last = run; }
            if (cross && run + tq > tau) { qs = q; base = run; }
            else run += tq;
        }
    }
    const bool exact = qs >= 0;
    if (!exact) { qs = q_last; base = run_last; }
    const int j = __builtin_amdgcn_readfirstlane(ls * PPL + qs);
    if (j % NW != wave) return;
    const float4 v = piece_values<ITEMS, VT>(a, j, lane, taken, n_taken);
    const double part = sum4(v);
    const double hi_lane = base + wave_scan_inclusive(part);
    const unsigned long long c2 = __ballot(hi_lane > tau), w2 = __ballot(part > 0.0);
    if (!c2 && !w2) {                       // (a piece whose total is rounding residue)
        if (lane == 0) *out = {4 * (64 * j + 63) + 3, 0.f, 1};
        return;
    }
    const bool found = exact && c2 != 0ull;
    const int l2 = found ? __ffsll((long long)c2) - 1 : 63 - __clzll((long long)(w2 ? w2 : c2));
    double lo = readlane_d(hi_lane, l2 > 0 ? l2 - 1 : 0);
    if (l2 == 0) lo = base;
    if (lane == l2) {
        const float w[4] = {v.x, v.y, v.z, v.w};
        double cum = lo, hi = hi_lane;
        int pick = -1, last_pos = -1;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double nxt = cum + (double)w[e];
            if (w[e] > 0.f) last_pos = e;
            if (found && pick < 0 && nxt > tau) { pick = e; lo = cum; hi = nxt; }
            cum = nxt;
        }
        int near = 1;
        if (pick >= 0) near = (fabs(tau - lo) < tol || fabs(hi - tau) < tol) ? 1 : 0;
        else pick = last_pos < 0 ? 3 : last_pos;
        float wt = w[0];
        if (pick == 1) wt = w[1];
        if (pick == 2) wt = w[2];
        if (pick == 3) wt = w[3];
        *out = {4 * (64 * j + lane) + pick, wt, near};
    }
}

// Index of the n-th set bit (n from 0) of a 128-bit mask, the masks of the children of a row.
struct Kids {
    unsigned long long m0, m1;
    __device__ __forceinline__ int count() const { return __popcll(m0) + __popcll(m1); }
    // rank of node `lane` / `64 + lane` among the children
    __device__ __forceinline__ int rank0(int lane) const { return __popcll(m0 & ((1ull << lane) - 1ull)); }
    __device__ __forceinline__ int rank1(int lane) const { return __popcll(m0) + __popcll(m1 & ((1ull << lane) - 1ull)); }
};

}  // namespace vocab
}  // namespace mcsd
