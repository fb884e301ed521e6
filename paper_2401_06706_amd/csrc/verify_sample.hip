// Multi-candidate speculative sampling on gfx950: Algorithm 1 (with replacement),
// Algorithm 2 (without replacement), the endpoint draws and the root-to-leaf walk.
//
// One workgroup owns one row of the tree (the root or a node).  Both logit rows of the node are read
// from HBM exactly once with 128-bit loads and stay on the compute unit, in registers and (the larger
// vocabularies) partly in LDS, for all k sequential accept/reject rounds; every round reads the
// resident data once and adds up.
//
// Algorithm 2's removal of a rejected token from q needs no pass: that token's residual is already
// 0 and stays 0 whatever is subtracted from it later, so only Z_q changes, by exactly the fp32 weight
// of the token.  (A residual that vanished stays what it was; a token that leaves q with some of its p left keeps that in a list.)
//
// Instead of renormalising after each rejection the kernels have an
// unnormalised residual a(x) and its sum A (p-hat = a / A), and the unnormalised
// draft weights e_q(x) with the running mass Z_q of the tokens not yet removed
// (q-bar = e_q / Z_q).  Algorithm 1/2's update p := max(0, p - q) / sum(...) then
// reads a := max(0, a - beta e_q) with beta = A / Z_q, A := sum a, and the normaliser the paper
// divides by (the probability of the rejection, Appendix A) is A_new / A_old.  What is once zero stays zero, so
// a is max(0, e_p - C e_q) with C the sum of the betas: no row is rewritten, but for the seldom one of which little is left.
//
// The handful of numbers that decide an accept test - a(x), e_q(x) at the k
// candidate tokens - are tracked separately in fp64 by one lane per candidate, in every wavefront,
// so that the comparison u <= min(1, p/q) is taken at far better than the 1e-6
// near-tie band; vocabulary-wide passes are fp32 with fp64 accumulation.
#include <math.h>

#include "mcsd_internal.h"
#include "vocab_row.h"

namespace mcsd {
namespace {

using namespace vocab;

constexpr float LOG2E_F = 1.44269504088896340736f;
constexpr int MAX_BASES = 16;      // a row is written anew when 2^-16 of its sum is left: of 1 down to the smallest float ten times

struct VerifyParams {
    int B, N, V, P, variant, gamma_max, per_seq, ranked;
    float eps;
    const float *target_logits, *draft_logits;
    const int32_t *q_row, *parent, *cand_tok;
    const float *u_accept, *u_endpoint, *temperature;
    int32_t *n_accepted, *accepted_path, *out_tokens, *acc_child, *endpoint;
    float *ratio;
    uint32_t *flags;
    float *residual_out;
};

// 2^x in fp64 for x <= 0 (one wavefront evaluates it for the candidates of a row): x = n + f with
// |f| <= 1/2, 2^f = exp(f ln 2) by its Taylor series to degree 13 (|f ln 2| <= 0.35: truncation
// below 1e-17), scaled by 2^n.  Arguments below -1000 return 0.  (The coefficients are named where they
// are used: the compiler would keep all of them in registers through the loop over the rounds.)
__device__ __forceinline__ double coefficient(double c)
{
    asm volatile("" : "+s"(c));
    return c;
}

__device__ __forceinline__ double exp2_neg(double x)
{
    if (!(x > -1000.0)) return 0.0;
    const double n = rint(x);
    const double y = (x - n) * coefficient(0.69314718055994530942);
    double r = coefficient(1.0 / 6227020800.0);
    r = fma(r, y, coefficient(1.0 / 479001600.0));
    r = fma(r, y, coefficient(1.0 / 39916800.0));
    r = fma(r, y, coefficient(1.0 / 3628800.0));
    r = fma(r, y, coefficient(1.0 / 362880.0));
    r = fma(r, y, coefficient(1.0 / 40320.0));
    r = fma(r, y, coefficient(1.0 / 5040.0));
    r = fma(r, y, coefficient(1.0 / 720.0));
    r = fma(r, y, coefficient(1.0 / 120.0));
    r = fma(r, y, coefficient(1.0 / 24.0));
    r = fma(r, y, coefficient(1.0 / 6.0));
    r = fma(r, y, 0.5);
    r = fma(r, y, 1.0);
    r = fma(r, y, 1.0);
    return ldexp(r, (int)n);
}

// e_q of four logits, bit for bit what every pass (and the thread that tracks a candidate
// token) computes: subtraction first, then the scale, then v_exp_f32.
__device__ __forceinline__ float4 exp_weights(const float4 &z, float m, float c)
{
    return make_float4(__builtin_amdgcn_exp2f((z.x - m) * c), __builtin_amdgcn_exp2f((z.y - m) * c),
                       __builtin_amdgcn_exp2f((z.z - m) * c), __builtin_amdgcn_exp2f((z.w - m) * c));
}

// A condition that is the same in all lanes though the compiler can not know it: as a scalar, so that
// the branch on it is one.
__device__ __forceinline__ bool uniform(bool c) { return __builtin_amdgcn_readfirstlane(c ? 1 : 0) != 0; }
__device__ __forceinline__ double uniform(double v) { return readlane_d(v, 0); }

// The sequence of rank y when the sampled sequences come before the argmax ones (each group in its
// own order), and its temperature.  Workgroups start in the order y, x, and a sampled sequence costs
// a workgroup about three times what an argmax sequence costs (two rows, exponentials, k dependent
// rounds against one row and an argmax): handed out first, the cheap ones fill the end of the launch.
// Every wavefront finds it by itself, without a barrier.  Not where all workgroups start at once
// (the row would be requested a trip to memory later for nothing); batches above 512 keep their order.
__device__ __forceinline__ void ranked_sequence(const float *temperature, bool ranked, int B, int y, int lane, int *seq, float *T)
{
    if (!ranked || B > 512) {
        *seq = y;
        *T = temperature[y];
        return;
    }
    auto pick = [&](unsigned long long m, int n, float t, int base) {      // n-th set bit of m
        const bool here = ((m >> lane) & 1ull) && __popcll(m & ((1ull << lane) - 1ull)) == n;
        const int l = __ffsll((long long)__ballot(here)) - 1;
        *seq = base + l;
        *T = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), l));
    };
    if (B <= 64) {
        const float t = (lane < B) ? temperature[lane] : 0.f;
        const unsigned long long in = B < 64 ? (1ull << B) - 1ull : ~0ull, sampled = __ballot(t != 0.f) & in;
        const int total = __popcll(sampled);
        if (y < total) pick(sampled, y, t, 0);
        else pick(in & ~sampled, y - total, t, 0);
        return;
    }
    float t[8];
    int total = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) t[c] = (64 * c + lane < B) ? temperature[64 * c + lane] : 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) total += __popcll(__ballot(t[c] != 0.f));
    const bool want_sampled = y < total;
    int n = want_sampled ? y : y - total;
    *seq = 0;
    *T = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const int left = B - 64 * c;
        const unsigned long long in = left >= 64 ? ~0ull : (left > 0 ? (1ull << left) - 1ull : 0ull);
        const unsigned long long sampled = __ballot(t[c] != 0.f), m = want_sampled ? sampled : (in & ~sampled);
        const int have = __popcll(m);
        if (n >= 0 && n < have) pick(m, n, t[c], 64 * c);
        n -= have;
    }
}

// Sums in the lanes of the first row of 16, in order (0 in the others): the lane with the smallest number whose
// running sum from *from on exceeds tau (while *crossing: there is one), or the last that carries weight where
// rounding leaves none (then *crossing goes false), -1 without any weight.  *from goes on to the sum ahead of that lane.
__device__ __forceinline__ int find_crossing(double sum, double tau, int lane, bool *crossing, double *from)
{
    double incl = sum;
    incl += dpp_d<DPP_ROW_SHR1, 0xf>(0.0, incl);
    incl += dpp_d<DPP_ROW_SHR2, 0xf>(0.0, incl);
    incl += dpp_d<DPP_ROW_SHR4, 0xf>(0.0, incl);
    incl += dpp_d<DPP_ROW_SHR8, 0xf>(0.0, incl);
    const unsigned cross = (unsigned)__ballot(*from + incl > tau && sum > 0.0) & 0xffffu, weight = (unsigned)__ballot(sum > 0.0) & 0xffffu;
    *crossing = *crossing && cross != 0u;
    const int at = *crossing ? __ffs((int)cross) - 1 : (weight ? 31 - __clz((int)weight) : -1);
    if (at > 0) *from += readlane_d(incl, at - 1);
    return at;
}

// The token of a crossing among 256 consecutive ones, four per lane (`first`: the first of them, `base`: the
// weight ahead of them), as draw_token finds it: the smallest whose cumulative weight exceeds tau, or, without one, the last
// that carries weight.  `exact`: a crossing is expected here (false: only the fallback counts).  *holder: the lane whose
// result it is.
__device__ __forceinline__ Drawn search_piece(const float4 &v, double base, double tau, double tol, bool exact, int first, int lane, int *holder)
{
    const double part = sum4(v);
    const double hi_lane = base + wave_scan_inclusive(part);
    const unsigned long long c2 = __ballot(hi_lane > tau), w2 = __ballot(part > 0.0);
    const bool found = exact && c2 != 0ull;
    const int l2 = found ? __ffsll((long long)c2) - 1 : (c2 | w2) ? 63 - __clzll((long long)(w2 ? w2 : c2)) : 63;
    *holder = l2;
    double cum = l2 > 0 ? readlane_d(hi_lane, l2 > 0 ? l2 - 1 : 0) : base, lo = cum, hi = cum;     // (of lane l2)
    const float w[4] = {v.x, v.y, v.z, v.w};
    int pick = -1, last_pos = 3;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const double nxt = cum + (double)w[e];
        if (pick < 0 && w[e] > 0.f) last_pos = e;
        if (found && pick < 0 && nxt > tau) { pick = e; lo = cum; hi = nxt; }
        cum = nxt;
    }
    if (pick < 0) return {first + 4 * lane + last_pos, 0.f, 1};
    return {first + 4 * lane + pick, 0.f, (fabs(tau - lo) < tol || fabs(hi - tau) < tol) ? 1 : 0};
}

// The same number, unknown to the compiler: what follows from it is computed where it is used and not kept in
// registers from an earlier use, or from before a loop, on.
__device__ __forceinline__ int anew(int x)
{
    asm volatile("" : "+s"(x));
    return x;
}

// The kernel's arguments, read again: for what is needed late, or seldom.
__device__ __forceinline__ const VerifyParams *arguments()
{
    unsigned long long x = (unsigned long long)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(x));
    return (const VerifyParams *)(const __attribute__((address_space(4))) VerifyParams *)x;
}

// What one wavefront holds of a row: `items` x 256 consecutive tokens, 4 per lane and item.
// DEALT: the items are consecutive too, the wavefronts in the order of the tokens.  Then the totals of the wavefronts,
// which every sum over the workgroup leaves in LDS, say which of them holds the endpoint, and that one finds it by itself.
// The 256-token pieces of the row are dealt evenly.
// Otherwise wavefront w holds the pieces w, w + NW, ...: the workgroup reads a row in order, which HBM takes better when
// all units read at once (16 x 61 argmax rows of 32000 23.9 us against 25.8 dealt).
template <int VT, bool ALIGNED, bool DEALT>
struct Share {
    static constexpr int NW = VT / 64, STEP = DEALT ? 64 : VT;      // float4 of the row between two items
    int items, first;       // `first`: the first token
    int n4;                 // the float4 of the row that follow `first`, those of the share at least (0: none)
    int tail;               // place of the incomplete float4 at the end of the row behind `first`, -1 if it is not here
    __device__ __forceinline__ Share(int V, int wave)
    {
        const int pieces = (V + 255) >> 8;
        if (DEALT) {
            const int from = wave * pieces / NW;
            items = (wave + 1) * pieces / NW - from;
            first = from * 256;
        } else {
            items = (pieces + NW - 1) / NW;
            first = wave * 256;
        }
        const int left = (V >> 2) - (first >> 2), most = DEALT ? 64 * items : left;
        n4 = left < 0 ? 0 : (left < most ? left : most);
        tail = (!ALIGNED && left >= 0 && (!DEALT || left < most)) ? left : -1;
    }
    __device__ __forceinline__ int token(int i, int lane) const { return first + 4 * (STEP * i + lane); }
    // the item of a token, if this lane holds it (-1: it does not)
    __device__ __forceinline__ int item_of(int token, int lane) const
    {
        const int x = token - first, i = x / (4 * STEP);
        return (x >= 0 && i < items && x - i * (4 * STEP) < 256 && ((x >> 2) & 63) == lane) ? i : -1;
    }
    // The float4 of a row, requested with 128-bit loads through a resource that ends with them: those past
    // the row or the share come as zeros without a trip to memory.  A row whose
    // length is no multiple of four starts at any 4-byte address, which these loads allow; its last
    // tokens (fewer than four) come by single loads, so that no load straddles the end of the resource.
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t resource(const float *row) const
    {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(row) + first, 0, n4 * 16, 0x00020000);
    }
    template <int ITEMS>
    __device__ __forceinline__ void request(__amdgpu_buffer_rsrc_t rs, int lane, float4 (&r)[ITEMS]) const
    {
        constexpr int NT = 2;                   // non-temporal: a logit row is read once
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, i * (STEP * 16), NT);
            r[i] = make_float4(__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3]));
        }
    }
    __device__ __forceinline__ float4 request_tail(const float *row, int V) const
    {
        const float ninf = -INFINITY;
        const int V4 = V & ~3;
        const __amdgpu_buffer_rsrc_t rt = row_resource(row, V);
        float4 t = make_float4(ninf, ninf, ninf, ninf);
        if (!ALIGNED) {
            const float x = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rt, 0, V4 * 4, 2));
            const float y = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rt, 4, V4 * 4, 2));
            const float z = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rt, 8, V4 * 4, 2));
            if (V4 < V) t.x = x;
            if (V4 + 1 < V) t.y = y;
            if (V4 + 2 < V) t.z = z;
        }
        return t;
    }
    __device__ __forceinline__ bool whole(int i) const { return STEP * i + 64 <= n4; }       // (uniform)
    // item i with -inf past the row
    __device__ __forceinline__ void settle(int i, int lane, float4 &r, const float4 &t) const
    {
        const float ninf = -INFINITY;
        const int e = STEP * i + lane;
        const bool past = e >= n4, at = !ALIGNED && e == tail;
        r = make_float4(past ? (at ? t.x : ninf) : r.x, past ? (at ? t.y : ninf) : r.y, past ? (at ? t.z : ninf) : r.z, past ? ninf : r.w);
    }
};

// One workgroup per tree row.  Both logit rows are read from HBM once and stay on the compute unit
// for all rounds: the target row in registers (as unnormalised weights e_p), the draft row (as
// e_q) in registers up to item ITEMS - LQ and in LDS beyond.  LQ is chosen so that two workgroups
// share a compute unit (256 registers per thread, 80 KB of LDS each), one loading while the other
// computes: the two row pairs of 32000 tokens are 512 KB, as much as all registers of the unit.
//
// The residual of round n is max(0, e_p - C e_q) with C the sum of the betas so far (what is once zero
// stays zero), so that the target row need not change: a pass reads, clamps and adds up, and a rejection
// that would leave nothing is undone by keeping the old C.  C has 48 bits, as two floats, so what is
// left of a row may not become small beside what was subtracted: at 2^-16 the row is written anew, C begins
// at 0 again, and the candidates' tracks begin from the betas (which nothing but these seldom cases reads).
// Without that 2^-53 of p was nothing; with it, and with the exact quotient, 29 rows of 32000 take
// 15.8 us where they took 15.6 (candidates mostly rejected, from memory), 4 x 17 of 50001 with 16 rejections 59.5 and 57.8, 16 x 61 as before.
//
// Bound: HBM in a batch (16 sequences of 61 rows of 32000, 8 of them argmax: 171 MB in 33 us), the vector units of one CU
// for a single sequence (29 rows, 512 threads, a row with four rejections): the target row there 1.5 us and the draft row 3.8
// (256 KB through one CU, from memory), all exponentials and sums 6.4, 1.4 per rejection, 0.9 of which is the pass (two products, a
// conversion and an fp64 addition per token, at the full rate of a SIMD), 1.2 the endpoint.  With the residual in the row, the
// ratio and beta divided behind the barrier, and piece totals of the whole row for the endpoint it was 1.7 per rejection and
// 2.3 for the endpoint.  A call with its walk: c2's 29 rows 18.6 -> 17.3 us, 6 x 29 rows of 50001 32.8 -> 28.3 (its items
// past the row are not worked), 16 x 57 rows of 65536 110 -> 91, 16 x 61 of 20000 47.6 -> 40.5.
template <int ITEMS, int VT, int LQ, int WGS, bool DEALT, bool ALIGNED>
__global__ __launch_bounds__(VT) __attribute__((amdgpu_waves_per_eu(WGS * VT / 256)))
void verify_rows_kernel(VerifyParams p)
{
    constexpr int NWAVES = VT / 64, RQ = ITEMS - LQ, GI = ITEMS / 4;
    constexpr int GM = ITEMS < 8 ? ITEMS : 8, G = WGS * VT >= 1024 ? 2 : 4;         // items that are worked or skipped together: what their values in flight leave room for
    const int row = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int N = p.N, V = p.V;

    __shared__ float4 s_q[LQ ? LQ * VT : 1];            // [item - RQ][thread]: every thread reads only what is its own
    __shared__ double s_sum[2][2][NWAVES];
    __shared__ double s_part[DEALT ? 1 : 4][NWAVES], s_item[DEALT ? 1 : GI][NWAVES];
    __shared__ float s_max[2][NWAVES];
    __shared__ int s_besti[NWAVES];
    __shared__ int s_best;
    __shared__ int s_gone_tok[MCSD_MAX_NODES], s_kept_tok[MCSD_MAX_NODES];
    __shared__ double s_beta[MCSD_MAX_NODES];           // of the rejections; s_gone_tok: the token that left q by each, or -1
    __shared__ float s_base[MAX_BASES][2];              // C of the rows that were written anew
    __shared__ float s_kept[MCSD_MAX_NODES], s_kept_w[MCSD_MAX_NODES][2];       // what they keep; e_p and e_q
    __shared__ double s_cand[2][64];                    // e_p and e_q of the candidates of 64 nodes

    int b;
    float T_of_b;
    ranked_sequence(p.temperature, p.ranked, p.B, blockIdx.y, lane, &b, &T_of_b);
    const int qr_of_row = p.q_row[(p.per_seq ? (size_t)b * (1 + N) : 0) + row];
    const size_t rix = (size_t)b * (1 + N) + row, nodes = (size_t)b * N;
    const float *zp_row = p.target_logits + rix * (size_t)V;
    const bool naive = (p.variant == MCSD_NAIVE);      // the draft row is not needed: candidates are only compared
    const float NaN = __int_as_float(0x7fc00000);
    Share<VT, ALIGNED, DEALT> own(V, wave);
    constexpr int STEP = DEALT ? 64 : VT;

    // Requested ahead of the rows (memory answers in order), by every wavefront for itself: the parents and
    // the candidates; lane = node here, and 64 + lane.
    auto node_words = [&](const void *x) __attribute__((always_inline)) {      // 32 bits per node of the sequence
        return __builtin_amdgcn_make_buffer_rsrc((char *)x + 4 * nodes, 0, N * 4, 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t rs_parent = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(p.parent) + (p.per_seq ? nodes : 0), 0, N * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_tok = node_words(p.cand_tok);
    const int pa0 = __builtin_amdgcn_raw_buffer_load_b32(rs_parent, lane * 4, 0, 0), pa1 = __builtin_amdgcn_raw_buffer_load_b32(rs_parent, lane * 4, 256, 0);
    const int tok0 = __builtin_amdgcn_raw_buffer_load_b32(rs_tok, lane * 4, 0, 0), tok1 = __builtin_amdgcn_raw_buffer_load_b32(rs_tok, lane * 4, 256, 0);
    __builtin_amdgcn_sched_barrier(0);
    float4 a[ITEMS], eq[RQ];
    own.request(own.resource(zp_row), lane, a);
    const float4 tail_p = own.request_tail(zp_row, V);
    __builtin_amdgcn_sched_barrier(0);
    // A row has a draft row iff q_row says so; whether it also has children is known at about the same time
    // (a mismatch is flagged, the row then counts as a leaf and the extra row is ignored).
    // (as scalars: the branches on them below are then scalar too)
    const float T = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(T_of_b)));
    const int qr = __builtin_amdgcn_readfirstlane(qr_of_row);
    const bool have_q = (qr >= 0 && qr < p.P) && (T != 0.f) && !naive;
    const float *zq_row = have_q ? p.draft_logits + ((size_t)b * p.P + qr) * (size_t)V : zp_row;

    const bool f0 = lane < N && pa0 == row - 1, f1 = 64 + lane < N && pa1 == row - 1;
    const Kids kids = {__ballot(f0), __ballot(f1)};
    uint32_t fl = 0u;
    int k = kids.count();
    if (k > 0 && (qr < 0 || qr >= p.P)) {
        // a row with children needs a draft row; a bad map is reported, never dereferenced
        k = 0;
        fl = (uint32_t)MCSD_FLAG_BAD_TREE;
    }
    const bool rounds = k > 0 && have_q;
    // The candidates of the first 64 nodes that hold any, a lane each: token, uniform and the two logits
    // (naive sampling reads neither draft logits nor u_accept, argmax sampling nothing of this).
    int base = kids.m0 ? 0 : 64;
    int my_tok = base ? tok1 : tok0;
    bool valid = (base ? f1 : f0) && my_tok >= 0 && my_tok < V;
    const __amdgpu_buffer_rsrc_t rs_u = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.u_accept) + nodes, 0, have_q ? N * 4 : 0, 0x00020000);
    float my_u = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_u, lane * 4, base * 4, 0));
    const int at = valid && have_q ? my_tok * 4 : V * 4;    // (past the end: zero)
    float my_zp = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(row_resource(zp_row, V), at, 0, 0));
    float my_zq = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(row_resource(zq_row, V), at, 0, 0));
    const float u_end = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(row_resource(p.u_endpoint + rix, T != 0.f ? 1 : 0), 0, 0, 0));
    __builtin_amdgcn_sched_barrier(0);
    // (ahead of the passes over the row: a branch per item inside them costs more than the items skipped in them save)
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        if (!own.whole(j)) own.settle(j, lane, a[j], tail_p);
        // (One register per value on both ways; without this the compiler copies two of each four, and puts 8 registers aside for it
        // instead of 4: 16 x 61 rows of 32000 48.1 us, 47.3 with it.  Not where it is the other way round: 8 items, odd lengths two to a CU.)
        if (ITEMS >= 16 && (ALIGNED || WGS == 1)) asm("" : "+v"(a[j].x), "+v"(a[j].y), "+v"(a[j].z), "+v"(a[j].w));
    }
    if (T == 0.f) {
        // argmax sampling: lowest id on ties.  Ascending token order: a strict comparison keeps the
        // first of equal values; elements are named by their number in the thread (an inline constant).
        float bv = -INFINITY;
        int bc = -1;
#pragma unroll
        for (int g = 0; g < ITEMS; g += GM) {
            if (g > 0 && g >= own.items) continue;
#pragma unroll
            for (int j = g; j < g + GM; ++j) {
                const float v[4] = {a[j].x, a[j].y, a[j].z, a[j].w};
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (v[c] > bv) { bv = v[c]; bc = 4 * j + c; }
            }
        }
        int bi = bc >= 0 ? own.token(bc >> 2, lane) + (bc & 3) : 0x7fffffff;
        wave_argmax(bv, bi);
        if (lane == 0) { s_max[0][wave] = bv; s_besti[wave] = bi; }
        __syncthreads();
        bv = s_max[0][0]; bi = s_besti[0];
#pragma unroll
        for (int w = 1; w < NWAVES; ++w) {
            const float ov = s_max[0][w];
            const int oi = s_besti[w];
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        }
        if (bi == 0x7fffffff) bi = 0;
        if (wave == 0) {
            // the first child (ascending node id) that proposed the argmax is accepted
            const bool c0 = k > 0 && f0, c1 = k > 0 && f1;
            const unsigned long long m0 = __ballot(c0 && tok0 == bi), m1 = __ballot(c1 && tok1 == bi);
            if (__ballot((c0 && (tok0 < 0 || tok0 >= V)) || (c1 && (tok1 < 0 || tok1 >= V)))) fl |= (uint32_t)MCSD_FLAG_BAD_TOKEN;
            const int acc = m0 ? __ffsll((long long)m0) - 1 : (m1 ? 63 + __ffsll((long long)m1) : -1);
            if (lane == 0) {
                p.acc_child[rix] = acc;
                p.endpoint[rix] = acc < 0 ? bi : -1;
                p.flags[rix] = fl;
            }
            if (p.ratio) {
                if (c0) p.ratio[nodes + lane] = NaN;
                if (c1) p.ratio[nodes + 64 + lane] = NaN;
            }
        }
        if (p.residual_out) {
            float *dst = p.residual_out + rix * (size_t)V;
            for (int e = t; e < V; e += VT) dst[e] = (e == bi) ? 1.f : 0.f;
        }
    }
    // (no return above: with one, the compiler keeps what the other path needs alive beside this one)
    if (T != 0.f) {
        const float c2 = (1.0f / T) * LOG2E_F;
        // the maximum over the workgroup; one barrier
        auto row_top = [&](float m, int slot) __attribute__((always_inline)) {
            m = wave_max(m);
            if (lane == 63) s_max[slot][wave] = m;
            __syncthreads();
            m = s_max[slot][0];
#pragma unroll
            for (int w = 1; w < NWAVES; ++w) m = fmaxf(m, s_max[slot][w]);
            return m;
        };
        // The sum of x over the workgroup: every wavefront leaves its own, and behind a barrier each adds them
        // all (slot: 0 and 1 in turn, so that no writer overtakes a reader).
        auto leave_sum = [&](double x, int which, int slot) __attribute__((always_inline)) {
            x = wave_sum_all(x);
            if (lane == 0) s_sum[slot][which][wave] = x;
        };
        auto read_total = [&](int which, int slot) __attribute__((always_inline)) {
            double x = s_sum[slot][which][lane & (NWAVES - 1)];
            x += mov_dpp_d<DPP_QUAD_1032>(x);
            x += mov_dpp_d<DPP_QUAD_2301>(x);
            if (NWAVES == 8) x += mov_dpp_d<DPP_ROW_HALF_MIRROR>(x);
            return x;
        };

        float mp = -INFINITY, mq = -INFINITY;
        // e_p and e_q of the lanes' candidates in fp64, with the constants of the vector passes (float c2)
        // evaluated exactly, by one wavefront each
        auto leave_weights = [&]() __attribute__((always_inline)) {
            if (wave < 2) s_cand[wave][lane] = exp2_neg(((double)(wave ? my_zq : my_zp) - (double)(wave ? mq : mp)) * (double)c2);
        };
#pragma unroll
        for (int g = 0; g < ITEMS; g += GM) {
            if (g > 0 && g >= own.items) continue;
#pragma unroll
            for (int j = g; j < g + GM; ++j) {
                mp = max3_raw(max3_raw(mp, a[j].x, a[j].y), a[j].z, a[j].w);
            }
        }
        mp = row_top(mp, 0);
        // The draft row is requested when all of the target row is there and comes while that goes through
        // its exponentials (requested together, the last wavefront's share of the target row came with the draft row).
        // A row without rounds gets zeros by the same requests, with a resource that holds nothing.
        const __amdgpu_buffer_rsrc_t rs_q = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(zq_row) + own.first, 0, rounds ? own.n4 * 16 : 0, 0x00020000);
        own.request(rs_q, lane, eq);
        const float4 tail_q = own.request_tail(zq_row, V);
        if (LQ) {
            // straight into LDS (16 bytes per lane, consecutive): no registers while in flight
            typedef __attribute__((address_space(3))) void *lds_ptr;
#pragma unroll
            for (int i = 0; i < LQ; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_q, (lds_ptr)(s_q + i * VT + 64 * wave), 16, lane * 16, (RQ + i) * (STEP * 16), 0, 2);
        }
        __builtin_amdgcn_sched_barrier(0);
        // Sums of the row's weights (then of its residual) by fourths of the share, GI items each: who has the endpoint
        // looks for it in one of them.
        double part[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int g = 0; g < ITEMS; g += G) {
            if (g > 0 && g >= own.items) continue;
#pragma unroll
            for (int j = g; j < g + G; ++j) {
                a[j] = exp_weights(a[j], mp, c2);            // a = e_p
                part[j / GI] += sum4(a[j]);
            }
            __builtin_amdgcn_sched_barrier(0);      // (a few items at a time: more would not fit the registers)
        }
        double Zq = 0.0;
        if (rounds) {
            own.n4 = anew(own.n4);
            own.items = anew(own.items);
#pragma unroll
            for (int j = 0; j < RQ; ++j)
                if (!own.whole(j)) own.settle(j, lane, eq[j], tail_q);
#pragma unroll
            for (int g = 0; g < RQ; g += GM) {
                if (g > 0 && g >= own.items) continue;
#pragma unroll
                for (int j = g; j < g + GM && j < RQ; ++j) {
                    mq = max3_raw(max3_raw(mq, eq[j].x, eq[j].y), eq[j].z, eq[j].w);
                }
            }
            if (LQ) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // the part in LDS has arrived
#pragma unroll
                for (int j = RQ; j < ITEMS; ++j) {
                    if (j >= own.items) continue;
                    float4 z = s_q[(j - RQ) * VT + t];
                    if (!own.whole(j)) {
                        own.settle(j, lane, z, tail_q);
                        s_q[(j - RQ) * VT + t] = z;
                    }
                    mq = max3_raw(max3_raw(mq, z.x, z.y), z.z, z.w);
                }
            }
            mq = row_top(mq, 1);
            double partq[4] = {0.0, 0.0, 0.0, 0.0};     // (by fourths as well: equal rows have equal sums)
#pragma unroll
            for (int g = 0; g < ITEMS; g += G) {
                if (g > 0 && g >= own.items) continue;
#pragma unroll
                for (int j = g; j < g + G; ++j) {
                    if (j < RQ) {
                        eq[j < RQ ? j : 0] = exp_weights(eq[j < RQ ? j : 0], mq, c2);
                        partq[j / GI] += sum4(eq[j < RQ ? j : 0]);
                    } else if (j < own.items) {
                        const float4 e = exp_weights(s_q[(j - RQ) * VT + t], mq, c2);
                        s_q[(j - RQ) * VT + t] = e;
                        partq[j / GI] += sum4(e);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            leave_sum((partq[0] + partq[1]) + (partq[2] + partq[3]), 1, 0);
            leave_weights();
        }
        leave_sum((part[0] + part[1]) + (part[2] + part[3]), 0, 0);
        __syncthreads();
        double A = read_total(0, 0);
        if (rounds) Zq = read_total(1, 0);
        if (uniform((bool)(!((A > 0.0) & (A < INFINITY)) | (rounds & !((Zq > 0.0) & (Zq < INFINITY)))))) fl |= (uint32_t)MCSD_FLAG_NONFINITE;

        float Ch = 0.f, Cl = 0.f;                   // C as a two-term float, so that no common rounding of it biases the sums
        // The residual of a token and of item j; 0 <= e_p <= 1, so that the maximum with 0 is the clamp of the second product.
        // Items past the share may hold -inf as they were padded (the passes skip them by groups), and C e_q + e_p is NaN
        // there: v_med3_f32 gives the least of the other two for a NaN, 0, and so does the clamp bit it may become.
        auto residual_of = [&](float e_p, float e_q) __attribute__((always_inline)) {
            return __builtin_amdgcn_fmed3f(fmaf(-Cl, e_q, fmaf(-Ch, e_q, e_p)), 0.f, 1.f);
        };
        auto residual = [&](int j, const float4 &e) __attribute__((always_inline)) {
            return make_float4(residual_of(a[j].x, e.x), residual_of(a[j].y, e.y), residual_of(a[j].z, e.z), residual_of(a[j].w, e.w));
        };
        int tq = t;                                 // (set anew per pass: the reads of s_q stay where they are written)
        auto draft_item = [&](int j) __attribute__((always_inline)) { return j < RQ ? eq[j < RQ ? j : 0] : s_q[(j < RQ ? 0 : j - RQ) * VT + tq]; };
        auto sum_residual = [&]() __attribute__((always_inline)) {
            part[0] = part[1] = part[2] = part[3] = 0.0;
            asm volatile("" : "+v"(tq), "+v"(Ch));
            const int items = anew(own.items);
#pragma unroll
            for (int g = 0; g < ITEMS; g += G) {
                if (g > 0 && g >= items) continue;
#pragma unroll
                for (int j = g; j < g + G; ++j) part[j / GI] += sum4(residual(j, draft_item(j)));
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        int slot = 0;                               // where the totals of the residual's wavefronts are
        bool stale = false;                         // they, and part, are not those of the residual as it is now
        int accepted = -1;
        bool rejected = false;
        int n_kept = 0;                             // tokens that have left q and keep a residual that C does not lower (see below)
        if (rounds) {
            // Every wavefront follows the candidates of 64 nodes in fp64, a lane each, so that all of them take the
            // same decisions without a barrier; a round costs the one of its sum.
            double C = 0.0;
            float z_low = (float)Zq * 0x1p-16f, a_low = (float)A * 0x1p-16f;
            int n_bases = 0, n_left = 0;
            const bool removes = p.variant == MCSD_WITHOUT_REPLACEMENT;
            unsigned long long left = base ? kids.m1 : kids.m0;
            bool acc, low = false;
            auto split_C = [&](double c) __attribute__((always_inline)) {
                Ch = (float)c;
                Cl = (float)(c - (double)Ch);
            };
            // The rejections of some lanes, in their order behind the n_left that were left so far: how many they are then
            // (every wavefront writes the same, for itself).
            auto leave_rejections = [&](unsigned long long lanes, double my_beta) __attribute__((always_inline)) {
                if ((lanes >> lane) & 1ull) {
                    const int n = n_left + __builtin_amdgcn_mbcnt_hi((unsigned)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)lanes, 0u));
                    s_beta[n] = my_beta;
                    s_gone_tok[n] = removes && valid ? my_tok : -1;
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                return n_left + __popcll(lanes);
            };
            // the residual that the row has of a token
            auto in_row = [&](float e_p, float e_q) __attribute__((always_inline)) {
#pragma unroll 1
                for (int n = 0; n < n_bases; ++n) e_p = __builtin_amdgcn_fmed3f(fmaf(-s_base[n][1], e_q, fmaf(-s_base[n][0], e_q, e_p)), 0.f, 1.f);
                return residual_of(e_p, e_q);
            };
            for (;;) {
                // of the lane's candidate: the residual and e_q in fp64
                double my_a = s_cand[0][lane], my_q = s_cand[1][lane];
#pragma unroll 1
                for (int n = 0; n < n_left; ++n) {
                    my_a = fmax(0.0, my_a - s_beta[n] * my_q);
                    if (s_gone_tok[n] == my_tok) my_q = 0.0;
                }
                // What a decision needs besides A is computed while the sum is on its way.  x = a(x) Z_q / e_q(x): the
                // ratio is min(1, x / A), and u <= x / A is u A <= x.
                // Two per CU with LDS: x and 1 / Z_q at the end of a round, nothing across the pass, which leaves no registers
                // (16 x 61 rows of 32000 the other way 49.2 us, 48.1 this). Else the quotient stays until Z_q changes.
                constexpr bool LATE = LQ > 0 && WGS > 1;
                double x = 0.0, rz = 0.0, zr = 0.0;
                auto with_q = [&]() __attribute__((always_inline)) {
                    if (LATE) {
                        x = my_a * (Zq / my_q);
                        rz = Zq > 0.0 ? 1.0 / Zq : 0.0;
                    } else {
                        zr = Zq / my_q;
                    }
                };
                with_q();
                double of_x = 0.0, of_A = 0.0;      // the ratio that the lane's candidate was tested at: min(1, of_x / of_A)
                double my_beta = 0.0;               // of its rejection
                const unsigned long long all = left, good = __ballot(valid);
                unsigned long long no_q = 0ull;     // of those tested, the candidates that q did not have
                for (;;) {
                    const int l = __ffsll((long long)left) - 1;
                    left &= left - 1ull;
                    if (!LATE) x = my_a * zr;
                    const bool has_q = my_q > 0.0, sure = (has_q & !(x < A)) | (!has_q & (my_a > 0.0));     // a ratio of one
                    // (a token of probability zero - a duplicate of a rejected one, Sec. 3.2 - is never
                    // accepted, also not by a uniform of exactly 0 from outside the open interval)
                    const bool yes = valid & ((sure & (my_u <= 1.f)) | (!sure & has_q & (x > 0.0) & ((double)my_u * A <= x)));
                    acc = (__ballot(yes) >> l) & 1ull;
                    no_q |= __ballot(!has_q) & (1ull << l);
                    if (lane == l) {
                        of_x = sure ? INFINITY : (has_q ? x : 0.0);
                        of_A = A;
                    }
                    if (acc) {
                        accepted = base + l;
                        break;
                    }
                    // rejected: the residual with C + A / Z_q, in fp64 but for the two products per token.  (The token that
                    // leaves q keeps its e_q in the row: its residual is 0 now and stays 0 whatever is subtracted later.)
                    // A / Z_q, exactly 1 for equal sums; with 1 / Z_q at hand, their product and what is missing there.
                    // (Nothing left in q: the residual is p itself.)
                    double beta = LATE ? A * rz : A / Zq;
                    if (LATE) beta = fma(fma(-beta, Zq, A), rz, beta);
                    beta = Zq > 0.0 ? beta : 0.0;
                    if (lane == l) my_beta = beta;
                    rejected = true;
                    split_C(C + beta);
                    sum_residual();
                    slot ^= 1;
                    leave_sum((part[0] + part[1]) + (part[2] + part[3]), 0, slot);
                    my_a = fmax(0.0, my_a - beta * my_q);
                    const bool gone = removes && ((good >> l) & 1ull), at_one = (__ballot(sure) >> l) & 1ull;
                    const int tok = __builtin_amdgcn_readlane(my_tok, l);
                    if (gone) {
                        // Z_q loses exactly the fp32 weight that its sum contained (nothing where the token had left before)
                        const float w = __builtin_amdgcn_exp2f((__int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_zq), l)) - mq) * c2);
                        Zq -= (__ballot(has_q) >> l) & 1ull ? (double)w : 0.0;
                        if (my_tok == tok) my_q = 0.0;
                        if (!LATE) with_q();
                    }
                    if (LATE) with_q();
                    __syncthreads();
                    A = read_total(0, slot);
#pragma unroll 1
                    for (int n = 0; n < n_kept; ++n)        // in the place of what the row has of them
                        A += (double)s_kept[n] - (double)in_row(s_kept_w[n][0], s_kept_w[n][1]);
                    low = uniform(!(A > (double)a_low));
                    stale = low && uniform(!(A > 0.0));
                    if (stale) {
                        // max(0, p - q) vanished everywhere, which a rejection excludes in exact arithmetic
                        // (it needs p = q) and rounding or a bad candidate can produce: p stays as it was.
                        // (The candidates' tracks begin anew from the list of rejections, ahead of this loop.)
                        split_C(C);
                        A = readlane_d(of_A, l);
                        if (lane == l) my_beta = 0.0;
                        fl |= (uint32_t)MCSD_FLAG_ZERO_RESIDUAL;
                    } else {
                        C += beta;
                    }
                    if (gone) {
                        if (stale || at_one) {
                            // This token leaves q with some of its p left, or all (so does one that only a uniform above 1
                            // rejects): no later rejection may lower that.
                            bool known = false;
#pragma unroll 1
                            for (int n = 0; n < n_kept; ++n) known |= s_kept_tok[n] == tok;
                            const float zp = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(row_resource(zp_row, V), tok * 4, 0, 0));
                            const float e_p = __builtin_amdgcn_exp2f((zp - mp) * c2);
                            const float e_q = __builtin_amdgcn_exp2f((__int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_zq), l)) - mq) * c2);
                            if (uniform(!known)) {
                                if (lane == 0) { s_kept_tok[n_kept] = tok; s_kept[n_kept] = in_row(e_p, e_q); s_kept_w[n_kept][0] = e_p; s_kept_w[n_kept][1] = e_q; }
                                ++n_kept;
                            }
                        }
                        if ((left || (!base && kids.m1)) && uniform(Zq < (double)z_low)) {
                            // little of the mass is left and the difference has lost digits: the sum
                            // again without the removed tokens, from memory (rare; a pass over the
                            // resident row here would cost every row registers)
                            const __amdgpu_buffer_rsrc_t rs = row_resource(zq_row, V);
                            const int n_rejected = leave_rejections(all & ~left, my_beta);
                            double partq = 0.0;
#pragma unroll 1
                            for (int e0 = t; e0 < V; e0 += VT) {
                                const float e = __builtin_amdgcn_exp2f((__uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, e0 * 4, 0, 0)) - mq) * c2);
                                bool in = true;
#pragma unroll 1
                                for (int n = 0; n < n_rejected; ++n) in &= s_gone_tok[n] != e0;
                                if (in) partq += (double)e;
                            }
                            leave_sum(partq, 1, slot);
                            __syncthreads();
                            Zq = read_total(1, slot);
                            z_low = (float)Zq * 0x1p-16f;
                            with_q();
                        }
                    }
                    if (!left || low) break;
                }
                // their ratios (NaN: not tested) and flags
                const VerifyParams *late = arguments();
                const unsigned long long tested = all & ~left;
                const bool was = (tested >> lane) & 1ull;
                const double r = valid && of_x != 0.0 ? fmin(1.0, of_x / of_A) : 0.0;
                if (late->ratio && wave == 0 && ((all >> lane) & 1ull)) late->ratio[nodes + base + lane] = was ? (float)r : NaN;
                if (__ballot(was && fabs((double)my_u - r) < (double)late->eps)) fl |= (uint32_t)MCSD_FLAG_NEAR_TIE_ACCEPT;
                if (tested & ~good) fl |= (uint32_t)MCSD_FLAG_BAD_TOKEN;
                if (no_q & good) fl |= (uint32_t)MCSD_FLAG_ZERO_DRAFT_PROB;
                if (acc) {
                    if (!base && late->ratio && wave == 0 && ((kids.m1 >> lane) & 1ull)) late->ratio[nodes + 64 + lane] = NaN;
                    break;
                }
                if (!left && (base || !kids.m1)) break;
                n_left = leave_rejections(tested, my_beta);
                if (low && !stale && n_bases < MAX_BASES) {
                    // What is left is small beside what C e_q takes from e_p: C, of 48 bits as two floats, would lose it, and
                    // in the end nothing would be left.  The residual in the place of e_p, and C from 0 on, so that the error
                    // of C is 2^-33 of what is left at most.  (Seldom: with candidates drawn from q one row in 2^16.)
                    asm volatile("" : "+v"(tq), "+v"(Ch));
#pragma unroll
                    for (int j = 0; j < ITEMS; ++j) {
                        a[j] = residual(j, draft_item(j));
                        asm volatile("" : "+v"(a[j].x), "+v"(a[j].y), "+v"(a[j].z), "+v"(a[j].w), "+v"(tq));    // (item by item: LDS reads ahead do not fit the registers)
                    }
                    if (lane == 0) { s_base[n_bases][0] = Ch; s_base[n_bases][1] = Cl; }
                    ++n_bases;
                    C = 0.0;
                    Ch = Cl = 0.f;
                    a_low = (float)A * 0x1p-16f;
                }
                if (left) continue;
                base = 64;
                left = kids.m1;
                my_tok = __builtin_amdgcn_raw_buffer_load_b32(node_words(late->cand_tok), lane * 4, 256, 0);
                valid = f1 && my_tok >= 0 && my_tok < V;
                const int at1 = valid ? my_tok * 4 : V * 4;
                my_u = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(node_words(late->u_accept), lane * 4, 256, 0));
                my_zp = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(row_resource(zp_row, V), at1, 0, 0));
                my_zq = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(row_resource(zq_row, V), at1, 0, 0));
                leave_weights();                    // (no reader of the first is left behind the barriers of the rounds)
                __syncthreads();
            }
            if (n_kept && (accepted < 0 || p.residual_out)) {
                // the residual as it is, with the tokens that keep theirs
                __syncthreads();                    // the last of them is known
                asm volatile("" : "+v"(tq), "+v"(Ch));
#pragma unroll
                for (int j = 0; j < ITEMS; ++j) a[j] = residual(j, draft_item(j));
                Ch = Cl = 0.f;
                stale = true;
#pragma unroll 1
                for (int n = 0; n < n_kept; ++n) {
                    const int tok = s_kept_tok[n], item = own.item_of(tok, lane), c = tok & 3;
                    const float keeps = s_kept[n];
#pragma unroll
                    for (int j = 0; j < ITEMS; ++j)
                        if (j == item) {
                            if (c == 0) a[j].x = keeps;
                            if (c == 1) a[j].y = keeps;
                            if (c == 2) a[j].z = keeps;
                            if (c == 3) a[j].w = keeps;
                        }
                }
            }
        }
        if (LQ && !rounds) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // (the zeros in the place of the draft row)

        int endpoint = -1, acc_node = accepted;
        bool owner = wave == 0;                     // writes the row's outcome
        if (accepted < 0) {
            const double u = (double)u_end;
            asm volatile("" : "+v"(tq), "+v"(Ch));
            if (stale) {
                sum_residual();
                slot ^= 1;
                leave_sum((part[0] + part[1]) + (part[2] + part[3]), 0, slot);
                __syncthreads();
                A = read_total(0, slot);
            }
            if (uniform(isfinite(A))) {
                // Without a crossing, the last that carries weight; d: nothing does.
                const double tau = u * A, tol = (double)p.eps * A;
                double from = 0.0;
                bool crossing = true;
                int holder = 0;
                Drawn d = {-1, 0.f, 1};
                constexpr int REP = 16 / GI;                // lanes of a row that hold the same total of GI
                int which;
                // the items of one fourth of the share, as they are now
                float4 v[GI];
                double y[GI];
                auto fourth = [&](int f) __attribute__((always_inline)) {
                    asm volatile("" : "+v"(tq), "+v"(Ch));
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (f == q) {
#pragma unroll
                            for (int i = 0; i < GI; ++i) v[i] = residual(q * GI + i, draft_item(q * GI + i));
                        }
#pragma unroll
                    for (int i = 0; i < GI; ++i) y[i] = sum4(v[i]);
                };
                if (DEALT) {
                    // the wavefront of the crossing, then, by that one, the fourth of its share, the item and the token
                    const int ws = find_crossing(lane < NWAVES ? s_sum[slot][0][lane & (NWAVES - 1)] : 0.0, tau, lane, &crossing, &from);
                    owner = wave == (ws < 0 ? 0 : ws);
                    if (owner && ws >= 0) {
                        double sum = add_halves(add_rows(row_totals_scattered<4>(part, lane, which)));
                        int f = find_crossing((lane & 3) == 0 && lane < 16 ? sum : 0.0, tau, lane, &crossing, &from);
                        f = f < 0 ? 0 : f >> 2;
                        fourth(f);
                        sum = add_halves(add_rows(row_totals_scattered<GI>(y, lane, which)));
                        int is = find_crossing((lane & (REP - 1)) == 0 && lane < 16 ? sum : 0.0, tau, lane, &crossing, &from);
                        is = is < 0 ? 0 : is / REP;
#pragma unroll
                        for (int i = 1; i < GI; ++i)
                            if (i == is) v[0] = v[i];
                        d = search_piece(v[0], from, tau, tol, crossing, own.token(GI * f + is, 0), lane, &holder);
                    }
                } else {
                    // the fourth of the row, the item of the workgroup, and the wavefront, from totals of all of them: two barriers
                    double sum = add_halves(add_rows(row_totals_scattered<4>(part, lane, which)));
                    if ((lane & 3) == 0 && lane < 16) s_part[lane >> 2][wave] = sum;
                    __syncthreads();
                    auto over_waves = [&](const double *x) __attribute__((always_inline)) {
                        double t0 = x[0];
#pragma unroll
                        for (int w = 1; w < NWAVES; ++w) t0 += x[w];
                        return t0;
                    };
                    int f = find_crossing(lane < 4 ? over_waves(s_part[lane & 3]) : 0.0, tau, lane, &crossing, &from);
                    owner = f < 0 && wave == 0;
                    if (f >= 0) {
                        fourth(f);
                        sum = add_halves(add_rows(row_totals_scattered<GI>(y, lane, which)));
                        if ((lane & (REP - 1)) == 0 && lane < 16) s_item[lane / REP][wave] = sum;
                        __syncthreads();
                        int is = find_crossing(lane < GI ? over_waves(s_item[lane & (GI - 1)]) : 0.0, tau, lane, &crossing, &from);
                        is = is < 0 ? 0 : is;
                        const int ws = find_crossing(lane < NWAVES ? s_item[is][lane & (NWAVES - 1)] : 0.0, tau, lane, &crossing, &from);
                        owner = wave == (ws < 0 ? 0 : ws);
                        if (owner) {
#pragma unroll
                            for (int i = 1; i < GI; ++i)
                                if (i == is) v[0] = v[i];
                            d = search_piece(v[0], from, tau, tol, crossing, own.token(GI * f + is, 0), lane, &holder);
                        }
                    }
                }
                endpoint = __builtin_amdgcn_readlane(d.token, holder);
                if (__builtin_amdgcn_readlane(d.near, holder)) fl |= (uint32_t)MCSD_FLAG_NEAR_TIE_ENDPOINT;
            } else {
                // no distribution (a NaN logit): the last token that carries weight, reported
                if (t == 0) s_best = -1;
                int best = -1;
#pragma unroll
                for (int j = 0; j < ITEMS; ++j) {
                    const float4 r = residual(j, draft_item(j));
                    const float v[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (v[c] > 0.f) best = 4 * j + c;
                }
                __syncthreads();
                if (best >= 0) atomicMax(&s_best, own.token(best >> 2, lane) + (best & 3));
                __syncthreads();
                endpoint = s_best;
                fl |= (uint32_t)MCSD_FLAG_NEAR_TIE_ENDPOINT;
            }
            if (endpoint < 0 || endpoint >= V) endpoint = V - 1;
        }
        const VerifyParams *out = arguments();
        if (owner && naive && k > 0) {
            // multi-candidate naive sampling (the comparison rule of the ablation, Sec. 4.5): the
            // token just drawn from p is kept; a candidate equal to it is accepted, the first such
            const __amdgpu_buffer_rsrc_t rs = node_words(out->cand_tok);
            const int tok0 = __builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4, 0, 0), tok1 = __builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4, 256, 0);
            const unsigned long long m0 = __ballot(f0 && tok0 == endpoint && tok0 >= 0 && tok0 < V);
            const unsigned long long m1 = __ballot(f1 && tok1 == endpoint && tok1 >= 0 && tok1 < V);
            if (__ballot((f0 && (tok0 < 0 || tok0 >= V)) || (f1 && (tok1 < 0 || tok1 >= V)))) fl |= (uint32_t)MCSD_FLAG_BAD_TOKEN;
            acc_node = m0 ? __ffsll((long long)m0) - 1 : (m1 ? 63 + __ffsll((long long)m1) : -1);
            if (acc_node >= 0) endpoint = -1;
            if (out->ratio) {
                if (f0) out->ratio[nodes + lane] = NaN;
                if (f1) out->ratio[nodes + 64 + lane] = NaN;
            }
        }
        if (out->residual_out) {
            // Through a buffer resource (stores past the end of the row are dropped).  The offset of an item goes into
            // the per-thread offset, not into the scalar offset field: with a scalar register there, the compiler
            // inserts no wait between a 128-bit store and the next write to its data registers, and on this chip the
            // store then sent the next item's values for some lanes (seen as wrong residuals, in different
            // places from run to run).
            const __amdgpu_buffer_rsrc_t rs_out = row_resource(out->residual_out + rix * (size_t)V, V);
            const float inv = (A > 0.0) ? (float)(1.0 / A) : 0.f;
            asm volatile("" : "+v"(tq), "+v"(Ch));
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                if (j >= own.items) continue;
                // (nothing rejected: the weights as they are, a NaN among them too, which the clamp makes 0)
                const float4 r = rejected ? residual(j, draft_item(j)) : a[j];
                const int off = own.token(j, lane) * 4;
                if (ALIGNED) {
                    const u32x4 v = {__float_as_uint(r.x * inv), __float_as_uint(r.y * inv), __float_as_uint(r.z * inv), __float_as_uint(r.w * inv)};
                    __builtin_amdgcn_raw_buffer_store_b128(v, rs_out, off, 0, 0);
                } else {
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(r.x * inv), rs_out, off, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(r.y * inv), rs_out, off + 4, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(r.z * inv), rs_out, off + 8, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(r.w * inv), rs_out, off + 12, 0, 0);
                }
            }
        }
        if (owner && lane == 0) {
            out->acc_child[rix] = acc_node;
            out->endpoint[rix] = endpoint;
            out->flags[rix] = fl;
        }
    }
}

// one wavefront per sequence
__global__ __launch_bounds__(64) void walk_kernel(WalkParams w)
{
    walk_sequence(w, blockIdx.x);
}

template <int ITEMS, int VT, int LQ, int WGS, bool DEALT>
void launch_rows(VerifyParams p, hipStream_t stream)
{
    dim3 grid(1 + p.N, p.B), block(VT);
    p.ranked = (long)p.B * (1 + p.N) > 256 * WGS;        // more workgroups than start at once on 256 compute units
    if (p.V % 4 == 0)
        launch_kernel(K_VERIFY_ROWS, verify_rows_kernel<ITEMS, VT, LQ, WGS, DEALT, true>, grid, block, stream, p);
    else
        launch_kernel(K_VERIFY_ROWS, verify_rows_kernel<ITEMS, VT, LQ, WGS, DEALT, false>, grid, block, stream, p);
}

}  // namespace

WalkParams make_walk_params(const mcsd_verify_desc &d, const mcsd_verify_bufs &b)
{
    WalkParams w;
    w.B = d.B; w.N = d.N; w.gamma_max = d.gamma_max; w.flags = b.flags;
    w.acc_child = b.acc_child; w.endpoint = b.endpoint; w.cand_tok = b.cand_tok;
    w.n_accepted = b.n_accepted; w.accepted_path = b.accepted_path; w.out_tokens = b.out_tokens;
    return w;
}

int32_t launch_verify(const mcsd_verify_desc &d, const mcsd_verify_bufs &b, hipStream_t stream, bool with_walk)
{
    VerifyParams p;
    p.B = d.B; p.N = d.N; p.V = d.V; p.P = d.P; p.variant = d.variant; p.gamma_max = d.gamma_max;
    p.eps = d.near_tie_eps; p.per_seq = d.parent_per_seq;
    p.target_logits = b.target_logits; p.draft_logits = b.draft_logits;
    p.q_row = b.q_row; p.parent = b.parent; p.cand_tok = b.cand_tok;
    p.u_accept = b.u_accept; p.u_endpoint = b.u_endpoint; p.temperature = b.temperature;
    p.n_accepted = b.n_accepted; p.accepted_path = b.accepted_path; p.out_tokens = b.out_tokens;
    p.acc_child = b.acc_child; p.endpoint = b.endpoint; p.ratio = b.ratio; p.flags = b.flags;
    p.residual_out = b.residual_out;

    // Threads and the split between registers and LDS by the size of the row pair: up to 16384 tokens
    // everything in registers, several workgroups per compute unit; up to 32768 two per unit with 18 of
    // 32 items of the draft row in LDS; beyond, one per unit with the same split.  Measured for 16 x 61
    // rows of 32000 when a rejection still rewrote the row: 33.5 us; 512 threads with 9 of 16 items in LDS (128
    // registers, 16 spilled) 38.3 us; 1024 threads, all in registers, one workgroup per unit 42.5 us.
    // (Registers put aside in memory, per thread: 4 or 5 of the 128 where four wavefronts share a SIMD, 4 of the 256 of two per unit, 8 where
    // V is no multiple of four, 2 beyond 32768.)
    // With few rows nothing else loads beside a row, and two wavefronts per SIMD fill each other's waits:
    // 512 threads, both rows in registers, one workgroup per unit.  A call with its walk, trees of 4x2x2 whose candidates
    // are mostly rejected, from memory, two workgroups per unit / this: rows of 32000, 29 of them 20.4 / 16.1 us, 116 21.8 / 17.4, 261 27.2 / 21.9,
    // 348 28.0 / 26.9, 406 34.9 / 30.1, 435 35.5 / 32.1, 464 34.8 / 30.2, 522 36.1 / 36.0, 580 38.4 / 37.5, 976 (16 x 61) 48.7 / 52.6 (half of them argmax 36.0 / 39.5);
    // rows of 20000, 29 16.3 / 14.7, 261 21.5 / 20.1, 348 25.8 / 26.7, 435 26.5 / 27.3, 493 24.3 / 26.7, 580 28.8 / 32.8, 976 40.4 / 49.3.
    // One line between their crossings, at about 300 rows and 550.
    // Two per unit read the row in order (Share), the others dealt: that instance is the one bound by HBM.
    const long rows = (long)d.B * (1 + d.N);
    if (d.V <= 4096) launch_rows<4, 256, 0, 4, true>(p, stream);
    else if (d.V <= 8192) launch_rows<8, 256, 0, 4, true>(p, stream);
    else if (d.V <= 16384) launch_rows<8, 512, 0, 2, true>(p, stream);
    else if (d.V <= 32768 && rows <= 448) launch_rows<16, 512, 0, 1, true>(p, stream);
    else if (d.V <= 32768) launch_rows<32, 256, 18, 2, false>(p, stream);
    else launch_rows<32, 512, 18, 1, true>(p, stream);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error("verify_rows launch failed: %s", hipGetErrorString(e));
        return MCSD_E_HIP;
    }
    if (!with_walk) return MCSD_OK;
    launch_kernel(K_WALK, walk_kernel, dim3(d.B), dim3(64), stream, make_walk_params(d, b));
    e = hipGetLastError();
    if (e != hipSuccess) {
        set_error("walk launch failed: %s", hipGetErrorString(e));
        return MCSD_E_HIP;
    }
    return MCSD_OK;
}

}  // namespace mcsd
