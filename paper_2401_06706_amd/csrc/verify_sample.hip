// Multi-candidate speculative sampling on gfx950: Algorithm 1 (with replacement),
// Algorithm 2 (without replacement), the endpoint draws and the root-to-leaf walk.
//
// One workgroup owns one row of the tree (the root or a node).  Both logit rows of the node are read
// from HBM exactly once with 128-bit loads and stay on the compute unit, in registers and (the larger
// vocabularies) partly in LDS, for all k sequential accept/reject rounds; every round is one
// elementwise pass over the resident data plus one block reduction.
//
// Algorithm 2's removal of a rejected token from q needs no pass: that token's residual is already
// 0 and stays 0 whatever is subtracted from it later, so only Z_q changes, by exactly the fp32 weight
// of the token.  (A residual that vanished is put back without the removed tokens.)
//
// Instead of renormalising after each rejection the kernels carry an
// unnormalised residual a(x) and its sum A (p-hat = a / A), and the unnormalised
// draft weights e_q(x) with the running mass Z_q of the tokens not yet removed
// (q-bar = e_q / Z_q).  Algorithm 1/2's update p := max(0, p - q) / sum(...) then
// reads a := max(0, a - (A / Z_q) e_q), A := sum a, and the normaliser the paper
// divides by (the probability of the rejection, Appendix A) is A_new / A_old.
//
// The handful of numbers that decide an accept test - a(x), e_q(x) at the k
// candidate tokens - are tracked separately in fp64 by one thread per candidate,
// so that the comparison u <= min(1, p/q) is taken at far better than the 1e-6
// near-tie band; vocabulary-wide passes are fp32 with fp64 accumulation.
#include <math.h>

#include "mcsd_internal.h"
#include "vocab_row.h"

namespace mcsd {
namespace {

using namespace vocab;

constexpr float LOG2E_F = 1.44269504088896340736f;

struct VerifyParams {
    int B, N, V, P, variant, gamma_max, per_seq;
    float eps;
    const float *target_logits, *draft_logits;
    const int32_t *q_row, *parent, *cand_tok;
    const float *u_accept, *u_endpoint, *temperature;
    int32_t *n_accepted, *accepted_path, *out_tokens, *acc_child, *endpoint;
    float *ratio;
    uint32_t *flags;
    float *residual_out;
};

// 2^x in fp64 for x <= 0 (one thread per candidate token evaluates two of these): x = n + f with
// |f| <= 1/2, 2^f = exp(f ln 2) by its Taylor series to degree 13 (|f ln 2| <= 0.35: truncation
// below 1e-17), scaled by 2^n.  Arguments below -1000 return 0.
__device__ __forceinline__ double exp2_neg(double x)
{
    if (!(x > -1000.0)) return 0.0;
    const double n = rint(x);
    const double y = (x - n) * 0.69314718055994530942;
    double r = 1.0 / 6227020800.0;
    r = fma(r, y, 1.0 / 479001600.0);
    r = fma(r, y, 1.0 / 39916800.0);
    r = fma(r, y, 1.0 / 3628800.0);
    r = fma(r, y, 1.0 / 362880.0);
    r = fma(r, y, 1.0 / 40320.0);
    r = fma(r, y, 1.0 / 5040.0);
    r = fma(r, y, 1.0 / 720.0);
    r = fma(r, y, 1.0 / 120.0);
    r = fma(r, y, 1.0 / 24.0);
    r = fma(r, y, 1.0 / 6.0);
    r = fma(r, y, 0.5);
    r = fma(r, y, 1.0);
    r = fma(r, y, 1.0);
    return ldexp(r, (int)n);
}


// The residual row scaled by s, stored through a buffer resource (stores past the end of the row
// are dropped).  The offset of a piece goes into the per-thread offset, not into the scalar
// offset field: with a scalar register there, the compiler inserts no wait between a 128-bit
// store and the next write to its data registers, and on this chip the store then sent the
// next piece's values for some lanes (seen as wrong residuals, in different places from run to run).
template <int ITEMS, int VT, bool ALIGNED>
__device__ __forceinline__ void store_residual(float *dst, int V, const float4 (&a)[ITEMS], float s)
{
    const __amdgpu_buffer_rsrc_t rs_out = row_resource(dst, V);
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int off = threadIdx.x * 16 + i * (VT * 16);
        if (ALIGNED) {
            const u32x4 v = {__float_as_uint(a[i].x * s), __float_as_uint(a[i].y * s), __float_as_uint(a[i].z * s), __float_as_uint(a[i].w * s)};
            __builtin_amdgcn_raw_buffer_store_b128(v, rs_out, off, 0, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(a[i].x * s), rs_out, off, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(a[i].y * s), rs_out, off + 4, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(a[i].z * s), rs_out, off + 8, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(a[i].w * s), rs_out, off + 12, 0, 0);
        }
    }
}

// e_q of four logits, bit for bit what every pass (and the thread that tracks a candidate
// token) computes: subtraction first, then the scale, then v_exp_f32.
__device__ __forceinline__ float4 exp_weights(const float4 &z, float m, float c)
{
    return make_float4(__builtin_amdgcn_exp2f((z.x - m) * c), __builtin_amdgcn_exp2f((z.y - m) * c),
                       __builtin_amdgcn_exp2f((z.z - m) * c), __builtin_amdgcn_exp2f((z.w - m) * c));
}

// Gives token x (the same in all lanes) of a row the weight w; its own thread gets the weight it had.
template <int ITEMS, int VT>
__device__ __forceinline__ float set_token(float4 (&a)[ITEMS], int x, float w)
{
    const int item = (x >> 2) / VT, c = ((x >> 2) & (VT - 1)) == (int)threadIdx.x ? (x & 3) : -1;
    float was = 0.f;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        if (j == item) {
            float *v[4] = {&a[j].x, &a[j].y, &a[j].z, &a[j].w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c == e) { was = *v[e]; *v[e] = w; }
        }
    return was;
}

// A condition that is the same in all lanes though the compiler can not know it: as a scalar, so that
// the branch on it is one.
__device__ __forceinline__ bool uniform(bool c) { return __builtin_amdgcn_readfirstlane(c ? 1 : 0) != 0; }
__device__ __forceinline__ double uniform(double v) { return readlane_d(v, 0); }

// The sequence of rank y when the sampled sequences come before the argmax ones (each group in its
// own order), and its temperature.  Workgroups start in the order y, x, and a sampled sequence costs
// a workgroup about three times what an argmax sequence costs (two rows, exponentials, k dependent
// rounds against one row and an argmax): handed out first, the cheap ones fill the end of the launch.
// Every wavefront finds it by itself, without a barrier.  Batches above 512 keep their order.
__device__ __forceinline__ void ranked_sequence(const float *temperature, int B, int y, int lane, int *seq, float *T)
{
    if (B == 1 || B > 512) {
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

// One workgroup per tree row.  Both logit rows are read from HBM once and stay on the compute unit
// for all rounds: the target row in registers (as the unnormalised residual a), the draft row (as
// e_q) in registers up to item ITEMS - LQ and in LDS beyond.  LQ is chosen so that two workgroups
// share a compute unit (256 registers per thread, 80 KB of LDS each), one loading while the other
// computes: the two row pairs of 32000 tokens are 512 KB, as much as all registers of the unit.
//
// Bound: HBM in a batch (16 sequences of 61 rows, 8 of them argmax: 171 MB in 33.5 us = 5.1 TB/s;
// 42.5 us with one workgroup per unit), the vector units of one CU for a single sequence (256 threads,
// four rejections: 4 us until the rows are there, 3.7 us maxima, exponentials and sums, 1.9 us per
// rejection, of which fp64 conversions and additions are half, 2.3 us endpoint).
// 50001 tokens, 6 sequences of 29 rows: 30.5 us; 90 us when the draft row was streamed again for every
// pass.
template <int ITEMS, int VT, int LQ, int FULL, int WGS, bool ALIGNED>
__global__ __launch_bounds__(VT) __attribute__((amdgpu_waves_per_eu(WGS * VT / 256)))
void verify_rows_kernel(VerifyParams p)
{
    constexpr int NWAVES = VT / 64, RQ = ITEMS - LQ;
    using Row = Pieces<ITEMS, VT>;
    const int row = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int N = p.N, V = p.V;

    __shared__ float4 s_q[LQ ? LQ * VT : 1];            // [item - RQ][thread]: every thread reads only what is its own
    __shared__ double s_piece[4 * (ITEMS < 4 ? 4 : ITEMS) * NWAVES];
    __shared__ double s_sum[2][2][NWAVES];
    __shared__ float s_max[2][NWAVES];
    __shared__ int s_besti[NWAVES];
    __shared__ int s_tok[MCSD_MAX_NODES];
    __shared__ uint8_t s_kid[MCSD_MAX_NODES];
    __shared__ float s_u[MCSD_MAX_NODES], s_q32[MCSD_MAX_NODES];
    __shared__ double s_pa[MCSD_MAX_NODES], s_qa[MCSD_MAX_NODES];       // the logits of the candidates, then e_p and e_q in fp64
    // of the first 64 rejections (the pieces come last: every path to them from a round that reads s_beta
    // leads through the barrier of that round's sum)
    double *s_beta = s_piece;
    __shared__ Drawn s_drawn;

    int b;
    float T_of_b;
    ranked_sequence(p.temperature, p.B, blockIdx.y, lane, &b, &T_of_b);
    const int qr_of_row = p.q_row[(p.per_seq ? (size_t)b * (1 + N) : 0) + row];
    const int32_t *parent = p.parent + (p.per_seq ? (size_t)b * N : 0);
    const size_t rix = (size_t)b * (1 + N) + row;
    const float *zp_row = p.target_logits + rix * (size_t)V;
    const bool naive = (p.variant == MCSD_NAIVE);      // the draft row is not needed: candidates are only compared
    const float NaN = __int_as_float(0x7fc00000);

    // Requested ahead of the rows (memory answers in order): the parent array, by every wavefront for
    // itself, and by wavefront 0 the candidates; lane = node here.
    const int pa0 = lane < N ? parent[lane] : -2, pa1 = 64 + lane < N ? parent[64 + lane] : -2;
    int tok0 = -1, tok1 = -1;
    if (wave == 0) {
        if (lane < N) tok0 = p.cand_tok[(size_t)b * N + lane];
        if (64 + lane < N) tok1 = p.cand_tok[(size_t)b * N + 64 + lane];
    }
    __builtin_amdgcn_sched_barrier(0);
    // A row has a draft row iff q_row says so; whether it also has children is known a little later
    // (a mismatch is flagged, the row then counts as a leaf and the extra row is ignored).
    const int V4 = V & ~3;
    float4 a[ITEMS], eq[RQ];
    float4 tail_p, tail_q;
    request_pieces<ITEMS, VT, ALIGNED>(zp_row, V, t, a, tail_p);
    // (as scalars: the branches on them below are then scalar too)
    const float T = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(T_of_b)));
    const int qr = __builtin_amdgcn_readfirstlane(qr_of_row);
    const bool have_q = (qr >= 0 && qr < p.P) && (T != 0.f) && !naive;
    const float *zq_row = have_q ? p.draft_logits + ((size_t)b * p.P + qr) * (size_t)V : zp_row;
    if (have_q) {
        request_pieces<RQ, VT, ALIGNED>(zq_row, V, t, eq, tail_q);
        if (LQ) {
            // straight into LDS (16 bytes per lane, consecutive): no registers while in flight
            const __amdgpu_buffer_rsrc_t rs = row_resource(zq_row, ALIGNED ? V : V4);
            typedef __attribute__((address_space(3))) void *lds_ptr;
#pragma unroll
            for (int i = 0; i < LQ; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)(s_q + i * VT + 64 * wave), 16, t * 16, (RQ + i) * (VT * 16), 0, 2);
        }
    }

    const bool f0 = pa0 == row - 1, f1 = pa1 == row - 1;
    const Kids kids = {__ballot(f0), __ballot(f1)};
    uint32_t fl = 0u;
    int k = kids.count();
    if (k > 0 && (qr < 0 || qr >= p.P)) {
        // a row with children needs a draft row; a bad map is reported, never dereferenced
        k = 0;
        fl = (uint32_t)MCSD_FLAG_BAD_TREE;
    }
    if (wave == 0 && k > 0 && T != 0.f) {
        // candidate c (rank among the children) of the row: node, token, uniform and the two logits
        // (naive sampling reads neither draft logits nor u_accept)
        const bool v0 = f0 && tok0 >= 0 && tok0 < V && !naive, v1 = f1 && tok1 >= 0 && tok1 < V && !naive;
        const float u0 = (f0 && !naive) ? p.u_accept[(size_t)b * N + lane] : 0.f;
        const float u1 = (f1 && !naive) ? p.u_accept[(size_t)b * N + 64 + lane] : 0.f;
        const float p0 = v0 ? zp_row[tok0] : 0.f, q0 = v0 ? zq_row[tok0] : 0.f;
        const float p1 = v1 ? zp_row[tok1] : 0.f, q1 = v1 ? zq_row[tok1] : 0.f;
        if (f0) { const int c = kids.rank0(lane); s_kid[c] = lane; s_tok[c] = tok0; s_u[c] = u0; s_pa[c] = p0; s_qa[c] = q0; }
        if (f1) { const int c = kids.rank1(lane); s_kid[c] = 64 + lane; s_tok[c] = tok1; s_u[c] = u1; s_pa[c] = p1; s_qa[c] = q1; }
    }
    settle_pieces<ITEMS, VT, FULL, ALIGNED>(V, t, a, tail_p);

    if (T == 0.f) {
        // argmax sampling: lowest id on ties.  Ascending token order: a strict comparison keeps the
        // first of equal values; elements are named by their number in the thread (an inline constant).
        float bv = -INFINITY;
        int bc = -1;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const float v[4] = {a[j].x, a[j].y, a[j].z, a[j].w};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (v[c] > bv) { bv = v[c]; bc = 4 * j + c; }
        }
        int bi = bc >= 0 ? 4 * (t + VT * (bc >> 2)) + (bc & 3) : 0x7fffffff;
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
                if (c0) p.ratio[(size_t)b * N + lane] = NaN;
                if (c1) p.ratio[(size_t)b * N + 64 + lane] = NaN;
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
        const bool rounds = k > 0 && !naive;            // (then there is a draft row)
        float mp = row_max<ITEMS>(a), mq = -INFINITY;
        if (rounds) {
            settle_pieces<RQ, VT, (FULL < RQ ? FULL : RQ), ALIGNED>(V, t, eq, tail_q);
            mq = row_max<RQ>(eq);
            if (LQ) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // the part in LDS has arrived
#pragma unroll
                for (int i = 0; i < LQ; ++i) {
                    if (RQ + i >= FULL && 4 * VT * (RQ + i + 1) > V4) {  // uniform: the item that reaches past the row, and those behind it
                        const int e = 4 * (t + VT * (RQ + i));
                        if (e >= V4) s_q[i * VT + t] = (!ALIGNED && e == V4) ? tail_q : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
                    }
                    const float4 z = s_q[i * VT + t];
                    mq = max3_raw(max3_raw(mq, z.x, z.y), z.z, z.w);
                }
            }
        }
        mp = wave_max(mp);
        mq = wave_max(mq);
        if (lane == 63) { s_max[0][wave] = mp; s_max[1][wave] = mq; }
        __syncthreads();
        mp = s_max[0][0]; mq = s_max[1][0];
#pragma unroll
        for (int w = 1; w < NWAVES; ++w) { mp = fmaxf(mp, s_max[0][w]); mq = fmaxf(mq, s_max[1][w]); }
        mp = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(mp)));
        mq = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(mq)));

        if (rounds && wave < 2) {
            // e_p and e_q of the candidates in fp64, with the constants of the vector pass (float c2)
            // evaluated exactly; s_q32: e_q with the rounding of the vector passes
            const int c = 64 * wave + lane;
            if (c < k) {
                const double zp = s_pa[c], zq = s_qa[c];
                s_pa[c] = exp2_neg((zp - (double)mp) * (double)c2);
                s_qa[c] = exp2_neg((zq - (double)mq) * (double)c2);
                s_q32[c] = __builtin_amdgcn_exp2f(((float)zq - mq) * c2);
            }
        }
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) a[i] = exp_weights(a[i], mp, c2);        // a = e_p
        double A = 0.0, Zq = 0.0;
        // the sums of a and e_q over the workgroup, as scalars; one barrier (slot: 0 or 1 in turn)
        auto total = [&](double x, double y, int slot) __attribute__((always_inline)) {
            x = wave_sum(x);
            y = wave_sum(y);
            if (lane == 63) { s_sum[slot][0][wave] = x; s_sum[slot][1][wave] = y; }
            __syncthreads();
            double sx = 0.0, sy = 0.0;
#pragma unroll
            for (int w = 0; w < NWAVES; ++w) { sx += s_sum[slot][0][w]; sy += s_sum[slot][1][w]; }
            A = uniform(sx);
            Zq = uniform(sy);
        };
        if (rounds) {
            double part = 0.0, partq = 0.0;
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                part += sum4(a[i]);
                if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);     // (a few items at a time: more would not fit the registers)
            }
#pragma unroll
            for (int i = 0; i < RQ; ++i) {
                eq[i] = exp_weights(eq[i], mq, c2);
                partq += sum4(eq[i]);
                if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 0; i < LQ; ++i) {
                const float4 e = exp_weights(s_q[i * VT + t], mq, c2);
                s_q[i * VT + t] = e;
                partq += sum4(e);
                if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
            total(part, partq, 0);
            if (!(A > 0.0) || !isfinite(A) || !(Zq > 0.0) || !isfinite(Zq)) fl |= (uint32_t)MCSD_FLAG_NONFINITE;
        }

        int accepted = -1;
        if (rounds) {
            // Lane c of every wavefront follows candidate c in fp64 (in blocks of 64 candidates), so that
            // all of them take the same decisions without a barrier; a round costs the one of its sum.
            int my_tok = -1;
            double my_a = 0.0, my_q = 0.0;
            float my_u = 0.f, my_q32 = 0.f;             // my_q32: e_q with the rounding of the vector passes
            double z_base = Zq;
            int buf = 1;
            const bool removes = p.variant == MCSD_WITHOUT_REPLACEMENT;
            double kept_a = 0.0;                        // residual of tokens that have left q, put aside from the row (see below)
            int i = 0;
            bool acc;
            do {
                if ((i & 63) == 0) {
                    if (i > 0) __syncthreads();         // s_beta[63] is written behind the barrier of its own round
                    const int c = i + lane;
                    my_tok = -1;
                    my_a = my_q = 0.0;
                    if (c < k) {
                        my_tok = s_tok[c];
                        my_u = s_u[c];
                        if (my_tok >= 0 && my_tok < V) {
                            my_a = s_pa[c];
                            my_q = s_qa[c];
                            my_q32 = s_q32[c];
                            for (int j = 0; j < i; ++j) {       // the rejections before this block
                                my_a = fmax(0.0, my_a - s_beta[j] * my_q);
                                if (removes && s_tok[j] == my_tok) { my_q = 0.0; my_q32 = 0.f; }
                            }
                        }
                    }
                }
                const int tok = __builtin_amdgcn_readlane(my_tok, i & 63);
                const double ai = readlane_d(my_a, i & 63), qi = readlane_d(my_q, i & 63);
                const double u = (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_u), i & 63));
                const bool valid = tok >= 0 && tok < V;
                double ratio;
                if (!valid) {
                    ratio = 0.0;
                    fl |= (uint32_t)MCSD_FLAG_BAD_TOKEN;
                } else if (qi > 0.0) {
                    ratio = (ai * Zq) / (A * qi);
                    if (!(ratio < 1.0)) ratio = 1.0;
                } else {
                    ratio = ai > 0.0 ? 1.0 : 0.0;
                    fl |= (uint32_t)MCSD_FLAG_ZERO_DRAFT_PROB;
                }
                // (a token of probability zero - a duplicate of a rejected one, Sec. 3.2 - is never
                // accepted, also not by a uniform of exactly 0 from outside the open interval)
                acc = uniform((ratio > 0.0) && (u <= ratio));
                if (fabs(u - ratio) < (double)p.eps) fl |= (uint32_t)MCSD_FLAG_NEAR_TIE_ACCEPT;
                if (p.ratio && t == 0) p.ratio[(size_t)b * N + s_kid[i]] = (float)ratio;
                if (!acc) {
                    // rejected: a := max(0, a - beta e_q) with beta = A / Z_q in fp64, applied as a
                    // two-term float product so that no common rounding of beta biases the sum; 0 <= a <= 1,
                    // so that the max is the clamp of the second product.  (The
                    // token that leaves q keeps its e_q in the row: its residual is 0 now and stays 0
                    // whatever is subtracted later; what is added below is taken from it again.)
                    const double beta = (Zq > 0.0) ? A / Zq : 0.0;   // nothing left in q: the residual is p itself
                    float bh = (float)beta;
                    float bl = (float)(beta - (double)bh);
                    const bool last = i + 1 == k, remove = valid && removes;
                    const double A_old = A, Zq_old = Zq;
                    bool vanished = false;
                    for (;;) {
                        double part = 0.0;
                        int tq = t;
                        asm volatile("" : "+v"(tq));    // (the reads of s_q stay inside the loop over the rounds)
#pragma unroll
                        for (int j = 0; j < ITEMS; ++j) {
                            const float4 e = j < RQ ? eq[j < RQ ? j : 0] : s_q[(j < RQ ? 0 : j - RQ) * VT + tq];
                            a[j].x = __builtin_amdgcn_fmed3f(fmaf(-bl, e.x, fmaf(-bh, e.x, a[j].x)), 0.f, 1.f);
                            a[j].y = __builtin_amdgcn_fmed3f(fmaf(-bl, e.y, fmaf(-bh, e.y, a[j].y)), 0.f, 1.f);
                            a[j].z = __builtin_amdgcn_fmed3f(fmaf(-bl, e.z, fmaf(-bh, e.z, a[j].z)), 0.f, 1.f);
                            a[j].w = __builtin_amdgcn_fmed3f(fmaf(-bl, e.w, fmaf(-bh, e.w, a[j].w)), 0.f, 1.f);
                            part += sum4(a[j]);
                            if ((j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
                        }
                        total(part, 0.0, buf);
                        A += kept_a;
                        buf ^= 1;                       // (the next writers can not overtake a reader of this one)
                        if (A > 0.0 || vanished) break;
                        // max(0, p - q) vanished everywhere, which a rejection excludes in exact arithmetic
                        // (it needs p = q) and rounding or a bad candidate can produce: p stays as it
                        // was.  With every a(x) <= beta e_q(x) and equal sums, the old a is beta e_q:
                        // the same pass with the sign turned, on the zeros that are left.
                        vanished = true;
                        bh = -bh;
                        bl = -bl;
                    }
                    Zq = Zq_old;
                    if (vanished) {
                        A = A_old;
                        fl |= (uint32_t)MCSD_FLAG_ZERO_RESIDUAL;
                    } else {
                        my_a = fmax(0.0, my_a - beta * my_q);
                    }
                    if (t == 0 && !last && i < 64) s_beta[i] = vanished ? 0.0 : beta;      // (0: the candidates' track did not move)
                    if (remove) {
                        // Z_q loses exactly the fp32 weight that its sum contained
                        Zq -= (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_q32), i & 63));
                        Zq = uniform(Zq);
                        if (!last && uniform(Zq < z_base * 0x1p-16)) {
                            // little of the mass is left and the difference has lost digits: the sum
                            // again without the removed tokens, from memory (rare; a pass over the
                            // resident row here would cost every row registers)
                            const __amdgpu_buffer_rsrc_t rs = row_resource(zq_row, V);
                            double partq = 0.0;
#pragma unroll 1
                            for (int e0 = t; e0 < V; e0 += VT) {
                                const float w = __builtin_amdgcn_exp2f((__uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, e0 * 4, 0, 0)) - mq) * c2);
                                bool in = true;
#pragma unroll 1
                                for (int n = 0; n <= i; ++n) in &= s_tok[n] != e0;
                                if (in) partq += (double)w;
                            }
                            const double A_now = A;
                            total(0.0, partq, buf);
                            buf ^= 1;
                            A = A_now;
                            z_base = Zq;
                        }
                    }
                    if (remove && my_tok == tok) { my_q = 0.0; my_q32 = 0.f; }
                    if (uniform(removes && (vanished || (valid && ratio >= 1.0)))) {
                        // Put back, the row holds beta e_q for tokens that had left q and have p = 0.  And the
                        // token just rejected leaves q with some of its p left, or all (so does one that
                        // only a uniform above 1 rejects): no later rejection may lower that.
#pragma unroll 1
                        for (int n = vanished ? 0 : i; n <= i; ++n) {
                            const int x = __builtin_amdgcn_readfirstlane(s_tok[n]);
                            if (n == i && t == 0 && !valid) s_u[i] = 0.f;
                            if (x < 0 || x >= V) continue;
                            const float was = set_token<ITEMS, VT>(a, x, 0.f);
                            if (n == i && ((x >> 2) & (VT - 1)) == t) s_u[i] = was;      // (its uniform has been used)
                        }
                        __syncthreads();
                        const double was = uniform((double)s_u[i]);
                        if (was > 0.0 && t == 0) s_q32[i] = -1.f;      // marked (its weight has been used)
                        kept_a += was;
                    }
                }
            } while (!acc && ++i < k);
            if (acc) accepted = i;
            if (kept_a > 0.0) {
                __syncthreads();
#pragma unroll 1
                for (int n = 0; n < k; ++n)
                    if (uniform(s_q32[n] < 0.f)) set_token<ITEMS, VT>(a, __builtin_amdgcn_readfirstlane(s_tok[n]), s_u[n]);
            }
            // candidates after the accepted one were never tested
            if (p.ratio && accepted >= 0 && wave == 0)
                for (int c = accepted + 1 + lane; c < k; c += 64) p.ratio[(size_t)b * N + s_kid[c]] = NaN;
        }

        int endpoint = -1;
        if (accepted < 0) {
            const double u = (double)p.u_endpoint[rix];
            Row::store(a, lane, wave, s_piece);
            __syncthreads();
            Row P;
            P.read(s_piece, lane);
            const double incl = P.scan();
            if (!rounds) {
                A = readlane_d(incl, 63);
                if (!(A > 0.0) || !isfinite(A)) fl |= (uint32_t)MCSD_FLAG_NONFINITE;
            }
            if (isfinite(A)) {
                draw_token<ITEMS, VT>(a, P, incl, u * A, (double)p.eps * A, lane, wave, &s_drawn);
            } else {
                // no distribution (a NaN logit): the last token that carries weight, reported
                if (t == 0) { s_drawn.token = -1; s_drawn.near = 1; }
                int best = -1;
#pragma unroll
                for (int j = 0; j < ITEMS; ++j) {
                    const float v[4] = {a[j].x, a[j].y, a[j].z, a[j].w};
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (v[c] > 0.f) best = 4 * j + c;
                }
                __syncthreads();
                if (best >= 0) atomicMax(&s_drawn.token, 4 * (t + VT * (best >> 2)) + (best & 3));
            }
            __syncthreads();
            endpoint = s_drawn.token;
            if (s_drawn.near) fl |= (uint32_t)MCSD_FLAG_NEAR_TIE_ENDPOINT;
            if (endpoint < 0 || endpoint >= V) endpoint = V - 1;
        }
        int acc_node = accepted >= 0 ? s_kid[accepted] : -1;
        if (naive && k > 0) {
            // multi-candidate naive sampling (the comparison rule of the ablation, Sec. 4.5): the
            // token just drawn from p is kept; a candidate equal to it is accepted, the first such
            const unsigned long long m0 = __ballot(f0 && tok0 == endpoint && tok0 >= 0 && tok0 < V);
            const unsigned long long m1 = __ballot(f1 && tok1 == endpoint && tok1 >= 0 && tok1 < V);
            if (__ballot((f0 && (tok0 < 0 || tok0 >= V)) || (f1 && (tok1 < 0 || tok1 >= V)))) fl |= (uint32_t)MCSD_FLAG_BAD_TOKEN;
            acc_node = m0 ? __ffsll((long long)m0) - 1 : (m1 ? 63 + __ffsll((long long)m1) : -1);      // (right in wavefront 0, which writes it)
            if (acc_node >= 0) endpoint = -1;
            if (p.ratio && wave == 0) {
                if (f0) p.ratio[(size_t)b * N + lane] = NaN;
                if (f1) p.ratio[(size_t)b * N + 64 + lane] = NaN;
            }
        }
        if (p.residual_out) {
            const float inv = (A > 0.0) ? (float)(1.0 / A) : 0.f;
            store_residual<ITEMS, VT, ALIGNED>(p.residual_out + rix * (size_t)V, V, a, inv);
        }
        if (t == 0) {
            p.acc_child[rix] = acc_node;
            p.endpoint[rix] = endpoint;
            p.flags[rix] = fl;
        }
    }
}

// one wavefront per sequence
__global__ __launch_bounds__(64) void walk_kernel(WalkParams w)
{
    walk_sequence(w, blockIdx.x);
}

template <int ITEMS, int VT, int LQ, int FULL, int WGS>
void launch_rows(const VerifyParams &p, hipStream_t stream)
{
    dim3 grid(1 + p.N, p.B), block(VT);
    if (p.V % 4 == 0)
        launch_kernel(K_VERIFY_ROWS, verify_rows_kernel<ITEMS, VT, LQ, FULL, WGS, true>, grid, block, stream, p);
    else
        launch_kernel(K_VERIFY_ROWS, verify_rows_kernel<ITEMS, VT, LQ, FULL, WGS, false>, grid, block, stream, p);
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
    // rows of 32000: 33.5 us; 512 threads with 9 of 16 items in LDS (128 registers, 16 spilled) 38.3 us;
    // 1024 threads, all in registers, one workgroup per unit 42.5 us.
    // With few rows nothing else loads beside a row, and two wavefronts per SIMD fill each other's waits:
    // 512 threads, both rows in registers (175), one workgroup per unit.  Rows of 32000, a call with its walk,
    // two workgroups per unit / this: 29 rows 19.1 / 16.8 us, 116 24.7 / 21.8, 261 26.8 / 23.8, 340 31.3 / 27.6,
    // 348 32.4 / 28.7, 464 36.6 / 37.1, 976 36.4 / 42.6 (1024 threads: 18.8, 24.4, 26.8, 29.2, 31.1, 38.7, 45.4).
    const long rows = (long)d.B * (1 + d.N);
    if (d.V <= 4096) launch_rows<4, 256, 0, 0, 4>(p, stream);
    else if (d.V <= 8192) launch_rows<8, 256, 0, 4, 4>(p, stream);
    else if (d.V <= 16384) launch_rows<8, 512, 0, 4, 2>(p, stream);
    else if (d.V <= 32768 && rows <= 448) launch_rows<16, 512, 0, 8, 1>(p, stream);
    else if (d.V <= 32768) launch_rows<32, 256, 18, 16, 2>(p, stream);
    else launch_rows<32, 512, 18, 16, 1>(p, stream);
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
