// Draft-side candidate sampling on gfx950 (Sec. 3.1 of the paper; q-bar of Eq. (1) when the
// candidates are drawn without replacement).
//
// One workgroup owns one row of the tree that has children.  The draft logit row is read
// from HBM once with 128-bit loads and stays in registers; after one max and one exp/sum pass
// the k draws are k inverse-CDF searches over the resident weights (fp64, one barrier each, see
// Pieces in vocab_row.h).  Without replacement the drawn token's weight leaves the total of its
// piece and the mass, which is q-bar of Eq. (1) without a renormalising pass: the search compares
// against u times the remaining mass.  At temperature 0 the candidates are the k largest
// logits: k rounds of a workgroup arg max (lowest id on ties), each removing its winner.
//
// Bound by HBM once two rows fit a compute unit, one loading while the other computes: 16 x 45 rows
// of 32000 tokens (92 MB, 8 sequences greedy) in 20.7 us = 4.4 TB/s, 36.0 us with one row per unit
// (255 registers) and six barriers per draw.
#include <math.h>

#include "mcsd_internal.h"
#include "vocab_row.h"

namespace mcsd {
namespace {

using namespace vocab;

constexpr float LOG2E_F = 1.44269504088896340736f;

struct DraftParams {
    int B, N, V, P, variant, per_seq;
    float eps;
    const float *draft_logits;
    const int32_t *q_row, *parent;
    const float *u_draw, *temperature;
    int32_t *cand_tok;
    uint32_t *flags;
};

template <int ITEMS, int VT, int FULL, int WGS, bool ALIGNED>
__global__ __launch_bounds__(VT) __attribute__((amdgpu_waves_per_eu(WGS * VT / 256)))
void draft_rows_kernel(DraftParams p)
{
    constexpr int NWAVES = VT / 64;
    using Row = Pieces<ITEMS, VT>;
    const int row = blockIdx.x, b = blockIdx.y;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int N = p.N, V = p.V;

    __shared__ double s_piece[4 * (ITEMS < 4 ? 4 : ITEMS) * NWAVES];
    __shared__ float s_max[NWAVES];
    __shared__ int s_kid[MCSD_MAX_NODES];
    __shared__ float s_u[MCSD_MAX_NODES];
    __shared__ Drawn s_drawn[MCSD_MAX_NODES];
    __shared__ double s_rest;
    __shared__ float s_bestv[2][NWAVES];
    __shared__ int s_besti[2][NWAVES];

    // Every wavefront reads the parent array itself, ahead of the row: memory answers in order, so the
    // children are known while the row is still on its way, and no barrier is needed for them.
    const int qr = __builtin_amdgcn_readfirstlane(p.q_row[(p.per_seq ? (size_t)b * (1 + N) : 0) + row]);
    const int32_t *parent = p.parent + (p.per_seq ? (size_t)b * N : 0);
    const float T = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(p.temperature[b])));   // a scalar branch below
    const bool have_q = qr >= 0 && qr < p.P;
    const int pa0 = lane < N ? parent[lane] : -2, pa1 = 64 + lane < N ? parent[64 + lane] : -2;
    float u0 = 0.f, u1 = 0.f;
    if (wave == 0 && T != 0.f) {
        const float *u = p.u_draw + (size_t)b * N;
        if (lane < N) u0 = u[lane];
        if (64 + lane < N) u1 = u[64 + lane];
    }
    __builtin_amdgcn_sched_barrier(0);
    float4 a[ITEMS];
    // requested before it is known whether this tree row has children: in a well-formed input q_row
    // marks exactly the rows that do
    if (have_q) load_pieces<ITEMS, VT, FULL, ALIGNED>(p.draft_logits + ((size_t)b * p.P + qr) * (size_t)V, V, t, a);

    const Kids kids = {__ballot(pa0 == row - 1), __ballot(pa1 == row - 1)};
    const int k = kids.count();
    if (k == 0) return;
    const bool f0 = pa0 == row - 1, f1 = pa1 == row - 1;
    if (!have_q || k > V) {
        // children without a draft row (or more children than tokens): reported, nothing drawn
        if (wave == 0) {
            if (f0) { p.cand_tok[(size_t)b * N + lane] = -1; p.flags[(size_t)b * N + lane] = (uint32_t)MCSD_FLAG_BAD_TREE; }
            if (f1) { p.cand_tok[(size_t)b * N + 64 + lane] = -1; p.flags[(size_t)b * N + 64 + lane] = (uint32_t)MCSD_FLAG_BAD_TREE; }
        }
        return;
    }
    if (wave == 0) {
        if (f0) { s_kid[kids.rank0(lane)] = lane; s_u[kids.rank0(lane)] = u0; }
        if (f1) { s_kid[kids.rank1(lane)] = 64 + lane; s_u[kids.rank1(lane)] = u1; }
    }

    if (T == 0.f) {
        // Every wavefront keeps the best of its own elements; a round removes the winner, and only the
        // wavefront that held it looks through its elements again.  Elements are named by their number
        // in the thread (4 item + component, an inline constant), not by their token.
        auto token_of = [&](int code) { return 4 * (t + VT * (code >> 2)) + (code & 3); };
        constexpr int NONE = 0x7fffffff;
        const float gone = __int_as_float(0x7fc00000);      // (a NaN never wins a comparison)
        bool inf_too = false;               // a logit of -inf may win (once nothing above it is left)
        // The elements are kept in groups of 16, each with its best, so that a removal costs one group.
        constexpr int GI = ITEMS < 4 ? ITEMS : 4, NG = ITEMS / GI, ALL = -1, CLEAN = -2;
        float gv[NG];
        int gc[NG];
        int dirty = ALL;                    // the group to look through again (uniform)
        float wv = -INFINITY;               // the wavefront's best
        int wi = NONE, buf = 0, gone_code = -1;
        for (int i = 0; i < k;) {
            if (dirty != CLEAN) {
                float bv = -INFINITY;
                int bc = -1;
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    if (dirty == ALL || dirty == g) {
                        // ascending token order: a strict comparison keeps the lowest id among equal values
                        gv[g] = -INFINITY;
                        gc[g] = -1;
#pragma unroll
                        for (int j = g * GI; j < (g + 1) * GI; ++j) {
                            float v[4] = {a[j].x, a[j].y, a[j].z, a[j].w};
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                if (gone_code == 4 * j + c) v[c] = gone;
                                if (v[c] > gv[g]) { gv[g] = v[c]; gc[g] = 4 * j + c; }
                            }
                            a[j] = make_float4(v[0], v[1], v[2], v[3]);
                        }
                    }
                    if (gv[g] > bv) { bv = gv[g]; bc = gc[g]; }
                }
                if (inf_too && bc < 0) {
#pragma unroll
                    for (int j = ITEMS - 1; j >= 0; --j) {
                        const float v[4] = {a[j].x, a[j].y, a[j].z, a[j].w};
#pragma unroll
                        for (int c = 3; c >= 0; --c)
                            if (v[c] == -INFINITY) bc = 4 * j + c;
                    }
                    if (bc >= 0 && token_of(bc) >= V) bc = -1;      // only the padding past V is left
                }
                wv = bv;
                wi = bc >= 0 ? token_of(bc) : NONE;
                wave_argmax(wv, wi);
                gone_code = -1;
            }
            if (lane == 0) { s_bestv[buf][wave] = wv; s_besti[buf][wave] = wi; }
            __syncthreads();
            float rv = s_bestv[buf][0];
            int ri = s_besti[buf][0];
#pragma unroll
            for (int w = 1; w < NWAVES; ++w) {
                const float ov = s_bestv[buf][w];
                const int oi = s_besti[buf][w];
                if (ov > rv || (ov == rv && oi < ri)) { rv = ov; ri = oi; }
            }
            ri = __builtin_amdgcn_readfirstlane(ri);
            buf ^= 1;                       // (the next round's writers can not overtake a reader of this one)
            if (ri == NONE && !inf_too) {
                // nothing above -inf is left (every wavefront sees the same): once more, with -inf allowed
                inf_too = true;
                dirty = ALL;
                continue;
            }
            // nothing comparable left (only NaN logits remain): reported, token 0 handed out
            const bool none = (ri == NONE);
            if (none) ri = 0;
            if (t == 0) {
                p.cand_tok[(size_t)b * N + s_kid[i]] = ri;
                p.flags[(size_t)b * N + s_kid[i]] = none ? (uint32_t)MCSD_FLAG_NONFINITE : 0u;
            }
            ++i;
            // the winner leaves the row (ids are unique, one thread owns it)
            const int owner = (ri >> 2) & (VT - 1);
            const int code = ((ri >> 2) / VT) * 4 + (ri & 3);
            dirty = (owner >> 6) == wave ? code / (4 * GI) : CLEAN;
            if (owner == t) gone_code = code;
        }
    }
    // (no return above: with one, the compiler keeps the logits of the other path alive beside the
    // weights of this one, twice the registers)
    if (T != 0.f) {
        const float c2 = (1.0f / T) * LOG2E_F;
        const float wm = wave_max(row_max<ITEMS>(a));
        if (lane == 63) s_max[wave] = wm;
        __syncthreads();
        float m = s_max[0];
#pragma unroll
        for (int w = 1; w < NWAVES; ++w) m = fmaxf(m, s_max[w]);
        // a = e_q, and the totals of its pieces
#pragma unroll
        for (int i0 = 0; i0 < ITEMS; i0 += 4) {
            double x[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int i = 0; i < 4 && i0 + i < ITEMS; ++i) {
                float4 &z = a[i0 + i];
                z.x = __builtin_amdgcn_exp2f((z.x - m) * c2);
                z.y = __builtin_amdgcn_exp2f((z.y - m) * c2);
                z.z = __builtin_amdgcn_exp2f((z.z - m) * c2);
                z.w = __builtin_amdgcn_exp2f((z.w - m) * c2);
                x[i] = sum4(z);
            }
            Row::store4(x, i0, lane, wave, s_piece);
            __builtin_amdgcn_sched_barrier(0);      // (four items at a time: the sums in flight would not fit the registers)
        }
        __syncthreads();
        Row P;
        P.read(s_piece, lane);
        double incl = P.scan();
        double Z = readlane_d(incl, 63);
        const double least = Z * 0x1p-20;
        const bool finite = (Z > 0.0) && (Z < INFINITY);
        for (int i = 0; i < k; ++i) {
            const int node = s_kid[i];
            const bool ok = finite && Z > 0.0;
            Drawn d = {0, 0.f, 0};
            if (ok) {
                draw_token<ITEMS, VT>(a, P, incl, (double)s_u[i] * Z, (double)p.eps * Z, lane, wave, &s_drawn[i], s_drawn, p.variant == MCSD_WITHOUT_REPLACEMENT ? i : 0);
                __syncthreads();                // (a slot per draw: the next writer can not overtake a reader of this one)
                d = s_drawn[i];
                if (d.token < 0 || d.token >= V) d.token = V - 1;
            }
            if (t == 0) {
                p.cand_tok[(size_t)b * N + node] = d.token;
                p.flags[(size_t)b * N + node] = (d.near ? (uint32_t)MCSD_FLAG_NEAR_TIE_DRAW : 0u) | (ok ? 0u : (uint32_t)MCSD_FLAG_NONFINITE);
            }
            if (p.variant == MCSD_WITHOUT_REPLACEMENT && i + 1 < k && ok) {
                // q-bar of Eq. (1): the drawn token's weight leaves its piece and the mass (draw_token skips
                // the token itself; taking it out of its register in this loop would cost a copy of the row)
                const bool little = P.remove(d.token, d.weight, lane);
                Z -= (double)d.weight;
                if (__builtin_expect(little, 0)) {
                    // what is left of the piece, from its tokens: a rest of roundings could be drawn in their place
                    const int j = d.token >> 8;
                    if (j % NWAVES == wave) {
                        const double rest = wave_sum(sum4(piece_values<ITEMS, VT>(a, j, lane, s_drawn, i + 1)));
                        if (lane == 63) s_rest = rest;
                    }
                    __syncthreads();            // (the next writer is behind the barrier of another draw)
                    P.set(j, s_rest, lane);
                }
                incl = P.scan();
                if (__builtin_expect(Z < least, 0)) Z = readlane_d(incl, 63);       // (likewise)
            }
        }
    }
}

template <int ITEMS, int VT, int FULL, int WGS>
void launch_rows(const DraftParams &p, hipStream_t stream)
{
    dim3 grid(1 + p.N, p.B), block(VT);
    if (p.V % 4 == 0)
        launch_kernel(K_DRAFT_ROWS, draft_rows_kernel<ITEMS, VT, FULL, WGS, true>, grid, block, stream, p);
    else
        launch_kernel(K_DRAFT_ROWS, draft_rows_kernel<ITEMS, VT, FULL, WGS, false>, grid, block, stream, p);
}

}  // namespace

int32_t launch_draft_sample(const mcsd_draft_desc &d, const mcsd_draft_bufs &b, hipStream_t stream)
{
    DraftParams p;
    p.B = d.B; p.N = d.N; p.V = d.V; p.P = d.P; p.variant = d.variant; p.eps = d.near_tie_eps; p.per_seq = d.parent_per_seq;
    p.draft_logits = b.draft_logits; p.q_row = b.q_row; p.parent = b.parent;
    p.u_draw = b.u_draw; p.temperature = b.temperature; p.cand_tok = b.cand_tok; p.flags = b.flags;
    // The row stays in registers, 64 per thread at most: with the rest that is 104, so that two rows of
    // up to 32768 tokens share a compute unit.  Measured at 16 x 45 rows of 32000: 512 threads 20.7 us,
    // 1024 threads with half the registers 29.3 us (one row per unit), 256 threads with twice as many
    // 21.4 us (three rows, but longer rounds: 16 greedy candidates 47 us against 33 us).
    if (d.V <= 4096) launch_rows<4, 256, 0, 4>(p, stream);
    else if (d.V <= 8192) launch_rows<8, 256, 4, 4>(p, stream);
    else if (d.V <= 16384) launch_rows<8, 512, 4, 2>(p, stream);
    else if (d.V <= 32768) launch_rows<16, 512, 8, 2>(p, stream);
    else launch_rows<16, 1024, 8, 1>(p, stream);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error("draft_rows launch failed: %s", hipGetErrorString(e));
        return MCSD_E_HIP;
    }
    return MCSD_OK;
}

}  // namespace mcsd
