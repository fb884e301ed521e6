// Tree attention (Sec. 3.3 of the paper) for the storage types and head dimensions that the
// d = 128 bf16 kernels do not take, and for the launches of theirs that leave the chip half idle, on the
// matrix cores of gfx950.
//
//   tree_attn_bf16_kernel  bf16 storage, d a multiple of 8 up to 256 (padded to 64, 128 or 256)
//   tree_attn_f32_kernel   fp32 storage, d a multiple of 4 up to 256 (same paddings)
//
// In both, a lane of S^T = K Q^T holds scores of one query row, which is the B operand layout of
// O^T += V^T P^T: the weights never leave their lane.  The fp32 kernel multiplies in fp32
// (v_mfma_f32_16x16x4_f32); the bf16 kernel feeds PV with two bf16 terms per weight where d != 128, which hold
// it to 2^-17 (see weight_hi_bits), and with one at d = 128, as the other kernels for it.
#include <type_traits>

#include "attn_common.h"

namespace mcsd {
namespace {

// Where a tile of keys lies: K and V rows back to back from kb / vb, `bytes` of them valid (rows
// past the end read as zero through the buffer resource, 0 = nothing is read).
struct TileSrc {
    const char *kb, *vb;
    uint32_t bytes;
};

// The keys of a sequence: ceil(L / KW) prefix tiles, then ceil(N / KW) tree tiles.  All arguments
// are wave-uniform.  Tiles at or past t_end are empty, which keeps every request unconditional.
template <int KW>
__device__ __forceinline__ TileSrc tile_source(const AttnParams &p, int b, int g, int L, int tiles_prefix, int t, int t_end, uint32_t row_bytes)
{
    TileSrc s;
    const size_t kv_head = (size_t)b * p.H_kv + g;
    s.kb = static_cast<const char *>(p.k_tree);
    s.vb = static_cast<const char *>(p.v_tree);
    s.bytes = 0u;
    if (t >= t_end) return s;
    size_t row;
    if (t < tiles_prefix) {
        const int key = t * KW;
        if (p.block_table) {
            // an entry outside the pool never leaves it
            int blk = p.block_table[(size_t)b * p.max_pages + key / p.page_size];
            blk = __builtin_amdgcn_readfirstlane(min(max(blk, 0), p.n_pages - 1));
            row = ((size_t)blk * p.H_kv + g) * (size_t)p.page_size + (size_t)(key % p.page_size);
        } else {
            row = kv_head * (size_t)p.L_stride + (size_t)key;
        }
        s.kb = static_cast<const char *>(p.k_prefix);
        s.vb = static_cast<const char *>(p.v_prefix);
        s.bytes = (uint32_t)min(KW, L - key) * row_bytes;
    } else {
        const int node = (t - tiles_prefix) * KW;
        row = kv_head * (size_t)p.N + (size_t)node;
        s.bytes = (uint32_t)min(KW, p.N - node) * row_bytes;
    }
    s.kb += row * row_bytes;
    s.vb += row * row_bytes;
    return s;
}

constexpr uint32_t OFF_NOWHERE = 0x7fffffffu;       // beyond every extent: reads as zero

// The prefix rows of a (sequence, KV head) are read through one buffer resource: a contiguous cache, whose offsets stay
// far from 32 bits.
__host__ __device__ __forceinline__ bool one_resource(const AttnParams &p, uint32_t row_bytes)
{
    return !p.block_table && (uint64_t)p.L_stride * row_bytes <= 0x40000000u;
}

// ------------------------------------------------------------------------------ bf16
// A weight p >= 0 as hi + lo, both bf16: hi is p cut to bf16, taken one step lower where that cut
// would be exact, lo the rest rounded to bf16.  |hi + lo - p| <= 2^-17 p (hi alone: 2^-8), so
// that PV rounds far below the bf16 output; and lo > 0 whenever p > 0, so that a weight times an
// infinite value stays infinite instead of meeting 0 x inf in the second term.
__device__ __forceinline__ uint32_t weight_hi_bits(float p)
{
    return __builtin_elementwise_sub_sat(__float_as_uint(p), 1u) & 0xffff0000u;
}

// 16 bytes per lane from memory into LDS, lane after lane from `to` on (the same in all lanes).  Zeros from beyond the resource.
__device__ __forceinline__ void load_into_lds(__amdgpu_buffer_rsrc_t rs, uint32_t *to, uint32_t lane_offset, uint32_t offset)
{
    typedef __attribute__((address_space(3))) void *lds_ptr;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr)to, 16, lane_offset, offset, 0, 0);
}

// Workgroup of NW waves, one unit (sequence, KV head, row tile) with all of its keys, DS of the output
// columns.  Wave (rh, ks) owns 16 MT query rows and every KS-th tile; the TS tiles of a step are loaded
// one step ahead into registers, by all threads together or, where every wave has a tile to itself, by
// that wave without a barrier in the loop.  Those of all threads go through LDS in their natural order
// with row pitches against bank conflicts (K: 4 words, V: 8 words past a multiple of 32); a wave's own go straight
// into LDS (see OWN).  V is read back with the transposing LDS load.  The streams meet in LDS at the
// end: no memory besides the arguments, so that calls on several streams share nothing, and the
// bits of a result depend on the arguments alone.  (Which instantiation: launch_attn_any and, for d = 128, make_attn_plan.)
// Bound, a wave with its own tiles, by the instructions of two waves per SIMD and by LDS, behind 6 to 7 us of launch, first tiles,
// masks and epilogue: with all tiles read from L1 a launch takes as long, without exponentials 0.6 us less of 13.  Measured (d 64, 8 sequences of
// 200..2000 tokens, GQA 32/8, 28 nodes): one workgroup per (node, head) on the vector units, every one
// reading the cache again, 1262 us; the keys split over 512 workgroups of four waves, partials in
// the caller's workspace and a merge launch, 21.0 us; this kernel with the place of every tile worked out
// by every wave 19.4 us, with one resource for the prefix 18.4, and with tiles of their own instead of
// steps in lockstep 14.6; with tiles that go straight into LDS 13.4.  (One lane per tile for a wave's own tile, all waves through all steps and three
// barriers behind them: 9 sequences of 111 keys 8.0 against 7.1 us, paged, 4 x 1000 keys, GQA 32/8 13.1 against 11.4.)  That split is faster only
// for long prompts on few heads (one sequence of 16000 keys and 8 KV heads: 33 us, here 112, 4720 on the
// vector units; d 256, 2 heads, 1500 keys: 21, 34, 421), and it needs a workspace that these shapes
// never asked for.
// A row of workgroups appended to the grid along y carries the walk of a verification that ran before this launch
// on the same stream (see tree_attn_mfma_kernel).
//
// TERMS: bf16 terms per weight.  Two for d != 128; one for d = 128, as in the other kernels for it (a step of
// two terms has twice the PV matrix instructions and a third more vector instructions).
template <int DP, int DS, int NW, int RH, int MT, int TS, int TERMS>
__global__ __launch_bounds__(64 * NW, 2)
void tree_attn_bf16_kernel(AttnParams p, WalkParams w)
{
    if ((int)blockIdx.y * DS >= p.d) {
        const int first = (int)(blockIdx.z * gridDim.x + blockIdx.x) * NW + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        for (int wb = first; wb < w.B; wb += (int)(gridDim.z * gridDim.x) * NW) walk_sequence(w, wb);
        return;
    }
    constexpr int KS = NW / RH, NT = 64 * NW;
    static_assert(TS % KS == 0, "every key stream takes the same number of tiles of a step");
    constexpr int WROWS = 16 * MT, ROWS = WROWS * RH;
    constexpr int GR = DP / 8, GV = DS / 8;              // 16-byte granules per row of K and of V
    constexpr int NL = TS * KT * GR / NT, NV = TS * KT * GV / NT;        // K and V loads per thread and step
    static_assert(KT * GV % 64 == 0 && NV > 0, "a wave's share of a load lies in one tile");
    constexpr int PK = DP / 2 + 4, PV = DS / 2 + 8;      // row pitches in words
    constexpr int PO = DS + 4;                           // row pitch of the epilogue's fp32 area
    constexpr bool OWN = RH == 1 && TS == KS;
    constexpr int V_AT = OWN ? KT * DP / 2 : KT * PK;    // where V lies behind K
    constexpr int TILE_WORDS = OWN ? KT * (DP + DS) / 2 : KT * (PK + PV);
    constexpr int STREAM_WORDS = OWN && TILE_WORDS < ROWS * PO ? ROWS * PO : TILE_WORDS;        // (OWN: a wavefront's outputs take the place of its tile)
    constexpr int LDS_WORDS = TS * STREAM_WORDS > KS * ROWS * PO ? TS * STREAM_WORDS : KS * ROWS * PO;
    constexpr int NKK = DP / 32, NNT = DS / 16;

    __shared__ __attribute__((aligned(16))) uint32_t s_big[LDS_WORDS];
    __shared__ uint32_t s_anc[MCSD_MAX_NODES][4];
    __shared__ int s_parent[MCSD_MAX_NODES];
    __shared__ float s_m[KS][ROWS], s_l[KS][ROWS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rh = wave / KS, ks = wave % KS;
    const int lj = lane >> 4, lc = lane & 15;
    const int g = blockIdx.x % p.H_kv, b = blockIdx.z;
    const int row0 = blockIdx.x / p.H_kv * ROWS, d0 = blockIdx.y * DS;

    const int len = p.prefix_len[b];
    const int my_parent = parent_of_thread(p, b);
    const uint32_t row_bytes = (uint32_t)p.d * 2u;

    // OWN: every wavefront has a tile of the step to itself (32 rows: one row group), which it loads itself, without
    // a barrier in the loop.  Load i of a thread: granule gid + GS i of the TS x 32 rows of the step, or of the
    // wavefront's tile, row-major, that is column granule c of row r0 + i GS / GR.  Columns past d are
    // requested beyond every extent.
    // The tiles behind the first go from memory straight into LDS, 16 bytes per lane at consecutive places: the stores of
    // them through registers were what bounded a step (576 KB of ds_write_b128, 32 rows, 1500 keys, d 128 in slices of 64:
    // 3.8 of the 7.5 us of all steps with the loads, as much without them; GQA 32/8, 4 x 100..1500 keys 14.2 -> 12.7 us,
    // d 64, 8 x 200..2000 14.7 -> 13.4, d 96, 4 x 200..1500 14.7 -> 13.1, 28 rows, 512 keys, 32 heads 8.95 -> 8.7; launches of
    // one tile per wave as before).  Those places are the rows without
    // a gap, so a lane takes the granule of its row that keeps the reads free of bank conflicts: K granule c of row r lies
    // at place c ^ f(r), V in pairs of granules, pair n of row r at place n ^ h(r) (16 consecutive rows of an operand,
    // and the 8 of a transposing read, then meet all banks once).
    constexpr int GS = OWN ? 64 : NT;
    static_assert(OWN || TS > 2 || (NT / GR <= KT && NT / GV <= KT), "without block-table entries ahead");
    static_assert((GS / GR % KT == 0 || KT % (GS / GR) == 0) && (GS / GV % KT == 0 || KT % (GS / GV) == 0), "a wave's share of a load lies in one tile");
    const int gid = OWN ? lane : tid, my_tile = OWN ? ks : 0;
    constexpr int KR = 64 / GR, VR = 64 / GV;            // OWN: rows per load
    constexpr int KVAR = OWN ? 16 / KR : 1, VVAR = OWN && VR < 8 ? 8 / VR : 1;  // loads after which the places repeat
    static_assert(!OWN || (DP <= 128 && NL % KVAR == 0 && NV % VVAR == 0), "places");
    auto place_k = [](int r) __attribute__((always_inline)) { return DP == 128 ? r & 15 : (r >> 1) & 7; };
    auto place_v = [](int r) __attribute__((always_inline)) { return DS == 128 ? r & 7 : (DS == 64 ? (r >> 1) & 3 : (r >> 2) & 1); };
    uint32_t ko[KVAR], vo[VVAR];
#pragma unroll
    for (int i = 0; i < (OWN ? KVAR : 0); ++i) {
        const int c = lane % GR ^ place_k(KR * i + lane / GR);
        ko[i] = 8 * c < p.d ? lane / GR * row_bytes + 16u * c : OFF_NOWHERE;
    }
#pragma unroll
    for (int i = 0; i < (OWN ? VVAR : 0); ++i) {
        const int c = lane % GV ^ (2 * place_v(VR * i + lane / GV));
        vo[i] = d0 + 8 * c < p.d ? lane / GV * row_bytes + 2u * d0 + 16u * c : OFF_NOWHERE;
    }
    uint32_t *const own_tile = s_big + (OWN ? ks : 0) * STREAM_WORDS;
    const uint32_t k_col = 8 * (gid % GR) < p.d ? 16u * (gid % GR) : OFF_NOWHERE;
    const uint32_t v_col = d0 + 8 * (gid % GV) < p.d ? 2u * d0 + 16u * (gid % GV) : OFF_NOWHERE;
    const uint32_t k_off = k_col == OFF_NOWHERE ? k_col : k_col + gid / GR * row_bytes, k_off_tile = k_col == OFF_NOWHERE ? k_col : k_col + gid / GR % KT * row_bytes;
    const uint32_t v_off = v_col == OFF_NOWHERE ? v_col : v_col + gid / GV * row_bytes, v_off_tile = v_col == OFF_NOWHERE ? v_col : v_col + gid / GV % KT * row_bytes;
    u32x4 kraw[NL], vraw[NV];
    // A step of prefix tiles of a contiguous cache: one resource over the sequence's rows (those past the
    // last one read as zero), scalar offsets.
    const size_t kv_head = (size_t)b * p.H_kv + g, slab = kv_head * (size_t)p.L_stride * row_bytes;
    // OWN: a tile that starts `at` bytes into the resources, into registers or (dma) into its place in LDS
    auto request_own = [&](__amdgpu_buffer_rsrc_t rk, __amdgpu_buffer_rsrc_t rv, uint32_t at, auto dma) __attribute__((always_inline)) {
        // (places and offsets counted up as they are needed: kept ready for all loads they do not fit the scalar registers)
        int word = (int)(own_tile - s_big);
        uint32_t k_at = at, v_at = at;
        if constexpr (decltype(dma)::value) asm volatile("" : "+s"(word));
#pragma unroll
        for (int i = 0; i < NL; ++i, k_at += KR * row_bytes) {
            if constexpr (decltype(dma)::value) load_into_lds(rk, s_big + word + 256 * i, ko[i % KVAR], k_at);
            else kraw[i] = __builtin_amdgcn_raw_buffer_load_b128(rk, ko[i % KVAR], k_at, 0);
            if constexpr (decltype(dma)::value) asm volatile("" : "+s"(k_at));
        }
#pragma unroll
        for (int i = 0; i < NV; ++i, v_at += VR * row_bytes) {
            if constexpr (decltype(dma)::value) load_into_lds(rv, s_big + word + V_AT + 256 * i, vo[i % VVAR], v_at);
            else vraw[i] = __builtin_amdgcn_raw_buffer_load_b128(rv, vo[i % VVAR], v_at, 0);
            if constexpr (decltype(dma)::value) asm volatile("" : "+s"(v_at));
        }
    };
    auto request_prefix = [&](int t0, int rows, auto dma) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t rk = make_rsrc(static_cast<const char *>(p.k_prefix) + slab, (uint32_t)rows * row_bytes);
        const __amdgpu_buffer_rsrc_t rv = make_rsrc(static_cast<const char *>(p.v_prefix) + slab, (uint32_t)rows * row_bytes);
        const uint32_t at = (uint32_t)(t0 + my_tile) * (KT * row_bytes);
        if constexpr (OWN) {
            request_own(rk, rv, at, dma);
            return;
        }
#pragma unroll
        for (int i = 0; i < NL; ++i) kraw[i] = __builtin_amdgcn_raw_buffer_load_b128(rk, k_off, at + i * (GS / GR) * row_bytes, 0);
#pragma unroll
        for (int i = 0; i < NV; ++i) vraw[i] = __builtin_amdgcn_raw_buffer_load_b128(rv, v_off, at + i * (GS / GV) * row_bytes, 0);
    };
    // OWN: the first tiles are asked for before the length is there, as if the cache were full, where they are few
    // (first_tiles_ahead): all rows of the slab may be read, and what turns out not to be a (whole) prefix tile is
    // requested again below.  Not in lockstep, where a wave loads parts of all tiles of the step: with that request 16
    // sequences of 100 keys in a cache of 600, GQA 32/8, d 96 take 13.2 us, without it 11.5, and no size is faster
    // with it (the kernel is shorter by a copy of the requests, which counts for launches of a step or two: 64
    // sequences of 32 keys, d 64 11.5 and 10.3 us, 8 of 300, d 256 16.9 and 16.8).
    constexpr int REACH = OWN ? 1 : TS;         // tiles of a step that one request covers, the first at t0 + my_tile
    const bool contiguous = one_resource(p, row_bytes), ahead = OWN && p.first_ahead && p.L_stride >= (my_tile + REACH) * KT;
    if (ahead) request_prefix(0, p.L_stride, std::false_type());

    const int L = max(0, min(len, p.L_stride));
    const int tiles_prefix = (L + KT - 1) / KT, t_end = tiles_prefix + (p.N + KT - 1) / KT;
    // The other steps (a paged cache, the end of the prefix, the tree).  Lane j works out where tile j of the step lies
    // (all lanes the tile of their wavefront); a wave's share of a load lies in one tile.  The block-table
    // entries of a step are read one step before it, and page and row advance from step to step without a
    // division.  Tiles at or past t_end are empty, which keeps every request unconditional.
    const int lane_tile = OWN ? ks : lane & (TS - 1);
    int blk = 0, blk_row = 0;           // of this lane's tile in the step that is requested next
    int page = 0, page_row = 0, page_step = 0, row_step = 0;
    if (p.block_table) {
        const unsigned key = lane_tile * KT, size = p.page_size;
        page = key / size; page_row = key % size;
        page_step = TS * KT / size; row_step = TS * KT % size;
    }
    auto look_up = [&](int t0) __attribute__((always_inline)) {        // (t0 = 0, TS, 2 TS, ...)
        if (!p.block_table || (!OWN && TS <= 2)) return;
        if (t0 + lane_tile < tiles_prefix) blk = p.block_table[(size_t)b * p.max_pages + page];
        blk_row = page_row;
        page += page_step; page_row += row_step;
        if (page_row >= p.page_size) { page_row -= p.page_size; ++page; }
    };
    auto request_any = [&](int t0, auto dma) __attribute__((always_inline)) {
        constexpr bool SAME = !OWN && NT / GR <= KT && NT / GV <= KT;       // load i lies in the same tile for all waves
        if (SAME && TS <= 2) {
            // a few tiles by scalar arithmetic (32 x 64 keys, GQA 32/8, d 96, two tiles a step: 12.3 us, 13.0 the other way)
            TileSrc src[TS];
#pragma unroll
            for (int j = 0; j < TS; ++j) src[j] = tile_source<KT>(p, b, g, L, tiles_prefix, t0 + j, t_end, row_bytes);
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                const TileSrc &from = src[SAME ? NT * i / GR / KT : 0];
                kraw[i] = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc(from.kb, from.bytes), k_off_tile, i * (GS / GR) % KT * row_bytes, 0);
            }
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const TileSrc &from = src[SAME ? NT * i / GV / KT : 0];
                vraw[i] = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc(from.vb, from.bytes), v_off_tile, i * (GS / GV) % KT * row_bytes, 0);
            }
            return;
        }
        const int t = t0 + lane_tile, key = t * KT, node = key - tiles_prefix * KT;
        if (OWN && t >= t_end) return;          // (there is no such step)
        const int entry = OWN ? __builtin_amdgcn_readfirstlane(blk) : blk;
        const bool tree = t >= tiles_prefix;
        size_t row = kv_head * (size_t)p.L_stride + (size_t)key;
        if (p.block_table)      // (an entry outside the pool never leaves it)
            row = ((size_t)min(max(entry, 0), p.n_pages - 1) * p.H_kv + g) * (size_t)p.page_size + (size_t)blk_row;
        if (tree) row = kv_head * (size_t)p.N + (size_t)node;
        int rows = t >= t_end ? 0 : min(KT, (tree ? p.N - node : L - key));
        if (DP == 128 && p.d == 128 && !tree && (unsigned)entry >= (unsigned)p.n_pages && p.block_table) rows = 0;       // (d = 128: such a tile reads as zero keys)
        const size_t at = t >= t_end ? 0 : row * row_bytes;
        const int lo = (int)(uint32_t)at, hi = (int)(uint32_t)(at >> 32);
        auto tile = [&](const void *prefix, const void *tree_block, int j) __attribute__((always_inline)) {
            if constexpr (OWN) return make_rsrc(static_cast<const char *>(tree ? tree_block : prefix) + at, (uint32_t)rows * row_bytes);
            const size_t off = (uint32_t)__builtin_amdgcn_readlane(lo, j) | (size_t)(uint32_t)__builtin_amdgcn_readlane(hi, j) << 32;
            return make_rsrc(static_cast<const char *>(t0 + j >= tiles_prefix ? tree_block : prefix) + off, (uint32_t)__builtin_amdgcn_readlane(rows, j) * row_bytes);
        };
        if constexpr (OWN) {
            request_own(tile(p.k_prefix, p.k_tree, 0), tile(p.v_prefix, p.v_tree, 0), 0, dma);
            return;
        }
        if constexpr (SAME) {
            // tile by tile, K and V behind each other: the places of all four or eight tiles at once are more than the
            // scalar registers hold (51 and 63 of them spilled).  us with scalar arithmetic and all places at once / here,
            // GQA 32/8: 16 x 100 keys, d 96 12.4/11.3, through pages 12.7/11.5; 32 x 64, d 64 10.1/8.7, 10.3/8.8; 8 x 500,
            // d 256 22.6/22.0, 25.5/22.4
#pragma unroll
            for (int j = 0; j < TS; ++j) {
                const size_t off = (uint32_t)__builtin_amdgcn_readlane(lo, j) | (size_t)(uint32_t)__builtin_amdgcn_readlane(hi, j) << 32;
                const uint32_t bytes = (uint32_t)__builtin_amdgcn_readlane(rows, j) * row_bytes;
                const bool of_tree = t0 + j >= tiles_prefix;
                const __amdgpu_buffer_rsrc_t rk = make_rsrc(static_cast<const char *>(of_tree ? p.k_tree : p.k_prefix) + off, bytes);
                const __amdgpu_buffer_rsrc_t rv = make_rsrc(static_cast<const char *>(of_tree ? p.v_tree : p.v_prefix) + off, bytes);
#pragma unroll
                for (int i = NL / TS * j; i < NL / TS * (j + 1); ++i)
                    kraw[i] = __builtin_amdgcn_raw_buffer_load_b128(rk, k_off_tile, i * (GS / GR) % KT * row_bytes, 0);
#pragma unroll
                for (int i = NV / TS * j; i < NV / TS * (j + 1); ++i)
                    vraw[i] = __builtin_amdgcn_raw_buffer_load_b128(rv, v_off_tile, i * (GS / GV) % KT * row_bytes, 0);
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < NL; ++i)
            kraw[i] = __builtin_amdgcn_raw_buffer_load_b128(tile(p.k_prefix, p.k_tree, (wave * 64 + NT * i) / GR / KT), k_off_tile, i * (GS / GR) % KT * row_bytes, 0);
#pragma unroll
        for (int i = 0; i < NV; ++i)
            vraw[i] = __builtin_amdgcn_raw_buffer_load_b128(tile(p.v_prefix, p.v_tree, (wave * 64 + NT * i) / GV / KT), v_off_tile, i * (GS / GV) % KT * row_bytes, 0);
    };
    look_up(0);
    if (!ahead || (my_tile + REACH) * KT > L) request_any(0, std::false_type());
    look_up(TS);

    // Q operand: lane (lj, lc) holds Q[row0 + WROWS rh + 16 mt + lc][32 kk + 8 lj .. + 7]
    bf16x8 qreg[MT][NKK];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int r = row0 + WROWS * rh + 16 * mt + lc;
        const int rr = min(r, p.M - 1), node = rr / p.G, hh = rr % p.G;
        const uint16_t *src = static_cast<const uint16_t *>(p.q) + (((size_t)b * p.N + node) * p.H_q + (size_t)g * p.G + hh) * (size_t)p.d;
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (r < p.M && 32 * kk + 8 * lj < p.d) v = *reinterpret_cast<const u32x4 *>(src + 32 * kk + 8 * lj);
            qreg[mt][kk] = __builtin_bit_cast(bf16x8, v);
        }
    }
    build_ancestor_masks(p, my_parent, s_anc, s_parent);

    f32x4 oacc[NNT][MT];
    float m_used[MT], l_part[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        m_used[mt] = M_INIT;
        l_part[mt] = 0.f;
#pragma unroll
        for (int nt = 0; nt < NNT; ++nt) oacc[nt][mt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    const bool wave_active = row0 + WROWS * rh < p.M;
    const float c2 = p.scale_log2;
    typedef short v4i16 __attribute__((ext_vector_type(4)));
    typedef v4i16 __attribute__((address_space(3))) *lds_v4i16_ptr;

    // PLAIN (a promise of the caller): the tiles of this step (OWN: of this wavefront) are whole prefix tiles, and those
    // of the next one prefix tiles, of a contiguous cache.
    auto step = [&](const int t0, auto plain) __attribute__((always_inline)) {
        constexpr bool PLAIN = decltype(plain)::value;
        bf16x8 kop[OWN ? 2 * NKK : 1], vops[OWN ? NNT : 1];
        // Ahead of the scores in slices of 32 columns, behind their matrix instructions in wider ones (28 rows, 512 keys, 32 heads, slices of
        // 32: 8.7 us and 9.1; GQA 32/8, 4 x 100..1500 keys, slices of 64: 12.8 and 12.7; d 64, 8 x 200..2000: 13.6 and 13.4).
        auto v_and_next = [&]() __attribute__((always_inline)) {
            const uint32_t *vl = own_tile + V_AT + (4 * lj + (lc >> 2)) * (DS / 2) + (lc & 3) * 2;
            const int at_v = place_v(4 * lj + (lc >> 2));
#pragma unroll
            for (int nt = 0; nt < (OWN ? NNT : 0); ++nt) {
                const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)(vl + (nt ^ at_v) * 8));
                const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)(vl + 16 * (DS / 2) + (nt ^ at_v) * 8));
                vops[nt] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
            if (PLAIN || t0 + TS + my_tile < t_end) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // (all operands have left)
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (PLAIN) request_prefix(t0 + TS, L, std::true_type());
                else { request_any(t0 + TS, std::true_type()); look_up(t0 + 2 * TS); }
            }
        };
        if constexpr (OWN) {
            // The operands leave LDS for registers at once, and the next tile takes their place while this one is computed.
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const uint32_t *kt = own_tile + lc * (DP / 2);
#pragma unroll
            for (int kk = 0; kk < NKK; ++kk) {
                const int c = 4 * ((4 * kk + lj) ^ place_k(lc));
                kop[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kt + c));
                kop[NKK + kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kt + 16 * (DP / 2) + c));
            }
            if constexpr (DS < 64) v_and_next();
        } else {
            __syncthreads();                // the last step's operands have been read
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                const int row = (gid + GS * i) / GR;
                *reinterpret_cast<u32x4 *>(s_big + (my_tile + row / KT) * STREAM_WORDS + row % KT * PK + 4 * (gid % GR)) = kraw[i];
            }
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int row = (gid + GS * i) / GV;
                *reinterpret_cast<u32x4 *>(s_big + (my_tile + row / KT) * STREAM_WORDS + V_AT + row % KT * PV + 4 * (gid % GV)) = vraw[i];
            }
            if (PLAIN) request_prefix(t0 + TS, L, std::false_type());
            else if (t0 + TS < t_end) { request_any(t0 + TS, std::false_type()); look_up(t0 + 2 * TS); }
            __syncthreads();
        }
        if (!wave_active) return;
#pragma unroll 1
        for (int ts = ks; ts < TS; ts += KS) {
            const int t = t0 + ts;
            if (!PLAIN && !OWN && t >= t_end) break;
            const uint32_t *kt = s_big + ts * STREAM_WORDS, *vt = kt + V_AT;
            f32x4 sacc[2][MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) { sacc[0][mt] = (f32x4){0.f, 0.f, 0.f, 0.f}; sacc[1][mt] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
#pragma unroll
            for (int kk = 0; kk < NKK; ++kk) {
                const bf16x8 k0 = OWN ? kop[OWN ? kk : 0] : __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kt + lc * PK + 16 * kk + 4 * lj));
                const bf16x8 k1 = OWN ? kop[OWN ? NKK + kk : 0] : __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kt + (16 + lc) * PK + 16 * kk + 4 * lj));
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    sacc[0][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k0, qreg[mt][kk], sacc[0][mt], 0, 0, 0);
                    sacc[1][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1, qreg[mt][kk], sacc[1][mt], 0, 0, 0);
                }
            }
            if constexpr (OWN && DS >= 64) v_and_next();
            // lane (lj, lc): row 16 mt + lc, keys 16 sub + 4 lj + i
            const bool tree = !PLAIN && t >= tiles_prefix;
            const int nvalid = PLAIN || tree ? KT : min(KT, L - t * KT);          // (a tree tile's mask ends with the tree)
            // (whole prefix tiles, nearly all of them, pay nothing for the masks)
            const bool masked = tree || nvalid < KT;
            uint32_t vis[MT];
            float lmax[MT];
            bool raise = false;
            if constexpr (MT == 2) settle_scores(sacc[0][0], sacc[0][1], sacc[1][0], sacc[1][1]);
            else settle_scores(sacc[0][0], sacc[1][0]);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if (masked) {
                    vis[mt] = (1u << (nvalid & 31)) - 1u;
                    if (tree) vis[mt] = s_anc[min(row0 + WROWS * rh + 16 * mt + lc, p.M - 1) / p.G][t - tiles_prefix];
                    vis[mt] >>= 4 * lj;
#pragma unroll
                    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (!((vis[mt] >> (16 * sub + i)) & 1u)) sacc[sub][mt][i] = -INFINITY;
                }
                const float mr = max_of_scores(sacc[0][mt], sacc[1][mt]);
                lmax[mt] = (mr == -INFINITY) ? -INFINITY : mr * c2;
                raise |= lmax[mt] > m_used[mt] + RESCALE_GAP;
            }
            if (__any(raise)) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    float rm = lmax[mt];
                    rm = fmaxf(rm, __shfl_xor(rm, 16));
                    rm = fmaxf(rm, __shfl_xor(rm, 32));
                    const float m_new = fmaxf(m_used[mt], rm);
                    const float alpha = fast_exp2(m_used[mt] - m_new);
                    m_used[mt] = m_new;
                    l_part[mt] *= alpha;
#pragma unroll
                    for (int nt = 0; nt < NNT; ++nt) oacc[nt][mt] *= alpha;
                }
            }
            bf16x8 phi[MT], plo[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                float pv[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int sub = e >> 2, i = e & 3;
                    pv[e] = fast_exp2(fmaf(sacc[sub][mt][i], c2, -m_used[mt]));
                }
                if (masked) {
                    // (with scale == 0 a masked score can not be told apart by its value)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (!((vis[mt] >> (16 * (e >> 2) + (e & 3))) & 1u)) pv[e] = 0.f;
                }
                l_part[mt] += ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));
                u32x4 ph, plw;
                if constexpr (TERMS == 1) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) ph[j] = pack_bf16(pv[2 * j], pv[2 * j + 1]);
                } else {
                    uint32_t hi[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) hi[e] = weight_hi_bits(pv[e]);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        ph[j] = __builtin_amdgcn_perm(hi[2 * j + 1], hi[2 * j], 0x07060302u);
                        plw[j] = pack_bf16(pv[2 * j] - __uint_as_float(hi[2 * j]), pv[2 * j + 1] - __uint_as_float(hi[2 * j + 1]));
                    }
                    plo[mt] = __builtin_bit_cast(bf16x8, plw);
                }
                phi[mt] = __builtin_bit_cast(bf16x8, ph);
            }
            const uint32_t *vl = vt + (4 * lj + (lc >> 2)) * PV + (lc & 3) * 2;
#pragma unroll
            for (int nt = 0; nt < NNT; ++nt) {
                bf16x8 vop;
                if constexpr (OWN) {
                    vop = vops[nt];
                } else {
                    const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)(vl + nt * 8));
                    const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)(vl + 16 * PV + nt * 8));
                    vop = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    oacc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop, phi[mt], oacc[nt][mt], 0, 0, 0);
                    if constexpr (TERMS == 2) oacc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop, plo[mt], oacc[nt][mt], 0, 0, 0);
                }
            }
        }
    };
    if (OWN) {
        __syncthreads();                    // the masks are there (the other form passes a barrier before it reads them)
        // the first tile, through registers (it may have been asked for twice)
        if (my_tile < t_end) {
#pragma unroll
            for (int i = 0; i < NL; ++i) *reinterpret_cast<u32x4 *>(own_tile + 256 * i + 4 * lane) = kraw[i];
#pragma unroll
            for (int i = 0; i < NV; ++i) *reinterpret_cast<u32x4 *>(own_tile + V_AT + 256 * i + 4 * lane) = vraw[i];
        }
    }
    int t0 = 0;
    if (contiguous)
        for (; (t0 + my_tile + REACH) * KT <= L && t0 + TS + my_tile + REACH <= tiles_prefix; t0 += TS) step(t0, std::true_type());
    for (; t0 + my_tile < t_end; t0 += TS) step(t0, std::false_type());

    // ---- epilogue: every wave leaves its (m, l) per row and its O in LDS (OWN: in the area of its tiles); behind
    // a barrier the key streams are added up, each brought to the largest of the maxima, and whole rows written
    constexpr int AREA = OWN ? STREAM_WORDS : ROWS * PO;         // words of a key stream
    static_assert(AREA >= ROWS * PO && KS * AREA <= LDS_WORDS, "the outputs fit");
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        float lt = l_part[mt];
        lt += __shfl_xor(lt, 16);
        lt += __shfl_xor(lt, 32);
        if (lj == 0) { s_m[ks][WROWS * rh + 16 * mt + lc] = m_used[mt]; s_l[ks][WROWS * rh + 16 * mt + lc] = lt; }
    }
    if (!OWN) __syncthreads();              // every wave is done with the tiles
    float *area = reinterpret_cast<float *>(s_big);
#pragma unroll
    for (int nt = 0; nt < NNT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            *reinterpret_cast<f32x4 *>(area + ks * AREA + (WROWS * rh + 16 * mt + lc) * PO + 16 * nt + 4 * lj) = oacc[nt][mt];
    __syncthreads();
    const int rows_valid = min(ROWS, p.M - row0), d4n = min(DS, p.d - d0) / 4;
    for (int idx = tid; idx < rows_valid * d4n; idx += NT) {
        const bool whole = d4n == DS / 4;
        const int r = whole ? idx / (DS / 4) : idx / d4n, d4 = idx - r * d4n;
        float ms = s_m[0][r], ls = 0.f;
#pragma unroll
        for (int k2 = 1; k2 < KS; ++k2) ms = fmaxf(ms, s_m[k2][r]);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k2 = 0; k2 < KS; ++k2) {
            const float f = fast_exp2(s_m[k2][r] - ms);
            ls += f * s_l[k2][r];
            acc += f * *reinterpret_cast<const f32x4 *>(area + k2 * AREA + r * PO + 4 * d4);
        }
        const float inv = 1.0f / ls;
        const int gr = row0 + r, node = gr / p.G, hh = gr % p.G;
        uint16_t *ob = static_cast<uint16_t *>(p.out) + (((size_t)b * p.N + node) * p.H_q + (size_t)g * p.G + hh) * (size_t)p.d + d0 + 4 * d4;
        __builtin_nontemporal_store((u32x2){pack_bf16(acc[0] * inv, acc[1] * inv), pack_bf16(acc[2] * inv, acc[3] * inv)}, reinterpret_cast<u32x2 *>(ob));
    }
}

// ------------------------------------------------------------------------------ fp32
// fp32 multiplies on the matrix cores.  A workgroup of 8 waves owns 16 query rows of a KV head and
// DS output columns; every wave walks every 8th tile of 16 keys with its own online softmax and
// the streams are merged at the end (no workspace, no barrier in the loop).  Bound by the fp32
// matrix rate at one workgroup per CU (d 128, slices of 32 columns: 40 instructions of 32 cycles per wave
// and tile, two waves per SIMD, 9 us for 1000 keys): 2 sequences of 301 and 1000 tokens, 16 heads of
// 128, 28 nodes: 326 us with one workgroup per (node, head) on the vector units, 19.7 us with slices of 64
// columns, 17.7 us here; relative error against 64 bits 5.2e-7 on the vector units, 2.9e-7 since.
//   S^T: the contraction index is d; step (kk, j) of lane (lj, lc) takes d = 16 kk + 4 lj + j, so
//        that both operands are 16-byte pieces (K from LDS, Q in registers).
//   O^T: step i takes key 4 lj + i, the key whose weight the lane holds; row index lc of the matrix
//        (blk, e) is column 16 E blk + E lc + e (E = 4, or 2 for slices of 32 columns), so that V comes
//        straight from memory, E words per lane.
template <int DP, int DS>
__global__ __launch_bounds__(512, 2)
void tree_attn_f32_kernel(AttnParams p)
{
    constexpr int KW = 16, KS = 8, ROWS = 16;
    constexpr int GR = DP / 4, NL = KW * GR / 64;        // 16-byte granules per row; K loads per lane and tile
    constexpr int E = DS >= 64 ? 4 : DS / 16, NB = DS / (16 * E);        // columns of V per lane and load, loads per row
    constexpr int PK = DP + 4, PO = DS + 4;              // row pitches in words
    constexpr int NKK = DP / 16;
    typedef float fE __attribute__((ext_vector_type(E)));

    __shared__ __attribute__((aligned(16))) float s_big[KS][KW * PK];
    __shared__ uint32_t s_anc[MCSD_MAX_NODES][4];
    __shared__ int s_parent[MCSD_MAX_NODES];
    __shared__ float s_m[KS][ROWS], s_l[KS][ROWS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int ks = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lj = lane >> 4, lc = lane & 15;
    const int g = blockIdx.x % p.H_kv, b = blockIdx.z;
    const int row0 = blockIdx.x / p.H_kv * ROWS, d0 = blockIdx.y * DS;

    const int len = p.prefix_len[b];
    const int my_parent = parent_of_thread(p, b);
    const uint32_t row_bytes = (uint32_t)p.d * 4u;

    // K load i: granule lane + 64 i of the tile, row-major; V load (n, i): row 4 lj + i, columns d0 + 16 E n + E lc ..
    const uint32_t k_off = 4 * (lane % GR) < p.d ? lane / GR * row_bytes + 16u * (lane % GR) : OFF_NOWHERE;
    const uint32_t k_pos = lane / GR * PK + 4 * (lane % GR);             // + i (64 / GR) PK
    uint32_t v_off[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const int col = d0 + 16 * E * n + E * lc;
        v_off[n] = col < p.d ? (uint32_t)(4 * lj) * row_bytes + 4u * col : OFF_NOWHERE;
    }
    u32x4 kraw[NL];
    fE vraw[NB][4];
    auto request_k = [&](const __amdgpu_buffer_rsrc_t &rs, uint32_t at) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NL; ++i) kraw[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, k_off, at + i * (64 / GR) * row_bytes, 0);
    };
    auto request_v = [&](const __amdgpu_buffer_rsrc_t &rs, uint32_t at) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (E == 4) vraw[n][i] = __builtin_bit_cast(fE, __builtin_amdgcn_raw_buffer_load_b128(rs, v_off[n], at + i * row_bytes, 0));
                else vraw[n][i] = __builtin_bit_cast(fE, __builtin_amdgcn_raw_buffer_load_b64(rs, v_off[n], at + i * row_bytes, 0));
            }
    };
    // The prefix of a contiguous cache: one resource, scalar offsets.  (The first tiles ahead of the length, as in the
    // bf16 kernel: 20, 60, 100, 300 keys in a cache of 300, 32 heads of 128 7.2, 7.7, 8.3, 11.1 us, here 6.6, 7.3,
    // 8.0, 11.0; 128 heads 10.3, 11.0, 11.8, 15.8 and 7.6, 9.6, 11.2, 15.6.)
    const size_t slab = ((size_t)b * p.H_kv + g) * (size_t)p.L_stride * row_bytes;
    const bool contiguous = one_resource(p, row_bytes);
    const int L = max(0, min(len, p.L_stride));
    const int tiles_prefix = (L + KW - 1) / KW, t_end = tiles_prefix + (p.N + KW - 1) / KW;
    const __amdgpu_buffer_rsrc_t rs_k = make_rsrc(static_cast<const char *>(p.k_prefix) + slab, contiguous ? (uint32_t)L * row_bytes : 0u);
    const __amdgpu_buffer_rsrc_t rs_v = make_rsrc(static_cast<const char *>(p.v_prefix) + slab, contiguous ? (uint32_t)L * row_bytes : 0u);
    {
        const TileSrc s = tile_source<KW>(p, b, g, L, tiles_prefix, ks, t_end, row_bytes);
        request_k(make_rsrc(s.kb, s.bytes), 0);
        request_v(make_rsrc(s.vb, s.bytes), 0);
    }

    f32x4 qreg[NKK];
    {
        const int r = row0 + lc, rr = min(r, p.M - 1), node = rr / p.G, hh = rr % p.G;
        const float *src = static_cast<const float *>(p.q) + (((size_t)b * p.N + node) * p.H_q + (size_t)g * p.G + hh) * (size_t)p.d;
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) {
            qreg[kk] = (f32x4){0.f, 0.f, 0.f, 0.f};
            if (r < p.M && 16 * kk + 4 * lj < p.d) qreg[kk] = *reinterpret_cast<const f32x4 *>(src + 16 * kk + 4 * lj);
        }
    }
    build_ancestor_masks(p, my_parent, s_anc, s_parent);
    __syncthreads();

    f32x4 oacc[NB][E];
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int e = 0; e < E; ++e) oacc[n][e] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float m_used = M_INIT, l_part = 0.f;
    const float c2 = p.scale_log2;
    const int node_m = min(row0 + lc, p.M - 1) / p.G;
    float *area = s_big[ks];

    // PLAIN (a promise of the caller): tile t is a whole prefix tile, and t + KS a prefix tile, of a contiguous cache.
    auto step = [&](const int t, auto plain) __attribute__((always_inline)) {
        constexpr bool PLAIN = decltype(plain)::value;
        TileSrc next = {};
        if (!PLAIN) next = tile_source<KW>(p, b, g, L, tiles_prefix, t + KS, t_end, row_bytes);
        const uint32_t at = (uint32_t)(t + KS) * (KW * row_bytes);
#pragma unroll
        for (int i = 0; i < NL; ++i) *reinterpret_cast<u32x4 *>(area + k_pos + i * (64 / GR) * PK) = kraw[i];
        if (PLAIN) request_k(rs_k, at);
        else request_k(make_rsrc(next.kb, next.bytes), 0);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // two accumulators: half the length of the serial chain
        f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < NKK; kk += 2) {
            const f32x4 ka = *reinterpret_cast<const f32x4 *>(area + lc * PK + 16 * kk + 4 * lj);
            const f32x4 kb = *reinterpret_cast<const f32x4 *>(area + lc * PK + 16 * kk + 16 + 4 * lj);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(ka[j], qreg[kk][j], s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kb[j], qreg[kk + 1][j], s1, 0, 0, 0);
            }
        }
        f32x4 sc = s0 + s1;
        // lane (lj, lc): row lc, keys 4 lj + i
        uint32_t vis = 0xfu;
        if (!PLAIN) {
            const bool tree = t >= tiles_prefix;
            const int key0 = (t - tiles_prefix) * KW;                    // of a tree tile
            const int nvalid = tree ? KW : min(KW, L - t * KW);
            vis = tree ? s_anc[node_m][key0 >> 5] >> (key0 & 31) : 0xffffffffu;
            if (nvalid < KW) vis = (1u << nvalid) - 1u;
            vis >>= 4 * lj;
        }
        float mr = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (!PLAIN && !((vis >> i) & 1u)) sc[i] = -INFINITY;
            mr = fmaxf(mr, sc[i]);
        }
        const float lmax = (mr == -INFINITY) ? -INFINITY : mr * c2;
        if (__any(lmax > m_used + RESCALE_GAP)) {
            float rm = lmax;
            rm = fmaxf(rm, __shfl_xor(rm, 16));
            rm = fmaxf(rm, __shfl_xor(rm, 32));
            const float m_new = fmaxf(m_used, rm);
            const float alpha = fast_exp2(m_used - m_new);
            m_used = m_new;
            l_part *= alpha;
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int e = 0; e < E; ++e) oacc[n][e] *= alpha;
        }
        float pw[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pw[i] = fast_exp2(fmaf(sc[i], c2, -m_used));
            if (!PLAIN && !((vis >> i) & 1u)) pw[i] = 0.f;
        }
        l_part += (pw[0] + pw[1]) + (pw[2] + pw[3]);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int e = 0; e < E; ++e)
                    oacc[n][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vraw[n][i][e], pw[i], oacc[n][e], 0, 0, 0);
        if (PLAIN) request_v(rs_v, at);
        else request_v(make_rsrc(next.vb, next.bytes), 0);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");       // the K operands are read before the next tile is stored
        __builtin_amdgcn_wave_barrier();
    };
    int t = ks;
    if (contiguous && DP <= 128)            // (d = 256, 1000 keys: the general form is 2 to 4 % faster, 30.9 against 32.4 us)
        for (; (t + 1) * KW <= L && t + KS < tiles_prefix; t += KS) step(t, std::true_type());
    for (; t < t_end; t += KS) step(t, std::false_type());

    // ---- epilogue: merge the eight streams, each brought to the largest of the maxima, behind one barrier
    float lt = l_part;
    lt += __shfl_xor(lt, 16);
    lt += __shfl_xor(lt, 32);
    if (lj == 0) { s_m[ks][lc] = m_used; s_l[ks][lc] = lt; }
    // oacc[n][e][i] is row lc, column 16 E n + E (4 lj + i) + e
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            fE v;
#pragma unroll
            for (int e = 0; e < E; ++e) v[e] = oacc[n][e][i];
            *reinterpret_cast<fE *>(area + lc * PO + 16 * E * n + E * (4 * lj + i)) = v;
        }
    __syncthreads();
    const int rows_valid = min(ROWS, p.M - row0);
    for (int idx = tid; idx < ROWS * (DS / 4); idx += 512) {
        const int r = idx / (DS / 4), c = idx % (DS / 4);
        if (r >= rows_valid || d0 + 4 * c >= p.d) continue;
        float ms = s_m[0][r], ls = 0.f;
#pragma unroll
        for (int k2 = 1; k2 < KS; ++k2) ms = fmaxf(ms, s_m[k2][r]);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k2 = 0; k2 < KS; ++k2) {
            const float f = exp2f(s_m[k2][r] - ms);
            ls += f * s_l[k2][r];
            acc += f * *reinterpret_cast<const f32x4 *>(s_big[k2] + r * PO + 4 * c);
        }
        const int gr = row0 + r, node = gr / p.G, hh = gr % p.G;
        float *ob = static_cast<float *>(p.out) + (((size_t)b * p.N + node) * p.H_q + (size_t)g * p.G + hh) * (size_t)p.d + d0 + 4 * c;
        const float inv = 1.0f / ls;
        *reinterpret_cast<f32x4 *>(ob) = acc * inv;
    }
}

template <int DP, int DS, int NW, int RH, int MT, int TS, int TERMS = 2>
void launch_bf16(const AttnParams &p, hipStream_t stream, const WalkParams *tail_walk = nullptr)
{
    constexpr int ROWS = 16 * MT * RH;
    WalkParams w = {};
    if (tail_walk) w = *tail_walk;
    AttnParams q = p;
    q.first_ahead = one_resource(p, 2u * p.d) && first_tiles_ahead(p, TS, 2u * p.d);
    const dim3 grid((unsigned)p.H_kv * ((p.M + ROWS - 1) / ROWS), (p.d + DS - 1) / DS + (tail_walk ? 1 : 0), p.B);
    launch_kernel(p.d == 128 ? K_ATTN_MFMA : K_ATTN_GENERIC, tree_attn_bf16_kernel<DP, DS, NW, RH, MT, TS, TERMS>, grid, dim3(64 * NW), stream, q, w);
}

template <int DP, int DS>
void launch_f32(const AttnParams &p, hipStream_t stream)
{
    launch_kernel(K_ATTN_GENERIC, tree_attn_f32_kernel<DP, DS>, dim3((unsigned)p.H_kv * ((p.M + 15) / 16), (p.d + DS - 1) / DS, p.B), dim3(512), stream, p);
}

}  // namespace

int32_t launch_attn_sliced(const AttnParams &p, int columns, hipStream_t stream, const WalkParams *tail_walk)
{
    if (columns == 32) launch_bf16<128, 32, 8, 1, 2, 8, 1>(p, stream, tail_walk);
    else if (columns == 64) launch_bf16<128, 64, 8, 1, 2, 8, 1>(p, stream, tail_walk);
    else launch_bf16<128, 128, 8, 1, 2, 8, 1>(p, stream, tail_walk);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("tree_attn launch failed: %s", hipGetErrorString(e)); return MCSD_E_HIP; }
    return MCSD_OK;
}

int32_t launch_attn_any(const AttnParams &p, hipStream_t stream)
{
    if (p.B > 65535) { set_error("attn: B %d > 65535", p.B); return MCSD_E_UNSUPPORTED; }
    const int dp = p.d <= 64 ? 64 : (p.d <= 128 ? 128 : 256);
    if (p.dtype == MCSD_DTYPE_FP32) {
        // Few units: the output columns are split over workgroups as well (every slice scores the keys again):
        // slices of 32 columns while those fit one per CU, of 64 while the units would leave half of the
        // CUs idle.  us at 200 / 1000 keys, slices of 32, of 64 columns:
        //   d 64   16 units of 16 rows  6.6/12.3  7.1/14.3     64 units  6.9/12.6  7.4/14.6     96 units  7.0/12.7  7.5/14.6
        //   d 128  16                   8.5/17.4  8.9/19.6     64        9.1/20.2  9.4/21.1     96       13.6/32.2  9.5/22.4
        //   d 256  16                  13.1/28.9 13.6/32.4     64       25.0/59.4 14.4/35.6     96       36.4/87.2 26.0/65.2
        const long units16 = (long)p.B * p.H_kv * ((p.M + 15) / 16);
        const bool narrow = units16 * (dp / 32) <= 256, slices = units16 < 128;
        if (dp == 64) { if (narrow) launch_f32<64, 32>(p, stream); else launch_f32<64, 64>(p, stream); }
        else if (dp == 128) { if (narrow) launch_f32<128, 32>(p, stream); else if (slices) launch_f32<128, 64>(p, stream); else launch_f32<128, 128>(p, stream); }
        else { if (narrow) launch_f32<256, 32>(p, stream); else if (slices) launch_f32<256, 64>(p, stream); else launch_f32<256, 128>(p, stream); }
    } else {
        // Rows of a KV head per workgroup and wavefronts.  While the launch fits one workgroup per CU, few
        // rows by eight wavefronts: the walk over the keys is the time, and the key tiles that several
        // workgroups read come out of L2; and slices of the output columns as long as those fit, too, since
        // what counts is what a wavefront does in its step (1000 keys, 28 rows, 8 heads, d 96: 14.9 us whole, 10.9
        // in slices of 32; 1500 keys, d 64 12.1 and 10.7).  Beyond, four wavefronts (two workgroups per CU) and the
        // more rows the more workgroups there are, so that a tile is read for more of them.  (The figures for
        // 8 x 32 rows are of the form in lockstep, which took a quarter longer.)
        // d 64, us at 200 / 1500 keys, 32 rows x 8 wavefronts, 64 x 8, 32 x 4, 64 x 4, 128 x 4:
        //   64 units of 112 rows   (256, 128 workgroups of 32, 64 rows)  7.8/17.4  8.6/22  8.1/20  9.3/28  12/42
        //   256 units of 28        (256)                                 8.2/20.6  8.1/22  8.3/21  8.8/28  11/40
        //   128 units of 112       (512, 256)                            14/33     9.0/24  9.8/25  9.5/28  12/42
        //   192 units of 112       (768, 384)                            20/46     16/43   12/31   12/36   12/42
        //   256 units of 112       (1024, 512)                           26/60     16/43   16/42   12/36   13/43
        //   384 units of 112       (1536, 768)                           38/97     24/68   21/59   15/48   18/59
        //   512 units of 112       (2048, 1024)                          50/129    32/90   26/80   20/67   18/63
        // d 96, 384 units of 112 rows (768 of 64): 25/86 with 64 rows, 23/84 with 128; 256 units 16/54 and 17/61;
        // 192 units (768 of 32) 21/64 with 32 rows, 16/52 with 64.
        // d 256, eight wavefronts and 32 rows, slices of 64, 128, 256 columns, four wavefronts: 64 units 11/35
        // 12/41 13/41 15/51; 128 units 20/73 13/46 15/55 15/58; 192 units 29/103 23/86 16/61 16/62; 512 units
        // 73/273 46/174 33/145 26/142.
        // 257 to 512 workgroups of 32 rows, more than 32 rows, since a wavefront's own tiles go straight into LDS: 64 rows x 8 in
        // lockstep, eight tiles a step / 32 x 4, two workgroups per CU, with caches of 256, 320, 600, 1000 keys, all full; lengths
        // spread evenly from an eighth on; all of a quarter (the host knows the capacity only):
        //   d 64, 8 x 32 units of 56 rows  11.7/10.7 11.3/9.7 8.0/8.3   11.8/10.9 11.4/10.0 8.0/8.7   15.3/13.4 14.1/11.9 9.2/9.5   20.9/17.8 19.4/14.2
        //         9 x 8 of 112             10.4/10.1 10.5/9.6 7.7/7.6   10.4/10.1 10.5/9.5 7.8/8.0    12.9/12.2 12.8/10.8 8.4/8.8   17.9/15.1 17.7/13.2
        //   d 96, 8 x 32 of 56             16.3/14.2 15.1/12.1 10.8/10.1 17.2/14.8 15.6/12.8 10.9/10.7 22.0/18.5 19.8/15.3 12.5/12.0 34.0/27.8 28.8/19.6
        //         9 x 8 of 112             14.6/12.9 14.3/12.0 10.1/9.6  15.1/13.1 14.3/11.9 10.1/10.2 18.8/16.3 17.8/13.9 11.3/11.1 27.0/21.2 25.0/17.6
        // Below (200 keys: 9.8/10.0 9.1/9.7 8.0/8.6 and 13.5/13.2 12.2/12.0, 9 x 8 8.5/9.1 and 11.7/12.0) one step of the lockstep has all tiles.
        // So it has for short sequences in a larger cache, which therefore lose at d <= 64: all of 60 keys, caches of 512 to 2000, 7.8/8.3 (72 units
        // of 112 rows) to 8.4/9.1 (256 of 56), all of 128 of 512 8.8/9.5 to 9.5/10.2, while one full among sequences of 100 gains 13.0/10.4 to 27.3/19.0.
        // d 96 with more than 256 workgroups of 64 rows (65 to 96, 129 to 160 rows), four wavefronts of 64 rows, two tiles a step / this; caches of
        // 60, 200, 400, 1000 keys, full; spread; all of 60 keys in a cache of 1000:
        //   130 units of 70 rows   11.4/11.6 16.2/14.2 21.0/17.5 35.7/30.8   10.8/10.6 14.6/14.0 17.8/15.5 28.4/22.6   11.1/12.7
        //   140 of 70              13.0/11.7 17.6/14.5 23.0/17.9 38.5/32.3   12.5/10.7 16.2/14.3 19.7/15.6 30.5/23.5   12.6/12.8
        //   170 of 94              13.4/12.6 18.1/15.3 23.6/20.3 39.8/38.1   12.9/11.8 16.5/15.3 20.5/17.0 32.4/26.8   13.0/13.9
        //    88 of 132             11.0/10.9 15.9/13.1 20.3/15.4 35.0/24.9   10.4/10.0 14.1/12.8 17.4/14.1 27.9/20.8   10.8/11.1
        //   100 of 160             13.3/11.9 18.0/14.8 23.2/18.0 38.1/31.7   12.7/11.0 16.5/14.7 20.1/15.8 31.4/23.6   12.9/13.0
        // (with few more than 256 workgroups of 64 rows one has a CU to itself mostly, and short sequences lose most: 1.15 there.)
        const int tiles = (p.L_stride + 31) / 32 + (p.N + 31) / 32;
        const long units = (long)p.B * p.H_kv, wgs32 = units * ((p.M + 31) / 32), wgs64 = units * ((p.M + 63) / 64);
        if (dp == 64) {
            if (wgs32 <= 128 && p.d > 32) launch_bf16<64, 32, 8, 1, 2, 8>(p, stream);
            else if (wgs32 <= 256) launch_bf16<64, 64, 8, 1, 2, 8>(p, stream);
            else if (p.M > 32 && wgs64 <= 256 && tiles <= 16) launch_bf16<64, 64, 8, 2, 2, 8>(p, stream);
            else if (p.M <= 32 || wgs32 <= 768) launch_bf16<64, 64, 4, 1, 2, 4>(p, stream);
            else if (p.M <= 64 || wgs64 < 1024) launch_bf16<64, 64, 4, 2, 2, 4>(p, stream);
            else launch_bf16<64, 64, 4, 4, 2, 4>(p, stream);
        } else if (dp == 128) {
            if (wgs32 * ((p.d + 31) / 32) <= 256) launch_bf16<128, 32, 8, 1, 2, 8>(p, stream);
            else if (wgs32 <= 128) launch_bf16<128, 64, 8, 1, 2, 8>(p, stream);
            else if (wgs32 <= 256) launch_bf16<128, 128, 8, 1, 2, 8>(p, stream);
            else if (p.M > 32 && wgs64 <= 256 && tiles <= 8) launch_bf16<128, 128, 8, 2, 2, 8>(p, stream);
            else if (wgs32 <= 512 || p.M <= 32) launch_bf16<128, 128, 4, 1, 2, 4>(p, stream);
            else if (p.M <= 64 || wgs64 < 768) launch_bf16<128, 128, 4, 2, 2, 2>(p, stream);
            else launch_bf16<128, 128, 4, 4, 2, 2>(p, stream);
        } else {
            if (wgs32 <= 64) launch_bf16<256, 64, 8, 2, 1, 4>(p, stream);
            else if (wgs32 <= 128) launch_bf16<256, 128, 8, 2, 1, 4>(p, stream);
            else if (wgs32 <= 256) launch_bf16<256, 256, 8, 2, 1, 4>(p, stream);
            else if (p.M <= 32) launch_bf16<256, 256, 4, 2, 1, 2>(p, stream);
            else launch_bf16<256, 256, 4, 4, 1, 1>(p, stream);
        }
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("tree_attn launch failed: %s", hipGetErrorString(e)); return MCSD_E_HIP; }
    return MCSD_OK;
}

}  // namespace mcsd
