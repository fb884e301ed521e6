// Tree attention (Sec. 3.3 of the paper), bf16, d = 128, more than 64 query rows per KV head: the four
// waves of a workgroup share every K/V tile of one key stream through LDS.  (Fewer rows, the
// launch plan and the merge of the segments: tree_attn.hip.)
#include <type_traits>

#include "attn_common.h"

namespace mcsd {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Tiles per segment from the lengths the sequences really have.  The host's plan knows the capacity
// of the cache only; the compute units hold 512 workgroups at a time, and a launch a little above a
// multiple of that runs a nearly empty last round.  The segments are made so long that the launch
// just fits one round; two where a workgroup would walk more than 128 tiles (older and younger
// workgroups of a unit then even out), one workgroup per CU below 12 tiles (half the partials).
// Measured, attention and merge, against 1024 workgroups by capacity: one sequence of 16000 keys, GQA
// 64/8, 84 nodes: 68 against 83 us; 8 x 1000..3000 keys, 28 nodes: 44 against 52 us; one sequence of
// 8000 keys, 28 nodes: 25 against 39 us.  Every wavefront works it out from the lengths of up to 64 sequences.
// (*len: the length of sequence number `lane`)
__device__ __forceinline__ int segment_tiles(const AttnParams &p, int lane, int *len)
{
    int T = 0;
    *len = 0;
    if (lane < p.B) {
        *len = max(0, min(p.prefix_len[lane], p.L_stride));
        T = (*len + KT - 1) / KT + p.tiles_tree;
    }
    // sum over the wavefront without a trip through LDS: inside the rows of 16 lanes, then across them
    auto sum = [](int v) {
        v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, false);      // lanes 1 apart
        v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, false);      // 2 apart
        v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, false);     // mirror of 8
        v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, false);     // mirror of 16
        v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);     // rows 0, 2 into 1, 3
        v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);     // and into 2, 3
        return __builtin_amdgcn_readlane(v, 63);
    };
    const int units = p.H_kv * p.n_row_tiles;
    const long work = (long)sum(T) * units;
    const int slots_log2 = work > 512 * 128 ? 10 : (work < 512 * 12 ? 8 : 9), slots = 1 << slots_log2;
    int chunk = max(p.chunk_tiles, (int)((work + slots - 1) >> slots_log2));
    if (slots == 1024 && chunk == p.chunk_tiles) return chunk;      // the caches are as full as the host assumed
#pragma unroll 1
    for (int i = 0; i < 8; ++i) {
        const int n = lane < p.B ? max(1, (T + chunk / 2) / chunk) : 0;
        if (sum(n) * units <= slots) break;
        chunk += (chunk + 15) / 16;
    }
    return chunk;
}

// A workgroup of four waves owns 128 query rows of one KV head (32 per wave) and a segment of the key
// tiles.  Every wave loads a quarter of each 32-key tile and stores it to a double-buffered LDS
// tile, from which all of them read their operands after one workgroup barrier per tile.
//
//   S^T = K Q^T     v_mfma_f32_32x32x16_bf16, A = K (lane: key lane % 32, d = 16 kk + 8 h .. + 7 with
//                   h = lane / 32), B = Q in registers.  A lane ends up with 16 keys of one query row,
//                   row lane % 32: score i is key 8 (i / 4) + 4 h + i % 4.
//   O^T += V^T P^T  the same instruction; scores 8 m .. 8 m + 7 of a lane are the B operand of step m as
//                   they stand, so a weight never leaves its lane.  V comes out of LDS with the transposing
//                   load, which hands a lane four keys of one d column.
//
// LDS rows are in their natural order, K with a pitch of 68 words (16 lanes of a 128-bit read lie in
// 16 rows, 4 words apart modulo the 64 banks) and V of 80 (32 lanes of a transposing read lie in four
// rows of 16 words, 16 apart modulo the banks): both reads and the stores are free of bank conflicts.
//
// Bound, for long prefixes, by the power the chip may draw rather than by any one pipe: the same
// instruction stream on constant instead of random operands runs 1.2 to 1.4 times as fast, and so
// orders of it that hide more (scores of the next tile beside the weights of this one) gain nothing.  For short
// ones by the chain barrier -> K operands -> scores -> weights -> PV of a tile, which is what this
// instruction shortens: half the matrix instructions for the same work, which leave more room beside
// them (registers only, two waves per SIMD, 32768 multiply-adds: alone 15.9 against 17.2 ns for two 16x16x32,
// with six v_fma_f32 17.7 / 24.2, with four and two v_exp_f32 19.7 / 25.5), and one pair of
// lanes per row to agree on its maximum instead of four.  Against 16x16x32 with a test of all
// scores: a decode round of four layers, GQA 32/8, 4 x 100..1500 keys, 120.4 -> 110.3 us; 4 x 16384 keys, GQA
// 64/8, 84 nodes 216.3 -> 216.9 us with the merge (914 TFLOP/s over the keys past the first 16384).
template <bool PAGED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void tree_attn_shared_kernel(AttnParams p, WalkParams w)
{
    constexpr int NW = 4, NT = 256, WROWS = 32, ROWS = 128, D = 128;
    constexpr int TILE_BYTES = KT * D * 2;
    constexpr int PK = 68, PV = 80, BUF_WORDS = KT * (PK + PV);      // row pitches and size of a tile buffer, in words
    constexpr int PO = 68;                                           // row pitch of the epilogue's areas
    constexpr int LDS_WORDS = 2 * BUF_WORDS > NW * WROWS * PO ? 2 * BUF_WORDS : NW * WROWS * PO;
    // A row of workgroups appended to the grid along y carries the walk of a verification that ran
    // before this launch on the same stream (see tree_attn_mfma_kernel).
    if ((int)blockIdx.y >= p.n_chunks_max * p.n_row_tiles) {
        const int first = (int)(blockIdx.z * gridDim.x + blockIdx.x) * NW + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        for (int wb = first; wb < w.B; wb += (int)(gridDim.z * gridDim.x) * NW) walk_sequence(w, wb);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, l32 = lane & 31, lj = lane >> 4, lc = lane & 15;

    __shared__ __attribute__((aligned(16))) uint32_t s_big[LDS_WORDS];
    __shared__ uint32_t s_anc[MCSD_MAX_NODES][4];
    __shared__ int s_parent[MCSD_MAX_NODES];
    __shared__ PairRanks<NT> s_rank;

    // Load j (0, 1) of wave w: rows 8 w + 4 j + lj of the tile, 16-byte granule lc (1 KB, contiguous).
    const uint32_t load_off = (uint32_t)(2 * wave * 1024 + lane * 16);
    const uint32_t k_st = (8 * wave + lj) * PK + 4 * lc;                        // + 4 j PK
    const uint32_t v_st = KT * PK + (8 * wave + lj) * PV + 4 * lc;              // + 4 j PV
    const uint32_t k_ld = l32 * PK + 4 * h;                                     // + 8 kk
    // transposing read (m, half, nt): the 16 lanes of a group point at keys 16 m + 8 half + 4 h + (lc >> 2),
    // d columns 32 nt + 16 (lj & 1) + 4 (lc & 3) .. + 3
    const uint32_t v_ld = KT * PK + (4 * h + (lc >> 2)) * PV + 8 * (lj & 1) + 2 * (lc & 3);     // + (16 m + 8 half) PV + 16 nt
    const float c2 = p.scale_log2;      // >= 0 (checked by the host)

    // ---- this workgroup's segment: unit (b, g, rt), tiles [t_begin, t_end) of total_tiles
    int b = blockIdx.z, L, chunk = blockIdx.y / p.n_row_tiles;
    const int g = blockIdx.x, rt = blockIdx.y % p.n_row_tiles;
    int chunk_tiles = p.chunk_tiles, split_bias = p.split_bias, len_of_lane = 0;
    const bool lens_known = p.chunk_of_launch;
    int upto = 0, live = 0;             // segments of the sequences up to number `lane`; of all
    if (__builtin_expect(lens_known, 0)) {      // (out of the way of the launches without it)
        chunk_tiles = segment_tiles(p, lane, &len_of_lane);
        split_bias = chunk_tiles / 2;
        if (tid == 0 && blockIdx.x + blockIdx.y + blockIdx.z == 0) *p.chunk_of_launch = chunk_tiles;       // for the merge
        if (lane < p.B) {
            const int Tl = (len_of_lane + KT - 1) / KT + p.tiles_tree;
            int nl, segl;
            split_tiles(Tl, chunk_tiles, split_bias, 0, 0, &nl, &segl);
            upto = (Tl + segl - 1) / segl;
        }
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x111, 0xf, 0xf, false);      // running sum: inside the rows of 16
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x112, 0xf, 0xf, false);
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x114, 0xf, 0xf, false);
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x118, 0xf, 0xf, false);
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x142, 0xa, 0xf, false);
        upto += __builtin_amdgcn_update_dpp(0, upto, 0x143, 0xc, 0xf, false);
        live = __builtin_amdgcn_readlane(upto, 63);
    }
    if (__builtin_expect(lens_known && live * p.H_kv * p.n_row_tiles <= 512, 0)) {
        // All start at once: their order does not matter, but those without a segment come last (among
        // the others they would leave some CUs with two).  Without the ranking, cache of 16384 rows,
        // GQA 32/8, 28 nodes, 16384 / 8000 / 2000 / 500 keys 28.6 / 23.2 / 19.3 / 19.3 -> 26.4 / 20.7 / 16.7 / 16.7 us
        // (1024 workgroups by capacity: 92 / 52 / 26 / 18); four sequences of 400 keys 22.4 -> 19.3 (20.5).
        const int pair = blockIdx.z * p.n_chunks_max + chunk;
        if (pair >= live) return;
        b = __ffsll((long long)__ballot(upto > pair)) - 1;
        chunk = pair - (b > 0 ? __builtin_amdgcn_readlane(upto, b - 1) : 0);
        L = __builtin_amdgcn_readlane(len_of_lane, b);
    } else if (p.rank_pairs) {
        longest_first(p, s_rank, tid, (int)(blockIdx.z * p.n_chunks_max) + chunk, chunk_tiles, split_bias, 0,
                      [&](int seq) { return lens_known ? __shfl(len_of_lane, seq) : max(0, min(p.prefix_len[seq], p.L_stride)); },
                      &b, &chunk, &L);
    } else {
        L = lens_known ? __builtin_amdgcn_readlane(len_of_lane, b) : max(0, min(p.prefix_len[b], p.L_stride));
    }
    const int total_tiles = (L + KT - 1) / KT + p.tiles_tree;
    int n_seg, seg;
    split_tiles(total_tiles, chunk_tiles, split_bias, 0, 0, &n_seg, &seg);
    const int t_begin = chunk * seg;
    if (t_begin >= total_tiles) return;
    const int t_end = min(total_tiles, t_begin + seg);
    const bool direct = n_seg == 1;
    const int tilesP = (L + KT - 1) / KT;
    const int row0 = rt * ROWS + WROWS * wave;          // of this wave

    // Q operand: lane holds Q[row0 + l32][16 kk + 8 h .. + 7].  Lanes past the last row repeat it
    // (their results are not written): nothing looks at the values here, so that the first K/V requests
    // go out right behind these loads.
    const int my_row = min(row0 + l32, p.M - 1), my_node = my_row / p.G;
    const int my_parent = t_end > tilesP ? parent_of_thread(p, b) : -1;
    bf16x8 qreg[8];
    {
        const uint16_t *src = static_cast<const uint16_t *>(p.q) + (((size_t)b * p.N + my_node) * p.H_q + (size_t)g * p.G + my_row % p.G) * D + 8 * h;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) qreg[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(src + 16 * kk));
    }
    f32x16 oacc[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[nt][i] = 0.f;
    float m_used = M_INIT, l_part = 0.f;

    const size_t kv_head = (size_t)b * p.H_kv + g;
    // K and V of this (sequence, KV head) are read through buffer resources whose extent is
    // exactly the valid rows (prefix_len rows of the cache slab, N rows of the tree block):
    // the tile base is a scalar offset, the lane offset a constant, and rows past the end of
    // a partial tile read as zero instead of leaving the array (their scores are masked).
    // (paged cache: the prefix resources are empty and every prefix tile gets a resource of
    // its own over the page slice it lies in)
    const size_t slab = PAGED ? 0 : kv_head * (size_t)p.L_stride * (D * 2);
    const __amdgpu_buffer_rsrc_t rs_kpre = make_rsrc(static_cast<const char *>(p.k_prefix) + slab, PAGED ? 0u : (uint32_t)L * (D * 2));
    const __amdgpu_buffer_rsrc_t rs_vpre = make_rsrc(static_cast<const char *>(p.v_prefix) + slab, PAGED ? 0u : (uint32_t)L * (D * 2));
    const __amdgpu_buffer_rsrc_t rs_ktre = make_rsrc(static_cast<const char *>(p.k_tree) + kv_head * (size_t)p.N * (D * 2), (uint32_t)p.N * (D * 2));
    const __amdgpu_buffer_rsrc_t rs_vtre = make_rsrc(static_cast<const char *>(p.v_tree) + kv_head * (size_t)p.N * (D * 2), (uint32_t)p.N * (D * 2));

    struct TileRef { int off; int nvalid; bool tree; int tt; size_t page_off; bool paged; };
    // Tiles at or past t_end are requested at an offset beyond every buffer's extent: the
    // hardware returns zeros without touching memory.  This keeps the prefetch of the next
    // tile unconditional, so the wait for one tile's data never has to cover the loads issued
    // after it (a load under a branch makes the compiler wait for everything outstanding).
    constexpr int OFF_NOWHERE = 0x7fff0000;
    // (paged cache: blk = the block-table entry of the page the tile starts in)
    auto tile_ref_blk = [&](int t, int blk, int row_in_page) {
        TileRef r;
        r.page_off = 0; r.paged = false;
        if (t >= t_end) {
            r.off = OFF_NOWHERE; r.nvalid = KT; r.tree = false; r.tt = 0;
        } else if (t < tilesP) {
            r.off = t * TILE_BYTES; r.nvalid = min(KT, L - t * KT); r.tree = false; r.tt = 0;
            if (PAGED) {
                if ((unsigned)blk < (unsigned)p.n_pages) {
                    r.paged = true;
                    r.off = 0;
                    r.page_off = (((size_t)blk * p.H_kv + g) * (size_t)p.page_size + (size_t)row_in_page) * (D * 2);
                } else {
                    r.off = OFF_NOWHERE;       // an entry outside the pool reads as zero keys, never as memory
                }
            }
        } else {
            r.tt = t - tilesP;
            r.off = r.tt * TILE_BYTES; r.nvalid = min(KT, p.N - r.tt * KT); r.tree = true;
        }
        return r;
    };
    // The block table is only read by this kernel.  Through a pointer to the constant address
    // space its (wave-uniform) entries are fetched with scalar loads wherever the read stands;
    // through the plain pointer the compiler falls back to a vector load behind every barrier
    // or asm statement, and the wait for that load covers all K/V requests in flight.
    typedef const int32_t __attribute__((address_space(4))) *const_i32_ptr;
    const const_i32_ptr block_table_c = (const_i32_ptr)(uintptr_t)p.block_table;
    auto tile_ref = [&](int t) {
        int blk = -1;
        if (PAGED && t < t_end && t < tilesP) blk = block_table_c[(size_t)b * p.max_pages + (t * KT) / p.page_size];
        return tile_ref_blk(t, blk, PAGED ? (t * KT) % p.page_size : 0);
    };
    // Paged cache: the block-table entry of a tile is read one step before the tile is
    // requested, ahead of the workgroup barrier.  Scalar loads share the LDS counter and
    // return out of order, so using one right after issuing it would drain every LDS read in
    // flight; at the barrier that wait is made anyway.  The page and the row inside it of the
    // tile that is looked up next advance by one tile per step (no division in the loop).
    int ahead_page = 0, ahead_row = 0;          // of the tile whose entry is read next
    int blk_ahead = -1, row_ahead = 0;          // entry and row-in-page read last
    auto table_lookup_next = [&](int tt) {      // tt = index of that tile
        row_ahead = ahead_row;
        blk_ahead = (PAGED && tt < tilesP && tt < t_end) ? (int)block_table_c[(size_t)b * p.max_pages + ahead_page] : -1;
        ahead_row += KT;
        if (ahead_row >= p.page_size) { ahead_row = 0; ++ahead_page; }
    };
    // this wave's quarter of both tiles (two K and two V requests) into register stage st
    u32x4 kraw[4], vraw[4];
    auto load_kv = [&](const TileRef &r, const int st) __attribute__((always_inline)) {
        __amdgpu_buffer_rsrc_t rk = r.tree ? rs_ktre : rs_kpre;
        __amdgpu_buffer_rsrc_t rv = r.tree ? rs_vtre : rs_vpre;
        if (PAGED && r.paged) {
            rk = make_rsrc(static_cast<const char *>(p.k_prefix) + r.page_off, (uint32_t)r.nvalid * (D * 2));
            rv = make_rsrc(static_cast<const char *>(p.v_prefix) + r.page_off, (uint32_t)r.nvalid * (D * 2));
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            kraw[2 * st + j] = __builtin_amdgcn_raw_buffer_load_b128(rk, load_off + j * 1024, r.off, 0);
            vraw[2 * st + j] = __builtin_amdgcn_raw_buffer_load_b128(rv, load_off + j * 1024, r.off, 0);
        }
    };
    auto store_kv = [&](uint32_t *buf, const int st) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            *reinterpret_cast<u32x4 *>(buf + k_st + 4 * j * PK) = kraw[2 * st + j];
            *reinterpret_cast<u32x4 *>(buf + v_st + 4 * j * PV) = vraw[2 * st + j];
        }
    };

    int t = t_begin;
    // (read before the first K/V requests, as inside the loop: the wait at the loop top is the
    // longer of the two paths into it)
    if (PAGED) {
        ahead_page = ((t + 3) * KT) / p.page_size;
        ahead_row = ((t + 3) * KT) % p.page_size;
        table_lookup_next(t + 3);
    }
    // the first tile goes to its LDS buffer here, every later one inside the step before it;
    // requests run two to three tiles ahead of their use
    load_kv(tile_ref(t), 0);
    load_kv(tile_ref(t + 1), 1);
    store_kv(s_big, 0);
    load_kv(tile_ref(t + 2), 0);
    const bool wave_active = row0 < p.M;        // a wave whose rows all lie past M only helps to load
    // the masks are needed from the first tree tile on; built while the first loads are in flight
    if (t_end > tilesP) {
        build_ancestor_masks(p, my_parent, s_anc, s_parent);
        __syncthreads();
    }
    // PLAIN (a promise of the caller): tile t and the tile requested during this step are whole
    // prefix tiles inside the segment: nothing is masked, and with a contiguous cache the tile
    // references are plain offsets (a paged cache still looks its pages up).
    auto plain_ref = [&](int tt) {
        TileRef r;
        r.off = tt * TILE_BYTES; r.nvalid = KT; r.tree = false; r.tt = 0; r.page_off = 0; r.paged = false;
        return r;
    };
    typedef short v4i16 __attribute__((ext_vector_type(4)));
    typedef v4i16 __attribute__((address_space(3))) *lds_v4i16_ptr;
    auto tile_step = [&](const int t, auto stage, auto plain, auto active) __attribute__((always_inline)) {
        constexpr int ST = decltype(stage)::value;      // register stage and LDS buffer of this tile
        constexpr bool PLAIN = decltype(plain)::value;
        const TileRef cur = PLAIN ? plain_ref(t) : tile_ref(t);
        // Tile t is in buffer t & 1 once every wave has passed this barrier; tile t + 1 goes
        // from its registers to the other buffer while the matrix cores work on QK, and
        // tile t + 3 is requested into the registers that frees.  The other buffer is free:
        // it held tile t - 1, whose last read precedes every wave's arrival here.  One
        // barrier per tile, and no wave waits for memory or for its LDS stores at it.
        const uint32_t *cb = s_big + ST * BUF_WORDS;
        const int blk_next = blk_ahead, row_next = row_ahead;
        if (PAGED) table_lookup_next(t + 4);
        __syncthreads();
        if constexpr (!decltype(active)::value) {
            store_kv(s_big + (ST ^ 1) * BUF_WORDS, ST ^ 1);
            load_kv(PLAIN && !PAGED ? plain_ref(t + 3) : tile_ref_blk(t + 3, blk_next, row_next), ST ^ 1);
            return;
        }
        bf16x8 kop[8], vop[2][4];
        f32x16 s;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) kop[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(cb + k_ld + 8 * kk));
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kop[kk], qreg[kk], s, 0, 0, 0);
        // V^T operands by transposing LDS reads
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)(cb + v_ld + 16 * m * PV + 16 * nt));
                const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)(cb + v_ld + (16 * m + 8) * PV + 16 * nt));
                vop[m][nt] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        store_kv(s_big + (ST ^ 1) * BUF_WORDS, ST ^ 1);
        load_kv(PLAIN && !PAGED ? plain_ref(t + 3) : tile_ref_blk(t + 3, blk_next, row_next), ST ^ 1);
        if (PLAIN) {
            // all K operands first; the V operands, the stores of the next tile and the requests
            // between the matrix instructions
            __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
        }
        const bool masked = !PLAIN && (cur.nvalid < KT || cur.tree);
        uint32_t vis = 0xffffffffu;
        if (masked) {
            if (cur.tree) vis = s_anc[my_node][cur.tt];
            if (cur.nvalid < KT) vis &= (1u << cur.nvalid) - 1u;
            vis >>= 4 * h;
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (!((vis >> (8 * (i >> 2) + (i & 3))) & 1u)) s[i] = -INFINITY;
        }
        // Weights p = 2^(s c2 - m) of eight scores, masked keys 0; returns the lane's share of the row sum.
        auto weights = [&](const int m, const float x0, bf16x8 &pop) __attribute__((always_inline)) {
            float pv[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) pv[i] = fast_exp2(i == 0 ? x0 : fmaf(s[8 * m + i], c2, -m_used));
            if (masked) {
                // also covers scale == 0, where a masked score can not be told apart by its value
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (!((vis >> (8 * (2 * m + (i >> 2)) + (i & 3))) & 1u)) pv[i] = 0.f;
            }
            const u32x4 pk = {pack_bf16(pv[0], pv[1]), pack_bf16(pv[2], pv[3]), pack_bf16(pv[4], pv[5]), pack_bf16(pv[6], pv[7])};
            pop = __builtin_bit_cast(bf16x8, pk);
            return ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));
        };
        // Online softmax in the scaled base-2 domain with a lazily raised maximum: the reference point m
        // moves only where a weight outgrows 2^8.  For the first eight scores the test is on the sum of the
        // weights, which is formed anyway; the rare raise computes them again.
        bf16x8 pop0, pop1;
        float x0 = fmaf(s[0], c2, -m_used);
        // max3_raw must not read a matrix result early, which the compiler does not see to (attn_common.h):
        // behind this statement the scores have been read by an instruction that it waits for
        asm volatile("" : "+v"(s), "+v"(x0));
        float sum0 = weights(0, x0, pop0);
        float mx = max3_raw(s[8], s[9], s[10]);
        mx = max3_raw(mx, s[11], s[12]);
        mx = max3_raw(max3_raw(mx, s[13], s[14]), s[15], s[15]);
        if (__builtin_expect(__any(sum0 > 256.f || fmaf(mx, c2, -m_used) > RESCALE_GAP), 0)) {
            float rm = -INFINITY;
#pragma unroll
            for (int i = 0; i < 16; ++i) rm = fmaxf(rm, s[i]);
            rm = (rm == -INFINITY) ? -INFINITY : rm * c2;
            rm = fmaxf(rm, __shfl_xor(rm, 32));
            const float m_new = fmaxf(m_used, rm);
            const float alpha = fast_exp2(m_used - m_new);
            m_used = m_new;
            l_part *= alpha;
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[nt][i] *= alpha;
            sum0 = weights(0, fmaf(s[0], c2, -m_used), pop0);
        }
        // A wave issues in order, and vector instructions placed behind a matrix instruction run while the
        // matrix pipe works on it: the weights of the second half between the PV instructions of the
        // first.  (O^T[d][row] += sum_key V[key][d] P[row][key])
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) oacc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[0][nt], pop0, oacc[nt], 0, 0, 0);
        l_part += sum0;
        l_part += weights(1, fmaf(s[8], c2, -m_used), pop1);
        if (!masked) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x402, 7, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) oacc[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[1][nt], pop1, oacc[nt], 0, 0, 0);
    };
    // Tiles alternate between the two register stages / LDS buffers.  The pair loop has no
    // branch around its second half: with one, the wait for a stage's data at the top of
    // the loop would have to cover the path on which no younger loads are in flight, that
    // is, wait for everything.  An odd last tile is handled after the loop.
    // The bulk of a long prefix goes through the plain step: while t + 4 is still a whole prefix tile
    // of this segment, so are t, t + 1 and the two tiles requested during the pair.
    // A wave without rows runs a loop of its own with the same barriers.
    auto all_tiles = [&](auto active) __attribute__((always_inline)) {
        const int t_plain = min(t_end, L / KT);
        asm volatile(".p2align 6");             // (the loop starts on an instruction-cache line)
        for (; t + 4 < t_plain; t += 2) {
            tile_step(t, std::integral_constant<int, 0>(), std::true_type(), active);
            tile_step(t + 1, std::integral_constant<int, 1>(), std::true_type(), active);
        }
        for (; t + 1 < t_end; t += 2) {
            tile_step(t, std::integral_constant<int, 0>(), std::false_type(), active);
            tile_step(t + 1, std::integral_constant<int, 1>(), std::false_type(), active);
        }
        if (t < t_end) tile_step(t, std::integral_constant<int, 0>(), std::false_type(), active);
    };
    if (wave_active) all_tiles(std::true_type());
    else all_tiles(std::false_type());

    // ---- epilogue: rows through LDS, two halves of d, each wave in an area of its own.
    // The lane indices are re-derived from an opaque copy so that the epilogue's address
    // arithmetic is not hoisted above the tile loop, where it would cost registers (and spill).
    __syncthreads();                            // the other waves may still read the last tile
    if (!wave_active) return;
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));
    const int h_e = lane_e >> 5, l32_e = lane_e & 31;
    const float l_row = l_part + __shfl_xor(l_part, 32);
    const size_t part_row = (((size_t)b * p.H_kv + g) * p.n_chunks_max + chunk) * (size_t)p.R + row0;
    const int rows_valid = min(WROWS, p.M - row0);
    float *area = reinterpret_cast<float *>(s_big) + wave * (WROWS * PO);
    const float f = direct ? 1.0f / l_row : 1.0f;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int n2 = 0; n2 < 2; ++n2)
#pragma unroll
            for (int j = 0; j < 4; ++j) {       // d = 64 half + 32 n2 + 8 j + 4 h + (0..3)
                const f32x16 &o = oacc[2 * half + n2];
                *reinterpret_cast<f32x4 *>(area + l32_e * PO + 32 * n2 + 8 * j + 4 * h_e) = (f32x4){o[4 * j] * f, o[4 * j + 1] * f, o[4 * j + 2] * f, o[4 * j + 3] * f};
            }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // one 16-byte piece per lane, neighbouring lanes neighbouring pieces: every store
        // instruction of the partial covers whole 256-byte runs
#pragma unroll
        for (int i = 0; i < WROWS * 16 / 64; ++i) {
            const int r = (lane_e >> 4) + 4 * i, d4 = lane_e & 15;
            const f32x4 v = *reinterpret_cast<const f32x4 *>(area + r * PO + 4 * d4);
            if (r >= rows_valid) continue;
            const int dcol = 64 * half + 4 * d4;
            // outputs and partials are written once and not read again by this kernel: stored
            // non-temporally they do not sit dirty in L2 until the end-of-kernel write-back
            if (direct) {
                const int gr = row0 + r, node = gr / p.G, hh = gr % p.G;
                uint16_t *ob = static_cast<uint16_t *>(p.out);
                __builtin_nontemporal_store((u32x2){pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])},
                                            reinterpret_cast<u32x2 *>(ob + (((size_t)b * p.N + node) * p.H_q + (size_t)g * p.G + hh) * D + dcol));
            } else {
                __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(p.part_o + (part_row + r) * D + dcol));
            }
        }
    }
    if (!direct && lane_e < rows_valid) {
        p.part_m[part_row + lane_e] = m_used;
        p.part_l[part_row + lane_e] = l_row;
    }
}

}  // namespace

void launch_attn_shared(const AttnParams &p, dim3 grid, hipStream_t stream, const WalkParams &w)
{
    if (p.block_table) launch_kernel(K_ATTN_MFMA, tree_attn_shared_kernel<true>, grid, dim3(256), stream, p, w);
    else launch_kernel(K_ATTN_MFMA, tree_attn_shared_kernel<false>, grid, dim3(256), stream, p, w);
}

}  // namespace mcsd
