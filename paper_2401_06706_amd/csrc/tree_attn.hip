// Tree attention (Sec. 3.3 of the paper) on gfx950.
//
// All candidate tokens of the draft tree are scored in one pass over the shared
// prefix KV cache: the cache is streamed from HBM once and every tree node (times
// the query heads that share a KV head) is a row of the same tile, which is the
// saving the paper attributes to tree attention.  A node additionally attends to
// its ancestors and itself among the tree's own keys; that mask is a 128-bit
// ancestor bitmask per node held in LDS.
//
// Work decomposition (bf16, d = 128: tree_attn_mfma_kernel)
//   keys of a sequence = ceil(L/32) prefix tiles followed by ceil(N/32) tree tiles
//   unit      = (sequence b, KV head g, tile of 32/64/128 query rows)
//   segment   = a run of consecutive key tiles of a unit, processed by one workgroup
//               (4 waves): wave (rh, ks) owns 32 rows and every KS-th tile of the run and
//               runs an independent online softmax with no workgroup barrier in the loop
//               (32- and 64-row tiles); more than 64 rows per KV head run the kernel of
//               tree_attn_shared.hip, whose four waves share every tile of one key stream.
//   The T tiles of a unit are cut into round(T / chunk_tiles) equal segments (at least one):
//   grid (KV head, segment x row tile, sequence).  The (sequence, segment) pairs are handed
//   out longest first.  A segment that covers its whole unit writes the output rows itself;
//   otherwise its (max, sum, O) partial goes to the workspace and tree_attn_combine_kernel
//   merges the partials of a unit by log-sum-exp.
//   The prefix cache is either one contiguous slab per (sequence, KV head) or a pool of
//   pages addressed through a block table (PAGED instantiation); the tiles are the same.
//
// Everything else (fp32 storage, other head dims) runs the kernels of tree_attn_any.hip.
#include <math.h>

#include <atomic>
#include <type_traits>

#include "attn_common.h"

namespace mcsd {
namespace {

// --------------------------------------------------------------------- MFMA path
// RH = row groups per workgroup, KS = key streams per workgroup.  Wave (rh, ks) owns query rows
// [32 rh, 32 (rh+1)) of the workgroup's row tile and the key tiles t_begin + ks, + KS, ... of the
// segment.  Waves of one key stream read the same K/V tiles (the second read is served by the
// L1/L2 caches).
//
// Data movement per 32-key tile and wave (8 KB of K, 8 KB of V, one 16.9 KB LDS area):
//   K  global -> registers with fully contiguous 1 KB loads (issued one tile ahead),
//      registers -> LDS in MFMA-operand order (16-byte granules, XOR-swizzled so that
//      both the stores and the operand loads are bank-conflict free), LDS -> operand.
//      Loading K straight into operand registers would make neighbouring lanes read
//      different cache lines, which stalls the address path of the vector memory unit.
//   V  global -> registers (a lane reads 8 key rows x 16 contiguous bytes, neighbouring
//      lanes neighbouring bytes; one tile ahead), in-lane 8x8 transpose of the 16-bit
//      elements, registers -> the same LDS area -> operand (exchange inside 16-lane groups).
//
// WHOLE (contiguous cache, no sequence is split, room for KS tiles, few units: first_tiles_ahead): a workgroup owns all keys of its unit, so
// that the first tiles lie at the start of the slab whatever the length is: they are asked for
// as soon as the arguments are there, as if the cache were full (all rows of the slab may be read), and a wave
// whose first tile is not a whole one of the prefix asks again.  That takes the length's trip to memory and some
// 300 instructions out of the chain; with it, and one barrier instead of five behind the loop, one sequence of 300
// keys and 32 heads 10.0 -> 8.4 us (9.2 without the requests ahead).
template <int RH, int KS, bool PAGED, bool WHOLE>
__global__ __launch_bounds__(RH * KS * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void tree_attn_mfma_kernel(AttnParams p, WalkParams w)
{
    // A row of workgroups appended to the grid along y carries the walk of a verification that ran
    // before this launch on the same stream (one wavefront per sequence; the row has H_kv B workgroups
    // of four, for as many sequences as the verification has), when the caller asked for that: a step whose attention needs no merge launch then has
    // no launch for the walk either.
    if ((int)blockIdx.y >= p.n_chunks_max * p.n_row_tiles) {
        const int first = (int)(blockIdx.z * gridDim.x + blockIdx.x) * (RH * KS) + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        for (int wb = first; wb < w.B; wb += (int)(gridDim.z * gridDim.x) * (RH * KS)) walk_sequence(w, wb);
        return;
    }
    constexpr int MT = 2;                   // 16-row MFMA tiles per wave
    constexpr int NW = RH * KS;
    constexpr int NT = NW * 64;
    constexpr int WROWS = 16 * MT;          // rows per wave
    constexpr int ROWS = WROWS * RH;        // rows per workgroup
    constexpr int D = 128;
    constexpr int TILE_BYTES = KT * D * 2;  // 8192
    constexpr int PO = D + 4;               // row pitch of the epilogue
    constexpr int AREA_WORDS = WROWS * PO;  // per-wave LDS area: >= 2048 words of staging, the wave's output in the epilogue
    static_assert(AREA_WORDS >= 2048, "staging needs 8 KB per wave");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keeps tile indices and pointers scalar
    const int rh = wave / KS, ks = wave % KS;
    const int lj = lane >> 4, lc = lane & 15;

    __shared__ __attribute__((aligned(16))) uint32_t s_big[NW * AREA_WORDS];
    __shared__ uint32_t s_anc[MCSD_MAX_NODES][4];
    __shared__ int s_parent[MCSD_MAX_NODES];
    __shared__ float s_m[KS][ROWS], s_l[KS][ROWS];
    __shared__ PairRanks<WHOLE ? 1 : NT> s_rank;

    // LDS positions (in 16-byte granules inside this wave's area).
    //   K granule (row r, granule c) is the operand of lane (c & 3, r & 15) for (sub = r >> 4, kk = c >> 2):
    //   position (sub 4 + kk) 64 + (c & 3) 16 + ((r & 15) ^ c)
    uint32_t *area = s_big + wave * AREA_WORDS;
    uint32_t kst_pos[4];        // store position of K load i: kst_pos[i & 3] + (i >> 2) * 256
#pragma unroll
    for (int j = 0; j < 4; ++j) kst_pos[j] = (lc >> 2) * 64 + (lc & 3) * 16 + ((4 * j + lj) ^ lc);
    uint32_t kld_pos[4];        // operand position for kk: kld_pos[kk] + sub * 256
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) kld_pos[kk] = kk * 64 + lj * 16 + (lc ^ (4 * kk + lj));
    //   V: column 8 lc + e of the lane's 8x8 block is the operand of lane 8 (lc & 1) + e for d-tile
    //   lc >> 1.  Position of (d-tile nt, lane hi 8 + lo) in the k-group's 128 granules:
    //   nt 16 + hi 8 + (lo ^ ((2 nt + hi) & 7)): eight neighbouring lanes cover all banks in the
    //   stores (fixed e: 2 nt + hi = lc runs through eight values) and in the loads (fixed nt: lo does).
    const uint32_t vst_base = lj * 128 + lc * 8;            // store position = vst_base + (e ^ vst_x)
    const uint32_t vst_x = lc & 7;
    const uint32_t vld_base = lj * 128 + (lc >> 3) * 8;     // load position = vld_base + nt 16 + (vld_x ^ ((2 nt) & 7))
    const uint32_t vld_x = (lc & 7) ^ (lc >> 3);
    // Per-lane byte offsets inside a tile (row pitch 256 B).
    //   K load i (0..7): row 4 i + lj, 16-byte granule lc  ->  i * 1024 + lane * 16
    //   V load s (0..7): row (s < 4 ? 0 : 16) + 4 lj + (s & 3), granule lc
    const uint32_t k_lane_off = lane * 16;
    const uint32_t v_lane_off = lj * 1024 + lc * 16;
    const float c2 = p.scale_log2;      // >= 0 (checked by the host)
    const uint16_t *qb = static_cast<const uint16_t *>(p.q);

    // ---- this workgroup's segment: unit (b, g, rt), tiles [t_begin, t_end) of total_tiles
    int b, g, rt, t_begin, t_end, total_tiles, L;
    bool direct = true;
    size_t part_row = 0;                // first row of this segment's partial in the workspace
    u32x4 kraw[8], vcur[8];             // the K and V tile requested last
    if constexpr (WHOLE) {
        g = blockIdx.x; b = blockIdx.z; rt = blockIdx.y;
        L = p.prefix_len[b];
        const size_t slab = ((size_t)b * p.H_kv + g) * (size_t)p.L_stride * (D * 2);
        const __amdgpu_buffer_rsrc_t rk = make_rsrc(static_cast<const char *>(p.k_prefix) + slab, (uint32_t)p.L_stride * (D * 2));
        const __amdgpu_buffer_rsrc_t rv = make_rsrc(static_cast<const char *>(p.v_prefix) + slab, (uint32_t)p.L_stride * (D * 2));
#pragma unroll
        for (int i = 0; i < 8; ++i) kraw[i] = __builtin_amdgcn_raw_buffer_load_b128(rk, k_lane_off + i * 1024, ks * TILE_BYTES, 0);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            vcur[i] = __builtin_amdgcn_raw_buffer_load_b128(rv, v_lane_off + ((i < 4) ? 0 : 4096) + (i & 3) * 256, ks * TILE_BYTES, 0);
        __builtin_amdgcn_sched_barrier(0);
        L = max(0, min(L, p.L_stride));
        total_tiles = (L + KT - 1) / KT + p.tiles_tree;
        t_begin = 0;
        t_end = total_tiles;
    } else {
        // (the ranking, which waits for every length, only where the launch does not fit the chip at once)
        g = blockIdx.x; b = blockIdx.z;
        rt = blockIdx.y % p.n_row_tiles;
        int chunk = blockIdx.y / p.n_row_tiles;
        if (p.rank_pairs)
            longest_first(p, s_rank, tid, (int)(blockIdx.z * p.n_chunks_max) + chunk, p.chunk_tiles, p.split_bias, p.even_units,
                          [&](int seq) { return max(0, min(p.prefix_len[seq], p.L_stride)); }, &b, &chunk, &L);
        else
            L = max(0, min(p.prefix_len[b], p.L_stride));
        total_tiles = (L + KT - 1) / KT + p.tiles_tree;
        int n_seg, seg;
        split_tiles(total_tiles, p.chunk_tiles, p.split_bias, p.even_units, p.even_n, &n_seg, &seg);
        t_begin = chunk * seg;
        if (t_begin >= total_tiles) return;
        t_end = min(total_tiles, t_begin + seg);
        direct = (n_seg == 1);
        part_row = (((size_t)b * p.H_kv + g) * p.n_chunks_max + chunk) * (size_t)p.R + (size_t)rt * ROWS;
    }
    {
        const int tilesP = (L + KT - 1) / KT;
        const int row0 = rt * ROWS;

        // Q operand, held in registers: lane (lj, lc) has Q[row0 + WROWS rh + 16 mt + lc][32 kk + 8 lj .. +7].
        // Lanes past the last row repeat it (their results are not written): nothing looks at the
        // values here, so that the first K/V requests go out right behind these loads.
        const int my_parent = WHOLE || t_end > tilesP ? parent_of_thread(p, b) : -1;
        bf16x8 qreg[MT][4];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int rr = min(row0 + WROWS * rh + 16 * mt + lc, p.M - 1);
            const int node = rr / p.G, hh = rr % p.G;
            const uint16_t *src = qb + (((size_t)b * p.N + node) * p.H_q + (size_t)g * p.G + hh) * D + 8 * lj;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) qreg[mt][kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(src + 32 * kk));
        }

        f32x4 oacc[8][MT];
#pragma unroll
        for (int nt = 0; nt < 8; ++nt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) oacc[nt][mt] = (f32x4){0.f, 0.f, 0.f, 0.f};
        float m_used[MT], l_part[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) { m_used[mt] = M_INIT; l_part[mt] = 0.f; }

        const size_t kv_head = (size_t)b * p.H_kv + g;
        // K and V of this (sequence, KV head) are read through buffer resources whose extent is
        // exactly the valid rows (prefix_len rows of the cache slab, N rows of the tree block):
        // the tile base is a scalar offset, the lane offset a constant, and rows past the end of
        // a partial tile read as zero instead of leaving the array (their scores are masked).
        // (paged cache: the prefix resources are empty and every prefix tile gets a resource of
        // its own over the page slice it lies in)
        const __amdgpu_buffer_rsrc_t rs_kpre = make_rsrc(static_cast<const char *>(p.k_prefix) + (PAGED ? 0 : kv_head * (size_t)p.L_stride * (D * 2)), PAGED ? 0u : (uint32_t)L * (D * 2));
        const __amdgpu_buffer_rsrc_t rs_vpre = make_rsrc(static_cast<const char *>(p.v_prefix) + (PAGED ? 0 : kv_head * (size_t)p.L_stride * (D * 2)), PAGED ? 0u : (uint32_t)L * (D * 2));
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
        auto load_k = [&](const TileRef &r) {
            __amdgpu_buffer_rsrc_t rs = r.tree ? rs_ktre : rs_kpre;
            if (PAGED && r.paged) rs = make_rsrc(static_cast<const char *>(p.k_prefix) + r.page_off, (uint32_t)r.nvalid * (D * 2));
#pragma unroll
            for (int i = 0; i < 8; ++i) kraw[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, k_lane_off + i * 1024, r.off, 0);
        };
        auto load_v = [&](const TileRef &r) {
            __amdgpu_buffer_rsrc_t rs = r.tree ? rs_vtre : rs_vpre;
            if (PAGED && r.paged) rs = make_rsrc(static_cast<const char *>(p.v_prefix) + r.page_off, (uint32_t)r.nvalid * (D * 2));
#pragma unroll
            for (int s = 0; s < 8; ++s)
                vcur[s] = __builtin_amdgcn_raw_buffer_load_b128(rs, v_lane_off + ((s < 4) ? 0 : 4096) + (s & 3) * 256, r.off, 0);
        };

        int t = t_begin + ks;
        if (!WHOLE || (ks + 1) * KT > L) {
            load_k(tile_ref(t));
            load_v(tile_ref(t));
        }
        // the masks are needed from the first tree tile on; built while the first loads are in flight
        if (t_end > tilesP) {
            build_ancestor_masks(p, my_parent, s_anc, s_parent);
            __syncthreads();
        }
        // PLAIN (a promise of the caller): tile t and the tile requested during this step are whole
        // prefix tiles inside the segment.  Nothing is masked, the step is one straight run of
        // instructions up to the (rare) raise of the running maxima, and with a contiguous cache
        // the tile references are plain offsets (a paged cache still looks its pages up).
        auto plain_ref = [&](int t) {
            TileRef r;
            r.off = t * TILE_BYTES; r.nvalid = KT; r.tree = false; r.tt = 0; r.page_off = 0; r.paged = false;
            return r;
        };
        auto tile_step = [&](const int t, auto plain) __attribute__((always_inline)) {
            constexpr bool PLAIN = decltype(plain)::value;
            const TileRef cur = PLAIN ? plain_ref(t) : tile_ref(t);
            // Both K and V run one tile ahead of their use: K(t) goes from its load registers to LDS
            // (operand order) and K(t + KS) is requested into the same registers; V(t + KS) is
            // requested further down, as soon as V(t) has left its registers.
#pragma unroll
            for (int i = 0; i < 8; ++i)
                *reinterpret_cast<u32x4 *>(area + 4 * (kst_pos[i & 3] + (i >> 2) * 256)) = kraw[i];
            load_k(PLAIN && !PAGED ? plain_ref(t + KS) : tile_ref(t + KS));
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

            // S^T[key][row] = sum_d K[key][d] Q[row][d]   (raw, the softmax scale is applied in the exponent)
            f32x4 sacc[2][MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) { sacc[0][mt] = (f32x4){0.f, 0.f, 0.f, 0.f}; sacc[1][mt] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
            // operands are fetched from LDS four at a time ahead of the eight MFMAs that use them, so
            // that one LDS latency is exposed per group instead of one per operand
#pragma unroll
            for (int kh = 0; kh < 2; ++kh) {
                bf16x8 kop[2][2];
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2) {
                    const int kk = 2 * kh + k2;
                    kop[k2][0] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(area + 4 * kld_pos[kk]));
                    kop[k2][1] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(area + 4 * (kld_pos[kk] + 256)));
                }
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        sacc[0][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[k2][0], qreg[mt][2 * kh + k2], sacc[0][mt], 0, 0, 0);
                        sacc[1][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[k2][1], qreg[mt][2 * kh + k2], sacc[1][mt], 0, 0, 0);
                    }
            }
            // lane (lj, lc) now holds, for its row 16 mt + lc, keys 16 sub + 4 lj + i
            const bool masked = !PLAIN && (cur.nvalid < KT || cur.tree);
            uint32_t onmask[MT];
            if (masked) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    // the node of this lane's row is recomputed here (tree tiles are rare) rather than
                    // kept in a register across the whole loop
                    const int node_m = min(row0 + WROWS * rh + 16 * mt + lc, p.M - 1) / p.G;
                    uint32_t vis = cur.tree ? s_anc[node_m][cur.tt] : 0xffffffffu;
                    if (cur.nvalid < KT) vis &= (1u << cur.nvalid) - 1u;
                    onmask[mt] = vis;
#pragma unroll
                    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (!((vis >> (16 * sub + 4 * lj + i)) & 1u)) sacc[sub][mt][i] = -INFINITY;
                }
            }
            // online softmax with a lazily raised running max (scaled, base-2 domain)
            settle_scores(sacc[0][0], sacc[0][1], sacc[1][0], sacc[1][1]);
            bool raise = false;
            float lmax[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
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
                    for (int nt = 0; nt < 8; ++nt) oacc[nt][mt] *= alpha;
                }
            }
            bf16x8 pop[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                float pv[8];
#pragma unroll
                for (int sub = 0; sub < 2; ++sub)
#pragma unroll
                    for (int i = 0; i < 4; ++i) pv[4 * sub + i] = fast_exp2(fmaf(sacc[sub][mt][i], c2, -m_used[mt]));
                if (masked) {
                    // also covers scale == 0, where a masked score can not be told apart by its value
#pragma unroll
                    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (!((onmask[mt] >> (16 * sub + 4 * lj + i)) & 1u)) pv[4 * sub + i] = 0.f;
                }
                l_part[mt] += ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));
                u32x4 pk = {pack_bf16(pv[0], pv[1]), pack_bf16(pv[2], pv[3]), pack_bf16(pv[4], pv[5]), pack_bf16(pv[6], pv[7])};
                pop[mt] = __builtin_bit_cast(bf16x8, pk);
            }

            // V tile -> V^T operands (the K operands in the area are dead by now: LDS ops of one wave
            // execute in order)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int w = e >> 1;
                const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
                u32x4 o;
                o[0] = __builtin_amdgcn_perm(vcur[1][w], vcur[0][w], sel);
                o[1] = __builtin_amdgcn_perm(vcur[3][w], vcur[2][w], sel);
                o[2] = __builtin_amdgcn_perm(vcur[5][w], vcur[4][w], sel);
                o[3] = __builtin_amdgcn_perm(vcur[7][w], vcur[6][w], sel);
                *reinterpret_cast<u32x4 *>(area + 4 * (vst_base + (vst_x ^ e))) = o;
            }
            load_v(PLAIN && !PAGED ? plain_ref(t + KS) : tile_ref(t + KS));
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // O^T[d][row] += sum_key V[key][d] P[row][key]
#pragma unroll
            for (int nh = 0; nh < 2; ++nh) {
                bf16x8 vop[4];
#pragma unroll
                for (int n4 = 0; n4 < 4; ++n4) {
                    const int nt = 4 * nh + n4;
                    vop[n4] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(area + 4 * (vld_base + nt * 16 + (vld_x ^ ((2 * nt) & 7)))));
                }
#pragma unroll
                for (int n4 = 0; n4 < 4; ++n4)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        oacc[4 * nh + n4][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop[n4], pop[mt], oacc[4 * nh + n4][mt], 0, 0, 0);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        {
            const int t_plain = min(t_end, L / KT);
            for (; t + KS < t_plain; t += KS) tile_step(t, std::true_type());
        }
        for (; t < t_end; t += KS) tile_step(t, std::false_type());

        // ---- epilogue: merge the key streams.  Every wave leaves its (m, l) per row and its O, unscaled, as
        // float4 rows [row][PO] in its own area; behind one barrier all threads add up the KS areas
        // of a row group, each brought to the largest of the maxima, and write the result.
        // The lane indices are re-derived from an opaque copy so that the epilogue's address
        // arithmetic is not hoisted above the tile loop, where it would cost registers (and spill).
        int tid_e = tid;
        asm volatile("" : "+v"(tid_e));
        const int lj_e = (tid_e & 63) >> 4, lc_e = tid_e & 15;
        float *farea = reinterpret_cast<float *>(area);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            float lt = l_part[mt];
            lt += __shfl_xor(lt, 16);
            lt += __shfl_xor(lt, 32);
            if (lj_e == 0) { s_m[ks][WROWS * rh + 16 * mt + lc_e] = m_used[mt]; s_l[ks][WROWS * rh + 16 * mt + lc_e] = lt; }
#pragma unroll
            for (int nt = 0; nt < 8; ++nt)          // d = 16 nt + 4 lj + (0..3), row 16 mt + lc
                *reinterpret_cast<f32x4 *>(farea + (16 * mt + lc_e) * PO + 16 * nt + 4 * lj_e) = oacc[nt][mt];
        }
        __syncthreads();
        const int rows_valid = min(ROWS, p.M - row0);
        // one 16-byte piece per lane, neighbouring lanes neighbouring pieces: every store
        // instruction of the partial covers whole 512-byte rows
#pragma unroll
        for (int j = 0; j < ROWS * 32 / NT; ++j) {
            const int r = (tid_e >> 5) + j * (NT / 32), d4 = tid_e & 31;
            if (r >= rows_valid) break;
            const int rg = r / WROWS, rl = r % WROWS;
            float ms = s_m[0][r], ls = 0.f;
#pragma unroll
            for (int k2 = 1; k2 < KS; ++k2) ms = fmaxf(ms, s_m[k2][r]);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k2 = 0; k2 < KS; ++k2) {
                const float f = fast_exp2(s_m[k2][r] - ms);
                ls += f * s_l[k2][r];
                acc += f * *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(s_big + (rg * KS + k2) * AREA_WORDS) + rl * PO + 4 * d4);
            }
            if (direct) {
                const float inv = 1.0f / ls;
                const uint2 pk = {pack_bf16(acc[0] * inv, acc[1] * inv), pack_bf16(acc[2] * inv, acc[3] * inv)};
                const int gr = row0 + r, node = gr / p.G, hh = gr % p.G;
                uint16_t *ob = static_cast<uint16_t *>(p.out);
                // outputs and partials are written once and not read again by this kernel: stored
                // non-temporally they do not sit dirty in L2 until the end-of-kernel write-back
                __builtin_nontemporal_store((u32x2){pk.x, pk.y}, reinterpret_cast<u32x2 *>(ob + (((size_t)b * p.N + node) * p.H_q + (size_t)g * p.G + hh) * D + 4 * d4));
            } else {
                __builtin_nontemporal_store(acc, reinterpret_cast<f32x4 *>(p.part_o + (part_row + r) * D + 4 * d4));
                if (d4 == 0) {
                    p.part_m[part_row + r] = ms;
                    p.part_l[part_row + r] = ls;
                }
            }
        }
    }
}

// Merges the chunks of one unit: out = sum_c 2^(m_c - m*) O_c / sum_c 2^(m_c - m*) l_c.
// A block of 256 threads takes 8 / S rows: S threads share a 16-byte piece of a row, each with every
// S-th chunk, eight of them requested before the first use (one trip to memory for up to 8 S chunks),
// and meet in LDS.  Bound by latency for few chunks (4 us), by the partials beyond.  S grows with the
// number of chunks: with one thread per piece walking all of them, 43 chunks of 224 rows and 8 KV
// heads took 32 us (40 MB of partials, two dependent trips per chunk).
// Blocks with blockIdx.x == nx_combine (H_kv B of them) carry the walk of a verification that ran
// before this launch on the same stream (one wavefront per sequence), when the caller asked for that.
template <int S>
__global__ __launch_bounds__(256) void tree_attn_combine_kernel(AttnParams p, int nx_combine, WalkParams w)
{
    constexpr int D = 128, ROWS = 8 / S;
    if ((int)blockIdx.x >= nx_combine) {
        const int first = (int)(blockIdx.z * gridDim.y + blockIdx.y) * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        for (int wb = first; wb < w.B; wb += (int)(gridDim.z * gridDim.y) * 4) walk_sequence(w, wb);
        return;
    }
    const int g = blockIdx.y, b = blockIdx.z;
    // both by scalar loads, together (the plain pointers would become one vector load after the other)
    typedef const int32_t __attribute__((address_space(4))) *const_i32_ptr;
    const const_i32_ptr lens = (const_i32_ptr)(uintptr_t)p.prefix_len;
    const const_i32_ptr chunk_word = p.chunk_of_launch ? (const_i32_ptr)(uintptr_t)p.chunk_of_launch : lens;
    const int L = max(0, min(lens[b], p.L_stride)), chunk_of_launch = *chunk_word;
    const int chunk_tiles = p.chunk_of_launch ? chunk_of_launch : p.chunk_tiles;
    const int total_tiles = (L + KT - 1) / KT + p.tiles_tree;
    int n_chunks, seg;
    split_tiles(total_tiles, chunk_tiles, chunk_tiles / 2, p.even_units, p.even_n, &n_chunks, &seg);
    n_chunks = (total_tiles + seg - 1) / seg;      // segments that are not empty
    if (n_chunks <= 1) return;      // the attention kernel wrote the output itself
    const int d4 = threadIdx.x & 31;        // 16-byte piece of the row
    const int share = (threadIdx.x >> 5) % S, rl = (threadIdx.x >> 5) / S, r = blockIdx.x * ROWS + rl;
    if (S == 1 && r >= p.M) return;
    const int rr = min(r, p.M - 1);         // (a row past the end is read again and not written)
    const size_t base = (((size_t)b * p.H_kv + g) * p.n_chunks_max) * (size_t)p.R + rr;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float ls = 0.f, ms = M_INIT;
    // Slots past n_chunks re-read chunk 0 (a cache hit) with weight zero, so the loads stay
    // unconditional; two sizes keep that waste below a factor of two.
    auto merge = [&](int c0, auto maxc, auto first) __attribute__((always_inline)) {
        constexpr int MAXC = decltype(maxc)::value;
        float mc[MAXC], lc[MAXC];
        f32x4 oc[MAXC];
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            const int c = c0 + i * S;
            const bool on = c < n_chunks;
            const size_t u = base + (size_t)(on ? c : 0) * p.R;
            mc[i] = on ? p.part_m[u] : M_INIT;
            lc[i] = on ? p.part_l[u] : 0.f;
            oc[i] = *reinterpret_cast<const f32x4 *>(p.part_o + u * D + 4 * d4);
        }
        const float m_old = ms;
#pragma unroll
        for (int i = 0; i < MAXC; ++i) ms = fmaxf(ms, mc[i]);
        if constexpr (!decltype(first)::value) {
            const float alpha = exp2f(m_old - ms);
            ls *= alpha;
            acc *= alpha;
        }
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            const float fsc = (c0 + i * S < n_chunks) ? exp2f(mc[i] - ms) : 0.f;
            ls += fsc * lc[i];
            acc += fsc * oc[i];
        }
    };
    if (n_chunks <= 4 * S) {
        merge(share, std::integral_constant<int, 4>(), std::true_type());
    } else {
        merge(share, std::integral_constant<int, 8>(), std::true_type());
        if constexpr (S == 8)               // (a smaller S never has more than 8 S)
            for (int c0 = share + 8 * S; c0 < n_chunks; c0 += 8 * S) merge(c0, std::integral_constant<int, 8>(), std::false_type());
    }
    if constexpr (S > 1) {
        __shared__ f32x4 s_acc[8][32];
        __shared__ float s_ms[8], s_ls[8];
        s_acc[rl * S + share][d4] = acc;
        if (d4 == 0) { s_ms[rl * S + share] = ms; s_ls[rl * S + share] = ls; }
        __syncthreads();
        if (share > 0) return;
#pragma unroll
        for (int i = 0; i < S; ++i) ms = fmaxf(ms, s_ms[rl * S + i]);
        acc = (f32x4){0.f, 0.f, 0.f, 0.f};
        ls = 0.f;
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const float fsc = exp2f(s_ms[rl * S + i] - ms);
            ls += fsc * s_ls[rl * S + i];
            acc += fsc * s_acc[rl * S + i][d4];
        }
    }
    if (r >= p.M) return;
    const float inv = 1.0f / ls;
    const uint2 pk = {pack_bf16(acc[0] * inv, acc[1] * inv), pack_bf16(acc[2] * inv, acc[3] * inv)};
    const int node = r / p.G, hh = r % p.G;
    uint16_t *ob = static_cast<uint16_t *>(p.out);
    __builtin_nontemporal_store((u32x2){pk.x, pk.y}, reinterpret_cast<u32x2 *>(ob + (((size_t)b * p.N + node) * p.H_q + (size_t)g * p.G + hh) * D + 4 * d4));
}

// Launch-plan overrides of mcsd_attn_plan_override (0 = automatic), process-wide.
std::atomic<int> g_force_variant{0}, g_force_chunk_tiles{0}, g_force_target_wgs{0};

}  // namespace

bool make_attn_plan(const mcsd_attn_desc &d, AttnPlan *plan)
{
    AttnPlan pl = {};
    const int G = d.H_q / d.H_kv;
    const int n_rows_tree = d.N + (d.root_row ? 1 : 0);      // rows of the tree block
    pl.rows_per_kv = n_rows_tree * G;
    pl.use_mfma = (d.dtype == MCSD_DTYPE_BF16 && d.d == 128);
    if (!pl.use_mfma) {
        if (d.d > MCSD_MAX_HEAD_DIM) return false;
        *plan = pl;
        return true;
    }
    // Kernel variant (4 waves, two workgroups per CU): 0 = 32 rows x 4 key streams for
    // rows_per_kv <= 32, 1 = 2 x 32 rows x 2 key streams up to 64 rows, 2 = 4 x 32 rows on one
    // key stream with tiles shared through LDS beyond that (several row tiles per KV head:
    // the matrix cores are the limit there, and the shared tiles cut the per-wave staging work).
    pl.variant = pl.rows_per_kv <= 32 ? 0 : (pl.rows_per_kv <= 64 ? 1 : 2);
    {
        const int forced_variant = g_force_variant.load();     // 1-based, 0 = automatic
        if (forced_variant >= 1 && forced_variant <= 3) pl.variant = forced_variant - 1;
    }
    pl.row_tile = 32 << pl.variant;
    const int key_streams = 4 >> pl.variant;
    pl.n_row_tiles = (pl.rows_per_kv + pl.row_tile - 1) / pl.row_tile;
    pl.tiles_prefix_max = (d.L_stride + KT - 1) / KT;
    pl.tiles_tree = (n_rows_tree + KT - 1) / KT;
    const long total_max = pl.tiles_prefix_max + pl.tiles_tree;
    const long units = (long)d.B * d.H_kv * pl.n_row_tiles;
    // Every segment pays a fixed prologue (Q, first tiles) and epilogue (merge, possibly one
    // [rows][d] fp32 partial written and read back by the combine kernel), which runs shorter
    // than 6 tiles per key stream do not amortise (measured).
    const long min_run = 6 * key_streams;

    // Workgroups per launch if every sequence had the maximum length (the CUs hold 512 at a time).
    // More, shorter segments balance the end of the launch better but every segment of a split
    // unit costs one fp32 partial written and read back; 1024 measured best both where the
    // kernel is HBM-bound (that traffic competes with the cache stream) and where the matrix
    // cores are the limit (768 .. 1536 within 2 %; beyond that the merge kernel grows faster
    // than the attention kernel shrinks).
    const int forced_target = g_force_target_wgs.load();
    const long target_wgs = forced_target > 0 ? forced_target : 1024;
    long chunk = (total_max * units + target_wgs - 1) / target_wgs;
    chunk = ((chunk + key_streams - 1) / key_streams) * key_streams;
    if (chunk < min_run) chunk = min_run;
    // A split plan that leaves CUs idle: with the merge launch paid anyway, segments of 3 tiles per key
    // stream (2 with four streams) as long as all fit one per CU; on shared tiles only up to the eight
    // that the merge takes in one trip.  With the merge, segments of 6 tiles per stream / these: 60 rows,
    // 32 KV heads, 2000 keys 19.3 / 16.0 us; 48 rows, 2 x 8 KV heads, 2000 keys 16.0 / 12.9; 24 rows, 8 KV heads,
    // 2000 keys 13.1 / 11.4; 112 rows, 9 x 8 KV heads, 300 keys 15.0 / 14.6, but 500 keys 16.1 / 18.3.
    if (forced_target <= 0 && (total_max + chunk / 2) / chunk > 1) {
        long fine = (total_max * units + 255) / 256;
        if (pl.variant == 2 && fine < (total_max + 7) / 8) fine = (total_max + 7) / 8;
        fine = (fine + key_streams - 1) / key_streams * key_streams;
        const long least = key_streams == 4 ? 8 : 3 * key_streams;
        if (fine < least) fine = least;
        if (fine < chunk) chunk = fine;
    }
    const int forced = g_force_chunk_tiles.load();
    // (see split_tiles.  By the real lengths, on the device: one sequence, 32 heads, a cache of 8192 rows,
    // 8192 / 5000 / 4000 / 2000 / 1000 keys: segments of 24 tiles 39.4 / 21.2 / 19.7 / 16.3 / 18.6 us, lengthened by
    // the capacity 28.0 / 21.9 / 20.1 / 18.1 / 17.6, here 28.6 / 20.2 / 19.0 / 15.3 / 17.5; 56 rows, 16 heads, a cache of
    // 16384: 16384 / 6000 keys 69.0 / 29.8, 41.8 / 19.4, 41.7 / 19.6; two sequences of 8000 keys, 16 heads 40.0, 26.9, 27.6)
    pl.even_units = pl.variant < 2 && forced_target <= 0 && forced <= 0 && units <= 128 ? (int)units : 0;
    if (forced > 0) chunk = forced;
    if (chunk > total_max) chunk = total_max;
    pl.chunk_tiles = (int)chunk;
    pl.n_chunks_max = (int)((total_max + chunk - 1) / chunk);
    if (pl.even_units) {        // (no shorter sequence has more segments then; workgroups without one would disturb the spread over the CUs)
        const long wgs = units * ((total_max + chunk / 2) / chunk);
        if (wgs > 256 && wgs < 448) pl.n_chunks_max = (int)(256 / units);
    }
    pl.partial_stride_rows = (size_t)pl.n_row_tiles * pl.row_tile;
    if (pl.n_chunks_max > 1) {
        size_t elems = (size_t)d.B * d.H_kv * pl.n_chunks_max * pl.partial_stride_rows * (size_t)(d.d + 2);
        pl.ws_bytes = (elems * sizeof(float) + 255) & ~(size_t)255;
        // (see segment_tiles; not with a forced plan, and not where the units alone fill the chip)
        if (pl.variant == 2 && d.B <= 64 && units <= 256 && units * pl.n_chunks_max > 512 &&
            forced <= 0 && forced_target <= 0) {
            pl.chunk_on_device = true;
            pl.ws_bytes += 256;
        }
    } else {
        pl.ws_bytes = 0;
    }
    // Launches that leave CUs idle and caches of middling capacity: no segments and no merge, but all keys of 32
    // rows and a slice of the output columns per workgroup of eight waves (tree_attn_bf16_kernel).  What
    // a wave does in its step is the time here, so the fewer columns it has the better: slices of
    // 32, 64 or 128 columns, as many as fit one workgroup per CU.  The host knows the capacity only, and the lines
    // go by it: with spare rows a launch keeps segments and merge however short the sequences are.  They are where
    // segments or, with up to 32 rows, the kernel above with its four waves get ahead (that one splits from 36 tiles on).
    // us without / with this, at 200, 500, 1000, 1500, 2000 keys, caches and sequences full:
    //   28 rows,  32 KV heads (32 columns)     7.3/7.1  10.6/9.4  17.1/11.6 12.6/13.7 14.3/15.8
    //   28 rows, 128 KV heads (64)             8.5/9.3  11.6/11.4 18.3/15.9 23.6/21.1 31.2/28.5
    //   28 rows, 256 KV heads (128)            9.8/12.0 15.8/16.8 35.4/28.7 44.1/38.8 58.9/50.0
    //   56 rows,  16 KV heads (32)            11.1/7.7  13.3/8.7  13.1/11.2 15.8/13.6 14.9/15.9
    //   56 rows,  40 KV heads (64)            11.4/8.4  14.3/10.4 14.4/12.9 16.4/15.3 19.3/17.6
    //   56 rows, 128 KV heads, GQA 2 (128)    10.7/10.9 18.6/13.4 (30: 7.9/8.4, 300: 12.4/11.5) 31.2/23.9 47.4/31.3
    //   60 rows, 128 KV heads (128)           12.3/11.6 17.8/13.8 22.5/18.2 33.6/25.9 45.3/32.5
    //   112 rows,  8 KV heads (32)            13.6/7.3  11.5/8.5  12.6/10.5 15.5/12.9 14.3/14.8
    //   112 rows, 32 KV heads (64)            14.1/8.3  13.8/10.3 15.3/12.9 18.0/15.5 21.0/17.5 (3000: 26.1/22.4)
    //   112 rows, 64 KV heads (128)           14.8/10.2 16.1/12.8 21.0/15.9 25.6/19.0 25.3/22.1
    //   672 rows,  8 KV heads (128)           14.5/10.0 15.5/11.7 20.2/14.7 23.2/18.0 23.3/21.6
    // One sequence full and the others of 100 keys: the long one has its slices' CUs only, where segments
    // take those of the short ones as well.  At 1500, 2000, 2500 keys (1600, 2000, 2400 where marked *):
    //   28 rows, 4 x 32 KV heads  15.4/15.6 17.5/17.6 19.3/19.8     8 x 32  17.3/20.1 19.1/23.6 19.9/30.4
    //   60 rows, 4 x 32           18.2/18.5 20.0/21.5 22.7/24.1
    //   112 rows, 4 x 8           15.8/14.5 18.1/17.0 18.4/19.0     3 x 8*  15.3/14.5 15.4/16.7 15.5/18.0
    //   224 rows, 2 x 8           16.5/14.2 17.4/17.3 17.6/19.5     8 x 4*  16.4/17.8 16.5/20.3 16.8/21.9
    // The upper lines are where that loss is no larger yet than the gain of full sequences.  These figures are of inputs
    // that the memory-side cache holds; from memory, 2000 keys, full and one full: 112 rows, 4 x 8 24.2/20.0 and
    // 19.2/18.6, 3 x 8 20.6/19.4 and 16.3/18.8 (1500: 17.8/16.4, 16.3/15.6), 60 rows, 4 x 32 47.9/33.4 and 22.4/26.8,
    // 2 x 32 24.3/22.8 and 21.6/21.4, but 56 rows, 40 heads 20.0/21.7 (1500: 17.8/18.0; warm 17.9/17.3 and 16.5/15.5).
    // 28 rows (4 and 24 alike) by more than 160 workgroups, since the tiles go straight into LDS (tree_attn_any.hip), from memory, without / with
    // this: full; lengths spread evenly from an eighth on; one full and the others of 100 keys:
    //   6 x 32 heads   1110 keys  30.3/25.2 25.9/21.9 17.9/17.3   1560  39.1/32.4 27.2/26.9 17.8/19.2   2000  49.2/39.5 35.0/32.6 16.2/20.6
    //   8 x 32                    36.2/30.9 27.6/23.0 17.8/16.7         47.0/40.4 35.6/31.1 19.7/18.9         58.8/50.4 39.2/37.2 19.9/22.2
    //   11 x 16                   29.5/24.6 27.3/21.1 15.8/14.6         38.3/30.4 26.6/26.0 17.8/17.3
    //   5 x 32 (160)  1500  34.7/28.1 22.7/25.6 17.8/19.7
    // Measured again between, 1250 and 1400 keys, with all of a quarter and all of 60 keys besides:
    //   6 x 32  34.2/29.1 26.5/24.0 19.3/19.3 16.4/12.2 11.9/9.8    36.2/31.7 26.2/26.2 19.3/20.6 17.5/12.7 12.0/9.8
    //   7 x 32  37.2/32.1 29.5/25.7 17.7/18.6 16.7/12.9 12.2/10.1   39.5/36.0 29.2/28.6 19.0/20.5 17.5/13.4 12.2/10.1
    // One full sequence among short ones pays up to 1.09 there for 0.73 to 0.91 of the others.
    // The lower lines, the kernel above whole / this, at 32, 96, 150, 180, 210, 240, 350 keys, all full (lengths spread: alike or better):
    //   28 rows,  32 KV heads (32)   7.6/7.1 7.7/7.1 7.8/7.6 7.6/7.6 7.6/7.7 8.5/8.1 9.5/8.8     (7 and 8 tiles go twice round its four waves)
    //   28 rows,   8 KV heads (32)   6.8/6.2 7.3/6.8 7.6/7.6 7.4/7.6 7.4/7.6 8.4/7.9 8.5/7.9
    //   28 rows,  96 KV heads (64)   30: 7.7/7.7, 60: 7.8/8.1, 200: 8.5/9.2, 400: 11.3/11.0, 550: 12.7/12.0
    //   28 rows, 192 KV heads (128)  30: 8.0/9.5, 60: 8.3/10.1, 200: 9.5/11.7, 550: 14.9/16.6, 700: 16.8/18.5
    //   60 rows (nodes), 128 KV heads (128)  10.2/9.8 10.7/10.8 12.0/11.1 12.1/11.4 13.0/11.8
    //   56 rows (nodes),  80 KV heads (128)   9.6/9.0 10.1/10.0 11.6/10.8 11.5/10.9 12.3/11.2
    //   56 rows, 28 nodes, 128 KV heads (128) 8.7/9.4  9.4/10.6 10.2/10.5 11.3/11.0 11.3/11.1 12.2/11.6    (one tile of the tree, not two)
    // Trees of more than 32 rows with the root's, one query head per KV head, from memory, at 30, 96, 160, 224 keys and with sequences of 60 keys in a cache of 224: the
    // kernel above does more for every node of the tree, so from about 50 rows on it is behind.
    //   33 rows, 128 KV heads   9.4/9.4  9.5/10.2 10.3/10.6 11.2/11.5  9.3/9.9     80 KV heads   9.3/9.2 9.1/9.6 10.1/10.1 11.0/10.8  9.0/9.4
    //   48                      9.9/9.8  9.7/10.2 10.6/10.6 11.7/11.6  9.6/10.1                  9.7/9.4 9.5/9.8 10.4/10.1 11.3/10.7  9.5/9.7
    //   56                     10.2/9.8  9.9/10.3 10.8/10.6 12.1/11.9  9.9/10.1                 10.1/9.4 9.7/9.7 10.6/10.1 11.5/10.7  9.7/9.7
    //   64                     10.6/10.0 10.2/10.5 11.2/10.8 12.0/11.5 10.3/10.3                10.5/9.7 10.0/9.9 10.9/10.2 11.8/10.8 10.1/9.8
    // (The workspace that a split plan of these sizes asks for stays asked for.)
    const long wgs32 = (long)d.B * d.H_kv * ((pl.rows_per_kv + 31) / 32);
    if (wgs32 <= 256 && g_force_variant.load() == 0 && forced <= 0 && forced_target <= 0) {
        const bool some = wgs32 > 64 && wgs32 <= 128;
        long least = 1, most = some && wgs32 > 96 ? 66 : 54;
        if (pl.rows_per_kv <= 32) { least = wgs32 <= 64 ? (total_max <= 6 ? 1 : 9) : (some ? 22 : 25); most = some || wgs32 > 160 ? 50 : 35; }
        else if (pl.rows_per_kv <= 64) { least = wgs32 <= 128 || n_rows_tree > 50 ? 1 : 10; most = wgs32 <= 128 ? 50 : 66; }
        if (total_max >= least && total_max <= most) {
            pl.slice_columns = wgs32 <= 64 ? 32 : (wgs32 <= 128 ? 64 : 128);
            pl.n_chunks_max = 1;
            pl.chunk_on_device = false;
        }
    }
    if ((long)pl.n_chunks_max * pl.n_row_tiles + 256L > 65535L || d.B > 65535) return false;     // (+ rows that may carry a walk)
    *plan = pl;
    return true;
}

int32_t attn_plan_override(int variant, int chunk_tiles, int target_wgs)
{
    if (variant < 0 || variant > 3 || chunk_tiles < 0 || target_wgs < 0) return MCSD_E_SHAPE;
    g_force_variant.store(variant);
    g_force_chunk_tiles.store(chunk_tiles);
    g_force_target_wgs.store(target_wgs);
    return MCSD_OK;
}

int32_t launch_tree_attn(const mcsd_attn_desc &d, const mcsd_attn_bufs &b, const AttnPlan &plan,
                         hipStream_t stream, const mcsd_paged_kv *paged, int phases, const WalkParams *tail_walk)
{
    AttnParams p = {};
    if (paged) {
        p.block_table = paged->block_table; p.page_size = paged->page_size;
        p.n_pages = paged->n_pages; p.max_pages = paged->max_pages_per_seq;
    }
    p.q = b.q; p.k_prefix = b.k_prefix; p.v_prefix = b.v_prefix; p.k_tree = b.k_tree; p.v_tree = b.v_tree;
    p.prefix_len = b.prefix_len; p.parent = b.parent; p.out = b.out;
    p.root_row = d.root_row ? 1 : 0;
    p.B = d.B; p.N = d.N + p.root_row; p.H_q = d.H_q; p.H_kv = d.H_kv; p.G = d.H_q / d.H_kv; p.d = d.d;
    p.L_stride = d.L_stride; p.M = plan.rows_per_kv; p.parent_per_seq = d.parent_per_seq; p.dtype = d.dtype;
    p.scale_log2 = d.scale * LOG2E_F;
    p.n_row_tiles = plan.n_row_tiles; p.chunk_tiles = plan.chunk_tiles; p.n_chunks_max = plan.n_chunks_max;
    p.tiles_tree = plan.tiles_tree; p.R = (int)plan.partial_stride_rows;
    p.split_bias = plan.chunk_tiles / 2;
    p.even_units = plan.even_units;
    p.even_n = plan.even_units ? 256 / plan.even_units : 0;
    p.rank_pairs = d.B * plan.n_chunks_max <= 256 && plan.n_chunks_max > 1 &&
                   (long)d.H_kv * plan.n_row_tiles * plan.n_chunks_max * d.B > 512;
    if (plan.ws_bytes > 0) {
        const size_t rows = (size_t)d.B * d.H_kv * plan.n_chunks_max * plan.partial_stride_rows;
        float *ws = static_cast<float *>(b.workspace);
        p.part_o = ws;
        p.part_m = ws + rows * d.d;
        p.part_l = p.part_m + rows;
        if (plan.chunk_on_device) p.chunk_of_launch = reinterpret_cast<int *>(static_cast<char *>(b.workspace) + plan.ws_bytes - 256);
    }
    if (!plan.use_mfma) return launch_attn_any(p, stream);
    if (plan.slice_columns) return phases & ATTN_PHASE_MAIN ? launch_attn_sliced(p, plan.slice_columns, stream, tail_walk) : MCSD_OK;
    hipError_t e;
    if (phases & ATTN_PHASE_MAIN) {
        // an unsplit attention has no merge launch to carry the walk: it rides on this one
        WalkParams mw = {};
        int walk_rows = 0;
        if (tail_walk && plan.n_chunks_max == 1) { mw = *tail_walk; walk_rows = 1; }
        const dim3 grid(d.H_kv, plan.n_chunks_max * plan.n_row_tiles + walk_rows, d.B);
        const int streams = 4 >> plan.variant;
        const bool whole = plan.n_chunks_max == 1 && d.L_stride >= KT * streams && first_tiles_ahead(p, streams, 256);      // (see tree_attn_mfma_kernel)
        if (plan.variant == 2) launch_attn_shared(p, grid, stream, mw);
        else if (paged) {
            if (plan.variant == 0) launch_kernel(K_ATTN_MFMA, tree_attn_mfma_kernel<1, 4, true, false>, grid, dim3(256), stream, p, mw);
            else launch_kernel(K_ATTN_MFMA, tree_attn_mfma_kernel<2, 2, true, false>, grid, dim3(256), stream, p, mw);
        } else if (whole) {
            if (plan.variant == 0) launch_kernel(K_ATTN_MFMA, tree_attn_mfma_kernel<1, 4, false, true>, grid, dim3(256), stream, p, mw);
            else launch_kernel(K_ATTN_MFMA, tree_attn_mfma_kernel<2, 2, false, true>, grid, dim3(256), stream, p, mw);
        } else {
            if (plan.variant == 0) launch_kernel(K_ATTN_MFMA, tree_attn_mfma_kernel<1, 4, false, false>, grid, dim3(256), stream, p, mw);
            else launch_kernel(K_ATTN_MFMA, tree_attn_mfma_kernel<2, 2, false, false>, grid, dim3(256), stream, p, mw);
        }
        e = hipGetLastError();
        if (e != hipSuccess) { set_error("tree_attn_mfma launch failed: %s", hipGetErrorString(e)); return MCSD_E_HIP; }
    }
    if ((phases & ATTN_PHASE_COMBINE) && plan.n_chunks_max > 1) {
        WalkParams w = {};
        int walk_blocks = 0;
        if (tail_walk) { w = *tail_walk; walk_blocks = 1; }
        auto merge = [&](auto kernel, int rows) {
            const int nx = (plan.rows_per_kv + rows - 1) / rows;
            launch_kernel(K_ATTN_COMBINE, kernel, dim3(nx + walk_blocks, d.H_kv, d.B), dim3(256), stream, p, nx, w);
        };
        if (plan.n_chunks_max <= 8) merge(tree_attn_combine_kernel<1>, 8);
        else if (plan.n_chunks_max <= 16) merge(tree_attn_combine_kernel<2>, 4);
        else if (plan.n_chunks_max <= 32) merge(tree_attn_combine_kernel<4>, 2);
        else merge(tree_attn_combine_kernel<8>, 1);
        e = hipGetLastError();
        if (e != hipSuccess) { set_error("tree_attn_combine launch failed: %s", hipGetErrorString(e)); return MCSD_E_HIP; }
    }
    return MCSD_OK;
}

}  // namespace mcsd
