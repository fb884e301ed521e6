// Shared by the tree-attention kernels: parameters, buffer resources, small arithmetic helpers,
// the split of a sequence's key tiles into segments and the ancestor masks.
#pragma once

#include <math.h>

#include "mcsd_internal.h"

namespace mcsd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr float LOG2E_F = 1.44269504088896340736f;
constexpr float M_INIT = -1.0e30f;     // "no key seen yet" running max (finite so that differences stay finite)
constexpr float RESCALE_GAP = 8.0f;    // running max is only raised when a score exceeds it by 2^8
constexpr int KT = 32;                 // keys per tile

struct AttnParams {
    const void *q, *k_prefix, *v_prefix, *k_tree, *v_tree;
    const int32_t *prefix_len, *parent;
    void *out;
    float *part_m, *part_l, *part_o;
    int B, N, H_q, H_kv, G, d, L_stride, M;
    int n_row_tiles, chunk_tiles, n_chunks_max, tiles_tree, parent_per_seq, dtype;
    int root_row;         // 1: row 0 of the tree block is the root, N counts it
    int R;                // rows per (b, g) in the partial buffers
    int split_bias;       // see split_tiles
    int even_units, even_n; // units of the launch and 256 / units where one workgroup per CU is wanted, or 0 (see split_tiles)
    int first_ahead;      // ask for the first tiles ahead of the length (see first_tiles_ahead)
    int rank_pairs;       // hand the (sequence, segment) pairs out longest first
    int *chunk_of_launch; // workspace word with the chunk_tiles of this launch, or nullptr: chunk_tiles holds
    float scale_log2;     // scale * log2(e)
    // paged prefix cache (block_table != nullptr): k_prefix / v_prefix are pools
    // [n_pages][H_kv][page_size][d]; logical row r of sequence b lives in page
    // block_table[b][r / page_size], slot r % page_size
    const int32_t *block_table;
    int page_size, n_pages, max_pages;
};


// Whether the workgroups of a launch ask for their first tiles before the length is there, as if the (contiguous)
// cache were full: it saves a trip to memory, but a short prefix in a larger cache then comes behind tiles that
// nothing needs.  Up to 8 MiB of them in all, `tiles` per (sequence, KV head), that costs less than it saves.
// us with / without at 20, 100 and 300 keys of a cache of 300:
//   d 128, 28 rows,  64 KV heads, 4 tiles (4 MiB)   7.2/7.2  7.5/8.3  8.9/9.9
//                   128 (8)                         7.9/7.3  8.1/8.9  9.6/10.2
//                   256 (16)                        9.8/7.7  9.9/9.3  12.1/11.8
//                   512 (32)                        13.6/10.2 13.6/13.1 18.4/18.6
//   d 128, 60 rows, 256, 2 tiles (8)                11.3/10.7 11.5/12.0 14.6/15.1
//   d 64,  28 rows, 128, 8 tiles (8)                6.8/5.7  7.0/6.4  7.5/8.0
//                   256 (16)                        9.3/6.3  9.5/7.8  9.7/10.0
//   d 96,  28 rows, 128, 8 tiles (12)               9.0/6.9  9.3/7.8  9.6/9.9
inline bool first_tiles_ahead(const AttnParams &p, int tiles, uint32_t row_bytes)
{
    return (uint64_t)p.B * p.H_kv * (2u * KT * tiles) * row_bytes <= (8u << 20);
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    bf16x2 v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, v);
}

// Raw buffer resource over [ptr, ptr + bytes): reads past the end return zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *ptr, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(ptr), 0, bytes, 0x00020000);
}

// max(a, b, c) as the one hardware instruction: fmaxf() on values the compiler knows nothing
// about (matrix-instruction results) costs an extra NaN-quieting v_max_f32 x, x per operand.
__device__ __forceinline__ float max3_raw(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// A vector instruction that reads the result of a matrix instruction has to keep a distance
// from it (seven wait states for v_mfma_f32_16x16x32_bf16) which the hardware does not enforce.
// The compiler keeps it for the instructions it selects itself, but not for the text of an asm
// statement: the four score accumulators pass through this statement before max3_raw reads
// them, so every matrix instruction that writes them has been issued before its wait states
// and every reader stands behind them.
__device__ __forceinline__ void settle_scores(f32x4 &a, f32x4 &b, f32x4 &c, f32x4 &d)
{
    asm volatile("s_nop 7\n\ts_nop 1" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}

__device__ __forceinline__ void settle_scores(f32x4 &a, f32x4 &b)
{
    asm volatile("s_nop 7\n\ts_nop 1" : "+v"(a), "+v"(b));
}

// the largest of the eight scores a lane holds for one row (two accumulators of four)
__device__ __forceinline__ float max_of_scores(const f32x4 &s0, const f32x4 &s1)
{
    const float m0 = max3_raw(s0[0], s0[1], s0[2]);
    const float m1 = max3_raw(s0[3], s1[0], s1[1]);
    return max3_raw(max3_raw(m0, m1, s1[2]), s1[3], s1[3]);
}

__device__ __forceinline__ float fast_exp2(float x)
{
    return __builtin_amdgcn_exp2f(x);      // v_exp_f32; results below the normal range flush to 0
}

__device__ __forceinline__ float bf16_bits_to_float(uint32_t bits16)
{
    return __uint_as_float(bits16 << 16);
}

// The T key tiles of a sequence are cut into n segments of seg tiles (the last one possibly
// shorter): n = (T + bias) / chunk_tiles, at least 1.  With bias = chunk_tiles / 2 that is
// T / chunk_tiles rounded to nearest, so a sequence a little longer than a multiple of
// chunk_tiles does not pay a partial for a sliver; seg < 1.5 chunk_tiles.  A launch of 257..447
// workgroups leaves the CUs that hold two of them behind: where even_units says so, a sequence whose
// segments would make it one gets as many as make one workgroup per CU.
__device__ __forceinline__ void split_tiles(int T, int chunk_tiles, int bias, int even_units, int even_n, int *n, int *seg)
{
    int nn = max(1, (T + bias) / chunk_tiles);
    if (even_units) {
        const int wgs = nn * even_units;
        if (wgs > 256 && wgs < 448) nn = even_n;
    }
    *n = nn;
    *seg = (T + nn - 1) / nn;
}

// anc[i] = {i} U anc[parent[i]]: one 128-bit mask per node, built by walking up.  Thread i asks for its own
// entry of the parent array ahead of the first K/V requests (memory answers in order: behind them it
// would come last, and the masks with it: attention of one head and 32 keys 4.94 -> 4.70 us, of 32 heads and
// 512 keys 12.1 -> 11.7, a step of 40 heads and 2048 keys 37.4 -> 36.4); the array goes through LDS, so that the walk (one dependent
// read per level) pays no global-memory latency per step.  With a root row the tree block has N rows of which row 0 is the root and row 1 + i
// candidate i: the root is every candidate's ancestor, and the caller's array (N - 1 entries, -1 = child
// of the root) is shifted by one.  (128 threads at least)
__device__ __forceinline__ int parent_of_thread(const AttnParams &p, int b)
{
    const int32_t *parent = p.parent + (p.parent_per_seq ? (size_t)b * (p.N - p.root_row) : 0);
    const int i = (int)threadIdx.x - p.root_row;
    int pa = -1;
    if (i >= 0 && (int)threadIdx.x < p.N) pa = parent[i];
    return pa;
}

// Contains a workgroup barrier; the caller adds the one that publishes the masks.
__device__ __forceinline__ void build_ancestor_masks(const AttnParams &p, int my_parent, uint32_t (*s_anc)[4], int *s_parent)
{
    const int i = threadIdx.x;
    static_assert(MCSD_MAX_NODES == 128, "four words per mask");
    if (i < MCSD_MAX_NODES) s_parent[i] = p.root_row && i > 0 && i < p.N ? max(my_parent, -1) + 1 : my_parent;
    __syncthreads();
    if (i < MCSD_MAX_NODES) {
        uint32_t m[4] = {0u, 0u, 0u, 0u};
        if (i < p.N) {
            int a = i;
            for (int step = 0; step < MCSD_MAX_NODES && a >= 0; ++step) {
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    if ((a >> 5) == w) m[w] |= 1u << (a & 31);
                const int pa = s_parent[a];
                a = (pa < a) ? pa : -1;      // a malformed array can not loop or index out of range
            }
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) s_anc[i][w] = m[w];
    }
}

// Workgroups start in the order z, y, x.  The (sequence, segment) pairs are handed out longest first (the
// short last segments of the sequences fill the end of the launch instead of a mostly idle last round
// of workgroups): pair number `slot` in dispatch order takes the pair of rank `slot` by length.  Done when
// the pairs fit one workgroup's threads and the launch does not fit the chip at once (two workgroups
// per CU start together anyway; the ranking is 1.4 us ahead of the first request).
template <int NT>
struct PairRanks { int len[NT], of_rank[NT], seq_L[NT]; };

template <int NT, typename LenOf>
__device__ __forceinline__ void longest_first(const AttnParams &p, PairRanks<NT> &s, int tid, int slot, int chunk_tiles, int split_bias,
                                              int even_units, LenOf len_of, int *b, int *chunk, int *L)
{
    const int n_pairs = p.B * p.n_chunks_max;
    const int seq = min(tid / p.n_chunks_max, p.B - 1), Lb = len_of(seq);      // (by all lanes: len_of may exchange between them)
    int my_len = 0;
    if (tid < n_pairs) {
        const int Tb = (Lb + KT - 1) / KT + p.tiles_tree;
        int nb, segb;
        split_tiles(Tb, chunk_tiles, split_bias, even_units, p.even_n, &nb, &segb);
        my_len = max(0, min(segb, Tb - (tid % p.n_chunks_max) * segb));
        s.len[tid] = my_len;
        if (tid % p.n_chunks_max == 0) s.seq_L[seq] = Lb;
    }
    __syncthreads();
    if (tid < n_pairs) {
        int rank = 0;
        for (int j = 0; j < n_pairs; ++j) {
            const int other = s.len[j];
            rank += (other > my_len || (other == my_len && j < tid)) ? 1 : 0;
        }
        s.of_rank[rank] = tid;
    }
    __syncthreads();
    const int pair = s.of_rank[slot];
    *b = __builtin_amdgcn_readfirstlane(pair / p.n_chunks_max);       // read from LDS: make it scalar again
    *chunk = __builtin_amdgcn_readfirstlane(pair % p.n_chunks_max);
    *L = __builtin_amdgcn_readfirstlane(s.seq_L[*b]);      // already loaded and clamped: no second trip to memory
}

// bf16, d = 128, more than 64 rows per KV head (tree_attn_shared.hip)
void launch_attn_shared(const AttnParams &p, dim3 grid, hipStream_t stream, const WalkParams &w);

// bf16, d = 128, all keys of a unit in one workgroup and `columns` (32, 64, 128) of the output (tree_attn_any.hip)
int32_t launch_attn_sliced(const AttnParams &p, int columns, hipStream_t stream, const WalkParams *tail_walk);

// fp32 storage and head dimensions other than 128 (tree_attn_any.hip): one launch, no workspace
int32_t launch_attn_any(const AttnParams &p, hipStream_t stream);

}  // namespace mcsd
