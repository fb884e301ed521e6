// Bookkeeping around the verification step, on the device: the candidate tree of a
// k-configuration (Sec. 3 / Sec. 4.3, generation order of Sec. 3.3) and the commit of the
// accepted path's keys and values to the prefix cache (Sec. 3.3).  Latency-sized kernels.
#include "mcsd_internal.h"

namespace mcsd {
namespace {

struct TreeParams {
    int k[MAX_GAMMA];
    int gamma, N, B, root_row;
    const int32_t *prefix_len;
    int32_t *parent, *depth, *q_row, *position_ids;
};

// One workgroup: thread i builds node i.  Level l (1-based) holds k_1 ... k_l nodes, its first
// node id is the sum of the earlier level sizes; node j of a level is child number j % k_l of
// node j / k_l of the level above.  Rows with children are exactly the rows above the last
// level, so their draft rows are numbered by the row index itself.
__global__ __launch_bounds__(256) void tree_build_kernel(TreeParams p)
{
    const int i = threadIdx.x;
    __shared__ int s_depth[MCSD_MAX_NODES];
    int internal_rows = 1;
    if (i < p.N) {
        int begin = 0, size = 1, prev_begin = -1, lvl = 0;
        for (int l = 1; l <= p.gamma; ++l) {
            const int sz = size * p.k[l - 1];
            if (i < begin + sz) {
                const int j = i - begin;
                p.parent[i] = (l == 1) ? -1 : prev_begin + j / p.k[l - 1];
                lvl = l;
                break;
            }
            prev_begin = begin;
            begin += sz;
            size = sz;
        }
        p.depth[i] = lvl;
        s_depth[i] = lvl;
    }
    {
        int size = 1;
        for (int l = 1; l < p.gamma; ++l) { size *= p.k[l - 1]; internal_rows += size; }
    }
    if (i <= p.N) p.q_row[i] = (i < internal_rows) ? i : -1;
    if (p.position_ids) {
        __syncthreads();
        // Without a root row the root is the last token of the prefix (position prefix_len - 1) and
        // a candidate of depth j sits at prefix_len + j - 1; with one, the root is the first new
        // token (entry 0, position prefix_len) and the candidates follow it.
        const int rows = p.N + p.root_row;
        for (int e = i; e < p.B * rows; e += blockDim.x) {
            const int b = e / rows, r = e % rows;
            p.position_ids[e] = p.root_row ? p.prefix_len[b] + (r == 0 ? 0 : s_depth[r - 1])
                                           : p.prefix_len[b] + s_depth[r] - 1;
        }
    }
}

struct CommitParams {
    int B, N, H_kv, L_stride, gamma_max, n_layers, root_row;
    int row_bytes;          // d * element size, multiple of 16
    char *k_prefix, *v_prefix;
    const char *k_tree, *v_tree;
    const int32_t *n_accepted, *accepted_path, *out_tokens;
    int32_t *prefix_len, *next_root;
    uint32_t *flags;
    // paged destination (block_table != nullptr): pools [n_layers][n_pages][H_kv][page_size][d]
    const int32_t *block_table;
    int page_size, n_pages, max_pages;
};

// What sequence b commits, found by one wavefront: every lane looks at one row, so that the path and
// the block table cost one trip to memory each instead of one per row.
struct CommitRows {
    int L;          // cache rows before the commit
    int wanted;     // rows this sequence would gain: the root (if it has a row), then the path
    int rows;       // the first of them that are good: path entries inside the tree, pages inside the pool
                    // (none with a count outside the path, not even the root)
    bool bad_count, full;
};

__device__ __forceinline__ CommitRows commit_rows(const CommitParams &p, int b, int lane)
{
    CommitRows c;
    int n = p.n_accepted[b];
    c.L = p.prefix_len[b];
    c.bad_count = n < 0 || n > p.gamma_max;
    if (c.bad_count) n = 0;
    c.wanted = n + p.root_row;
    c.full = c.L < 0 || (long)c.L + c.wanted > p.L_stride;
    c.rows = 0;
    if (c.full || c.bad_count) return c;
    for (int r0 = 0; r0 < c.wanted; r0 += 64) {
        const int r = r0 + lane;                            // row r holds path entry r - root_row
        bool good = r < c.wanted;
        if (good && r >= p.root_row) {
            const int nd = p.accepted_path[(size_t)b * p.gamma_max + (r - p.root_row)];
            good = nd >= 0 && nd < p.N;
        }
        if (p.block_table && r < c.wanted)
            good = good && (unsigned)p.block_table[(size_t)b * p.max_pages + (c.L + r) / p.page_size] < (unsigned)p.n_pages;
        const unsigned long long bad = ~__ballot(good);
        c.rows = r0 + (bad ? __ffsll((long long)bad) - 1 : 64);
        if (bad) break;
    }
    return c;
}

// grid (gamma_max + root_row, B, n_layers): block (j, b, layer) copies entry j of sequence b, all
// KV heads, K and V.  Without a root row, entry j is path entry j.  With one (the tree block has
// 1 + N rows, row 0 = the root, whose keys and values this forward pass produced as well), entry 0
// is the root and entry j >= 1 path entry j - 1: the root goes to cache row L, the candidate of
// depth j to row L + j.  prefix_len is only read here; kv_finish_kernel updates it afterwards.
__global__ __launch_bounds__(256) void kv_copy_kernel(CommitParams p)
{
    const int j = blockIdx.x, b = blockIdx.y, layer = blockIdx.z;
    const CommitRows c = commit_rows(p, b, threadIdx.x & 63);
    if (j >= c.rows) return;     // a bad entry anywhere up to j stops the copy there (the finish kernel reports it)
    const int L = c.L;
    const int tree_rows = p.N + p.root_row;
    const int src_row = (p.root_row && j == 0) ? 0 : p.root_row + p.accepted_path[(size_t)b * p.gamma_max + (j - p.root_row)];
    const int vec_per_row = p.row_bytes / 16;
    const size_t lb = (size_t)layer * p.B + b;
    size_t page_base = 0;       // paged: first row of the destination page slice of KV head 0
    if (p.block_table) {
        const int blk = p.block_table[(size_t)b * p.max_pages + (L + j) / p.page_size];
        page_base = ((size_t)layer * p.n_pages + blk) * (size_t)p.H_kv * p.page_size + (size_t)((L + j) % p.page_size);
    }
    for (int e = threadIdx.x; e < p.H_kv * vec_per_row; e += blockDim.x) {
        const int g = e / vec_per_row, c4 = e % vec_per_row;
        const size_t src = ((lb * p.H_kv + g) * (size_t)tree_rows + src_row) * p.row_bytes + (size_t)c4 * 16;
        const size_t dst = (p.block_table ? page_base + (size_t)g * p.page_size
                                          : (lb * p.H_kv + g) * (size_t)p.L_stride + (size_t)(L + j)) * p.row_bytes + (size_t)c4 * 16;
        *reinterpret_cast<uint4 *>(p.k_prefix + dst) = *reinterpret_cast<const uint4 *>(p.k_tree + src);
        *reinterpret_cast<uint4 *>(p.v_prefix + dst) = *reinterpret_cast<const uint4 *>(p.v_tree + src);
    }
}

// What a commit leaves for the next step, by one lane.
__device__ __forceinline__ void finish_sequence(const CommitParams &p, int b, const CommitRows &c, int next_root)
{
    p.next_root[b] = next_root;
    uint32_t fl = c.bad_count ? (uint32_t)MCSD_FLAG_BAD_TREE : 0u;
    if (c.full) {
        fl |= (uint32_t)MCSD_FLAG_CACHE_FULL;
    } else {
        if (c.rows < c.wanted) fl |= (uint32_t)MCSD_FLAG_BAD_TREE;
        p.prefix_len[b] = c.L + c.rows;
    }
    p.flags[b] = fl;
}

__device__ __forceinline__ int next_root_of(const CommitParams &p, int b, const CommitRows &c)
{
    const int n = c.bad_count ? 0 : c.wanted - p.root_row;
    return p.out_tokens[(size_t)b * (p.gamma_max + 1) + n];
}

// One wavefront per sequence.
__global__ __launch_bounds__(64) void kv_finish_kernel(CommitParams p)
{
    const int b = blockIdx.x, lane = threadIdx.x;
    const CommitRows c = commit_rows(p, b, lane);
    if (lane == 0) finish_sequence(p, b, c, next_root_of(p, b, c));
}

// A small commit in one launch: one workgroup per sequence copies all layers, so that nothing but
// its own first wavefront reads prefix_len[b], which may then move on at once.  A wavefront takes one
// (row, layer) pair at a time: all its KV heads, K and V.
constexpr int COMMIT_ROWS = 64, COMMIT_WAVES = 16;
constexpr size_t COMMIT_BYTES = 128 << 10;      // per sequence

__global__ __launch_bounds__(64 * COMMIT_WAVES) void kv_commit_kernel(CommitParams p)
{
    __shared__ int s_src[COMMIT_ROWS], s_page[COMMIT_ROWS];
    __shared__ int s_rows, s_L;
    const int b = blockIdx.x, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave == 0) {
        const CommitRows c = commit_rows(p, b, lane);
        if (lane < c.rows) {
            s_src[lane] = lane < p.root_row ? 0 : p.root_row + p.accepted_path[(size_t)b * p.gamma_max + (lane - p.root_row)];
            s_page[lane] = p.block_table ? p.block_table[(size_t)b * p.max_pages + (c.L + lane) / p.page_size] : 0;
        }
        if (lane == 0) {
            s_rows = c.rows;
            s_L = c.L;
            finish_sequence(p, b, c, next_root_of(p, b, c));
        }
    }
    __syncthreads();
    const int rows = __builtin_amdgcn_readfirstlane(s_rows), L = __builtin_amdgcn_readfirstlane(s_L);
    const int vec_per_row = p.row_bytes / 16, n_vec = p.H_kv * vec_per_row, tree_rows = p.N + p.root_row;
    const int g_step = 64 / vec_per_row, c_step = 64 % vec_per_row;
    for (int q = wave; q < rows * p.n_layers; q += COMMIT_WAVES) {
        const int j = q / p.n_layers, layer = q % p.n_layers;
        const size_t lb = (size_t)layer * p.B + b;
        const int src_row = __builtin_amdgcn_readfirstlane(s_src[j]);
        const size_t src0 = lb * p.H_kv * (size_t)tree_rows + src_row;
        size_t dst0, dst_pitch;
        if (p.block_table) {
            const int blk = __builtin_amdgcn_readfirstlane(s_page[j]);
            dst0 = ((size_t)layer * p.n_pages + blk) * (size_t)p.H_kv * p.page_size + (size_t)((L + j) % p.page_size);
            dst_pitch = p.page_size;
        } else {
            dst0 = lb * p.H_kv * (size_t)p.L_stride + (size_t)(L + j);
            dst_pitch = p.L_stride;
        }
        int g = lane / vec_per_row, c4 = lane % vec_per_row;
        for (int e0 = 0; e0 < n_vec; e0 += 128) {
            // Two pieces of K and of V per pass.  (The compiler keeps them in LDS, 64 KB of it, and waits for
            // the first pair before it requests the second; the figures at the launch are those of this form.)
            uint4 k[2], v[2];
            size_t dst[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                dst[i] = (dst0 + (size_t)g * dst_pitch) * p.row_bytes + (size_t)c4 * 16;
                const size_t src = (src0 + (size_t)g * tree_rows) * p.row_bytes + (size_t)c4 * 16;
                if (e0 + 64 * i + lane < n_vec) {
                    k[i] = *reinterpret_cast<const uint4 *>(p.k_tree + src);
                    v[i] = *reinterpret_cast<const uint4 *>(p.v_tree + src);
                }
                g += g_step;
                c4 += c_step;
                if (c4 >= vec_per_row) { c4 -= vec_per_row; ++g; }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (e0 + 64 * i + lane < n_vec) {
                    *reinterpret_cast<uint4 *>(p.k_prefix + dst[i]) = k[i];
                    *reinterpret_cast<uint4 *>(p.v_prefix + dst[i]) = v[i];
                }
        }
    }
}

}  // namespace

int32_t launch_tree_build(const int32_t *kconfig, int gamma, int n_nodes, int B, const int32_t *prefix_len,
                          int32_t *parent, int32_t *depth, int32_t *q_row, int32_t *position_ids, int root_row, hipStream_t stream)
{
    TreeParams p = {};
    for (int i = 0; i < gamma; ++i) p.k[i] = kconfig[i];
    p.gamma = gamma; p.N = n_nodes; p.B = B; p.root_row = root_row; p.prefix_len = prefix_len;
    p.parent = parent; p.depth = depth; p.q_row = q_row; p.position_ids = position_ids;
    launch_kernel(K_TREE_BUILD, tree_build_kernel, dim3(1), dim3(256), stream, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("tree_build launch failed: %s", hipGetErrorString(e)); return MCSD_E_HIP; }
    return MCSD_OK;
}

int32_t launch_kv_commit(const mcsd_commit_desc &d, const mcsd_commit_bufs &b, hipStream_t stream,
                         const mcsd_paged_kv *paged)
{
    CommitParams p;
    p.block_table = nullptr; p.page_size = p.n_pages = p.max_pages = 0;
    if (paged) {
        p.block_table = paged->block_table; p.page_size = paged->page_size;
        p.n_pages = paged->n_pages; p.max_pages = paged->max_pages_per_seq;
    }
    p.B = d.B; p.N = d.N; p.H_kv = d.H_kv; p.L_stride = d.L_stride; p.gamma_max = d.gamma_max; p.n_layers = d.n_layers;
    p.root_row = d.root_row ? 1 : 0;
    p.row_bytes = d.d * (d.dtype == MCSD_DTYPE_FP32 ? 4 : 2);
    p.k_prefix = static_cast<char *>(b.k_prefix); p.v_prefix = static_cast<char *>(b.v_prefix);
    p.k_tree = static_cast<const char *>(b.k_tree); p.v_tree = static_cast<const char *>(b.v_tree);
    p.n_accepted = b.n_accepted; p.accepted_path = b.accepted_path; p.out_tokens = b.out_tokens;
    p.prefix_len = b.prefix_len; p.next_root = b.next_root; p.flags = b.flags;
    // One launch where a sequence can bring at most 128 KB (all layers, K and V): a launch less is 3 us,
    // and one compute unit copies about 50 GB/s.  Reset of prefix_len and commit, 4 sequences, 4 layers,
    // 8 KV heads of 128, 4 rows each (64 KB): 9.8 us with the two launches below, 7.0 us; 8 layers (128 KB)
    // 10.2 and 7.8; 32 KV heads (256 KB) 10.2 and 10.0; 768 KB 10.1 and 21.5.
    const size_t most = (size_t)(d.gamma_max + p.root_row) * d.n_layers * d.H_kv * p.row_bytes * 2;
    if (d.gamma_max + p.root_row <= COMMIT_ROWS && most <= COMMIT_BYTES) {
        launch_kernel(K_KV_COPY, kv_commit_kernel, dim3(d.B), dim3(64 * COMMIT_WAVES), stream, p);
        const hipError_t e1 = hipGetLastError();
        if (e1 != hipSuccess) { set_error("kv_commit launch failed: %s", hipGetErrorString(e1)); return MCSD_E_HIP; }
        return MCSD_OK;
    }
    launch_kernel(K_KV_COPY, kv_copy_kernel, dim3(d.gamma_max + p.root_row, d.B, d.n_layers), dim3(256), stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_error("kv_copy launch failed: %s", hipGetErrorString(e)); return MCSD_E_HIP; }
    launch_kernel(K_KV_FINISH, kv_finish_kernel, dim3(d.B), dim3(64), stream, p);
    e = hipGetLastError();
    if (e != hipSuccess) { set_error("kv_finish launch failed: %s", hipGetErrorString(e)); return MCSD_E_HIP; }
    return MCSD_OK;
}

}  // namespace mcsd
