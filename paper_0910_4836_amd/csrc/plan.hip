// CRS row-block plans built on the GPU (spmv_crs_plan_ws): the same greedy
// blocks as the host planner of spmv_crs_plan, without the row pointer's way
// to the host and back.
//
// Greedy blocks look serial (a block starts where the one before it ended),
// but where a block ends depends on its first row alone, and no block holds
// more than 2048 rows.  So the rows are cut into tiles of 4096 and
//   1. plan_tiles_kernel finds, for every row of a tile, the end of the block
//      that would start there, and by pointer jumping in LDS where a chain
//      starting at one of the tile's first 2048 rows leaves the tile and how
//      many blocks it takes (a chain enters a tile only at those rows);
//   2. plan_groups_kernel composes the tables of 32 tiles;
//   3. plan_write_kernel follows the chain from row 0 over the groups, then
//      over the tiles of its own group, to its tile, and writes that tile's
//      blocks.
// Bound by latency (a few dependent loads per step); the row pointer is read
// once.  At 2 M rows and 31,000 blocks the plan takes 0.07 ms of kernels
// where the host planner, with its copies, took 6.5 ms.
#include "common.hpp"

namespace spmv {

constexpr int PT_THREADS = 1024;
constexpr int PT_ROWS = 4096;                              // rows per tile
constexpr int PT_SPAN = CRS_MAX_SHORT_BLOCK_ROWS;          // a block's most rows: how far a chain enters a tile
constexpr int PT_GROUP = 32;                               // tiles per group
constexpr int PT_WORDS = (PT_ROWS + PT_SPAN) / 64;

struct PlanEntry {
    int32_t at;        // rows past the start of the next tile (or group) where the chain goes on
    int32_t count;     // blocks taken
};

// step[r] = rows of the block that starts at row r; table[tile][e] as above;
// result[1] = 1 if row_ptr decreases, result[2]: longest row.
__global__ __launch_bounds__(PT_THREADS) void plan_tiles_kernel(const int32_t *__restrict__ rp, int32_t n, int32_t T,
                                                                uint16_t *__restrict__ step,
                                                                PlanEntry *__restrict__ table,
                                                                int32_t *__restrict__ result)
{
    __shared__ int32_t p[PT_ROWS + PT_SPAN + 1];
    __shared__ uint32_t jump[PT_ROWS];                     // rows past the tile's start | blocks << 16
    __shared__ int32_t wmax[PT_THREADS / WAVE];
    __shared__ uint64_t longer[PT_WORDS];                  // bit r: row r has more than CRS_SHORT_ROW entries
    const int t = (int)threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * PT_ROWS;
    const int32_t left = n - base < PT_ROWS + PT_SPAN ? (int32_t)(n - base) : PT_ROWS + PT_SPAN;   // rows in view
    const int32_t rows = left < PT_ROWS ? left : PT_ROWS;                                           // the tile's own
    for (int32_t i = t; i <= left; i += PT_THREADS) p[i] = rp[base + i];
    __syncthreads();
    bool dec = false;
    int32_t longest = 0;
    for (int32_t i = t; i < PT_ROWS + PT_SPAN; i += PT_THREADS) {          // whole wavefronts
        const int32_t len = i < left ? p[i + 1] - p[i] : 0;
        dec |= len < 0;
        longest = i < rows && len > longest ? len : longest;
        const uint64_t m = __ballot(len > CRS_SHORT_ROW);
        if (lane_id() == 0) longer[i / WAVE] = m;
    }
    if (__ballot(dec) && lane_id() == 0) atomicOr(result + 1, 1);
    for (int off = WAVE / 2; off > 0; off >>= 1) longest = max(longest, __shfl_xor(longest, off, WAVE));
    if (lane_id() == 0) wmax[t / WAVE] = longest;
    __syncthreads();
    if (t == 0) {
        for (int q = 1; q < PT_THREADS / WAVE; ++q) longest = max(longest, wmax[q]);
        atomicMax(result + 2, longest);
    }
    for (int32_t r = t; r < rows; r += PT_THREADS) {
        // most rows: 256, or up to the first longer row, at most 2048
        const int32_t most = left < r + PT_SPAN ? left : r + PT_SPAN;
        int32_t cap = r + CRS_MAX_BLOCK_ROWS < most ? r + CRS_MAX_BLOCK_ROWS : most;
        if (cap < most) {
            int32_t w = r >> 6;
            const int32_t last = (most - 1) >> 6;
            uint64_t m = longer[w] & (~0ull << (r & 63));
            while (m == 0 && w < last) m = longer[++w];
            const int32_t q = m ? (w << 6) + (int32_t)__ffsll((unsigned long long)m) - 1 : most;
            cap = q > cap ? (q < most ? q : most) : cap;
        }
        // largest end with at most T entries, at least one row
        int32_t lo = r + 1, hi = cap;
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) >> 1;
            if (p[mid] - p[r] <= T) lo = mid;
            else hi = mid - 1;
        }
        jump[r] = (uint32_t)lo | 1u << 16;
        step[base + r] = (uint16_t)(lo - r);
    }
    __syncthreads();
    // pointer jumping; an entry is one word, so a neighbour's newer value is
    // as good as its older one
    for (int hop = 1; hop < PT_ROWS; hop <<= 1) {
        for (int32_t r = t; r < rows; r += PT_THREADS) {
            const uint32_t a = jump[r];
            const int32_t to = (int32_t)(a & 0xffffu);
            if (to < rows) {
                const uint32_t b = jump[to];
                jump[r] = (b & 0xffffu) | ((a >> 16) + (b >> 16)) << 16;
            }
        }
        __syncthreads();
    }
    for (int32_t e = t; e < PT_SPAN; e += PT_THREADS) {
        PlanEntry x{0, 0};
        if (e < rows) {
            const uint32_t a = jump[e];
            x.at = (int32_t)(a & 0xffffu) - PT_ROWS;
            if (x.at < 0) x.at = 0;                         // the last tile: the chain ends at row n
            x.count = (int32_t)(a >> 16);
        }
        table[(int64_t)blockIdx.x * PT_SPAN + e] = x;
    }
}

__device__ __forceinline__ void plan_follow(const PlanEntry *__restrict__ table, int64_t first, int64_t last,
                                            int32_t &at, int64_t &count)
{
    for (int64_t i = first; i < last; ++i) {
        const PlanEntry x = table[i * PT_SPAN + at];
        at = x.at;
        count += x.count;
    }
}

__global__ __launch_bounds__(256) void plan_groups_kernel(const PlanEntry *__restrict__ table, int64_t tiles,
                                                          PlanEntry *__restrict__ group_table)
{
    const int64_t g = blockIdx.y;
    const int32_t e = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    const int64_t last = (g + 1) * PT_GROUP < tiles ? (g + 1) * PT_GROUP : tiles;
    int32_t at = e;
    int64_t count = 0;
    plan_follow(table, g * PT_GROUP, last, at, count);
    group_table[g * PT_SPAN + e] = PlanEntry{at, (int32_t)count};
}

// result[0] = number of blocks; the plan is written as far as cap reaches
__global__ __launch_bounds__(256) void plan_write_kernel(const uint16_t *__restrict__ step, int32_t n,
                                                         const PlanEntry *__restrict__ table,
                                                         const PlanEntry *__restrict__ group_table, int64_t tiles,
                                                         int32_t *__restrict__ plan, int32_t cap,
                                                         int32_t *__restrict__ result)
{
    __shared__ uint16_t st[PT_ROWS];
    const int t = (int)threadIdx.x;
    const int64_t tile = blockIdx.x, base = tile * PT_ROWS;
    const int32_t rows = n - base < PT_ROWS ? (int32_t)(n - base) : PT_ROWS;
    for (int32_t i = t; i < rows; i += 256) st[i] = step[base + i];
    int32_t at = 0;
    int64_t count = 0;
    if (t == 0) {
        const int64_t g = tile / PT_GROUP;
        plan_follow(group_table, 0, g, at, count);
        plan_follow(table, g * PT_GROUP, tile, at, count);
    }
    __syncthreads();
    if (t != 0) return;
    while (at < rows) {
        if (count < cap) plan[count] = (int32_t)(base + at);
        ++count;
        at += st[at];
    }
    if (tile == tiles - 1) {
        if (count < cap) plan[count] = n;
        result[0] = (int32_t)count;
    }
}

static int64_t plan_tile_count(int32_t n) { return ceil_div(n > 0 ? n : 1, PT_ROWS); }

}  // namespace spmv

using namespace spmv;

extern "C" {

size_t spmv_crs_plan_workspace_size(int32_t n_rows)
{
    const size_t n = (size_t)(n_rows > 0 ? n_rows : 1);
    const size_t tiles = (size_t)plan_tile_count(n_rows), groups = (size_t)ceil_div((int64_t)tiles, PT_GROUP);
    return align_up(3 * sizeof(int32_t), 256) + align_up(sizeof(uint16_t) * n, 256) +
           align_up(sizeof(PlanEntry) * PT_SPAN * tiles, 256) + align_up(sizeof(PlanEntry) * PT_SPAN * groups, 256) + 256;
}

spmv_status spmv_crs_plan_ws(int32_t n_rows, const int32_t *row_ptr, int32_t block_nnz, int32_t *plan,
                             int32_t plan_cap, int32_t *h_n_blocks, int32_t *h_longest, void *ws, size_t ws_bytes,
                             void *stream)
{
    SPMV_REQUIRE(n_rows >= 0, "spmv_crs_plan_ws: n_rows < 0");
    SPMV_REQUIRE(h_n_blocks, "spmv_crs_plan_ws: null h_n_blocks");
    SPMV_REQUIRE(row_ptr, "spmv_crs_plan_ws: null row_ptr");
    if (block_nnz == 0) block_nnz = crs_default_block_nnz();
    SPMV_REQUIRE(block_nnz >= CRS_THREADS && block_nnz <= CRS_MAX_BLOCK_NNZ,
                 "spmv_crs_plan_ws: block_nnz must be in [256, 4096]");
    SPMV_REQUIRE(plan || plan_cap == 0, "spmv_crs_plan_ws: null plan");
    SPMV_REQUIRE(ws && ws_bytes >= spmv_crs_plan_workspace_size(n_rows), "spmv_crs_plan_ws: workspace too small");
    hipStream_t s = as_stream(stream);
    if (n_rows == 0) {
        *h_n_blocks = 0;
        if (h_longest) *h_longest = 0;
        if (plan_cap < 1) return fail(SPMV_ERR_CAPACITY, "spmv_crs_plan_ws: plan capacity < n_blocks+1");
        SPMV_HIP(hipMemsetAsync(plan, 0, sizeof(int32_t), s));
        SPMV_HIP(hipStreamSynchronize(s));
        return SPMV_OK;
    }
    const int64_t tiles = plan_tile_count(n_rows), groups = ceil_div(tiles, PT_GROUP);
    WsCarver wc(ws, ws_bytes);
    int32_t *result = wc.take<int32_t>(3);                   // number of blocks, row_ptr decreases, longest row
    uint16_t *step = wc.take<uint16_t>((size_t)n_rows);
    PlanEntry *table = wc.take<PlanEntry>((size_t)tiles * PT_SPAN);
    PlanEntry *group_table = wc.take<PlanEntry>((size_t)groups * PT_SPAN);
    if (!wc.ok()) return fail(SPMV_ERR_INVALID_ARG, "spmv_crs_plan_ws: workspace too small");
    SPMV_HIP(hipMemsetAsync(result, 0, 3 * sizeof(int32_t), s));
    plan_tiles_kernel<<<(unsigned)tiles, PT_THREADS, 0, s>>>(row_ptr, n_rows, block_nnz, step, table, result);
    SPMV_CHECK_LAUNCH("crs plan tiles");
    if (groups > 1) {
        plan_groups_kernel<<<dim3(PT_SPAN / 256, (unsigned)groups), 256, 0, s>>>(table, tiles, group_table);
        SPMV_CHECK_LAUNCH("crs plan groups");
    }
    plan_write_kernel<<<(unsigned)tiles, 256, 0, s>>>(step, n_rows, table, group_table, tiles, plan, plan_cap, result);
    SPMV_CHECK_LAUNCH("crs plan");
    int32_t h[3] = {0, 0, 0};
    SPMV_HIP(hipMemcpyAsync(h, result, sizeof(h), hipMemcpyDeviceToHost, s));
    SPMV_HIP(hipStreamSynchronize(s));
    if (h[1]) return fail(SPMV_ERR_BAD_FORMAT, "spmv_crs_plan_ws: row_ptr decreases");
    *h_n_blocks = h[0];
    if (h_longest) *h_longest = h[2];
    if (plan_cap < h[0] + 1) return fail(SPMV_ERR_CAPACITY, "spmv_crs_plan_ws: plan capacity < n_blocks+1");
    return SPMV_OK;
}

}  // extern "C"
