// Format construction on the GPU (paper Section 2): COO -> CRS, CRS checks,
// CRS -> JDS (row permutation by decreasing length, jagged diagonals), JDS ->
// CRS, JDS -> blocked JDS (RBJDS, optionally SOJDS), CRS transpose, value
// rounding, vector permutation and gathers.
//
// All orderings are produced by a stable least-significant-digit radix sort
// written here (8-bit digits, wave ballots for the in-tile ranks), so every
// permutation is unique and reproducible; counts use integer atomics only.
#include <algorithm>
#include <vector>

#include "common.hpp"
#include "sort.hpp"

namespace spmv {

__global__ void validate_rows_kernel(const int32_t *__restrict__ rp, int32_t n_rows, int64_t nnz,
                                     int32_t *__restrict__ bad)
{
    GRID_LOOP(r, (int64_t)n_rows)
    {
        if (rp[r + 1] < rp[r]) atomicOr(bad, 1);
        if (r == 0 && rp[0] != 0) atomicOr(bad, 2);
        if (r == n_rows - 1 && (int64_t)rp[n_rows] != nnz) atomicOr(bad, 4);
    }
}

__global__ void validate_cols_kernel(const int32_t *__restrict__ col, int64_t nnz, int32_t n_cols,
                                     int32_t *__restrict__ bad)
{
    GRID_LOOP(k, nnz)
    {
        if (col[k] < 0 || col[k] >= n_cols) atomicOr(bad, 8);
    }
}

__global__ void row_len_kernel(const int32_t *__restrict__ rp, int32_t n, int32_t *__restrict__ len,
                               int32_t *__restrict__ maxlen)
{
    __shared__ int32_t wmax[4];                  // blocks of 256
    int32_t m = 0;
    GRID_LOOP(r, (int64_t)n)
    {
        int32_t l = rp[r + 1] - rp[r];
        len[r] = l;
        m = max(m, l);
    }
    // one atomic per workgroup, of at most 1024: one per row queued at the single
    // counter (360 us at 2 M rows)
    for (int off = WAVE / 2; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off, WAVE));
    if (lane_id() == 0) wmax[threadIdx.x / WAVE] = m;
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(maxlen, max(max(wmax[0], wmax[1]), max(wmax[2], wmax[3])));
}

// key may be len itself
__global__ void desc_key_kernel(const int32_t *len, int32_t n, int32_t ndiag, uint32_t *key)
{
    GRID_LOOP(r, (int64_t)n) key[r] = (uint32_t)(ndiag - len[r]);
}

__global__ void inverse_perm_kernel(const int32_t *__restrict__ perm, int32_t n, int32_t *__restrict__ iperm)
{
    GRID_LOOP(r, (int64_t)n) iperm[perm[r]] = (int32_t)r;
}

// count[d] = rows longer than d = first permuted row whose length is <= d
__global__ void diag_count_kernel(const uint32_t *__restrict__ skey, int32_t n, int32_t ndiag,
                                  int32_t *__restrict__ count)
{
    GRID_LOOP(d, (int64_t)ndiag)
    {
        // lengths ndiag - skey[r] never increase; find first r with length <= d
        int64_t lo = 0, hi = n;
        while (lo < hi) {
            int64_t mid = (lo + hi) >> 1;
            if ((int64_t)ndiag - (int64_t)skey[mid] > d) lo = mid + 1;
            else hi = mid;
        }
        count[d] = (int32_t)lo;
    }
}

// row containing CRS entry j: last r with rp[r] <= j
__device__ __forceinline__ int32_t row_of(const int32_t *__restrict__ rp, int32_t n, int64_t j)
{
    int32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        int32_t mid = (lo + hi + 1) >> 1;
        if ((int64_t)rp[mid] <= j) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// ---- CRS <-> JDS
// Both directions transpose: a row's entries lie together in CRS, a
// diagonal's in JDS.  Copied entry by entry one side of the copy is a 4- or
// 8-byte access per 128-byte line.
//   * Rows of more than 8 entries go through LDS in tiles of 64 permuted rows
//     x 32 diagonals, both sides runs of consecutive addresses; a grid of
//     fixed size walks the tiles.
//   * Shorter rows are too small for runs on the CRS side, and in permuted
//     order each of their lines would be fetched once per length that occurs
//     in it.  They go one lane per row in the original order: the CRS side
//     walks the arrays once, and as the sort is stable, rows of one length
//     in a stretch of rows are neighbours on every diagonal.
// Bound: the copy rate, and the partial lines at the ends of the runs.  30 M
// entries, FP64 values, 2 M power-law rows (0.72 GB): CRS -> JDS 1375 -> 284
// us, JDS -> CRS 1452 -> 312 us, of which the short rows take 66 (as tiles of
// 256 rows x 8: 85-95).  Tiles of 128 or 256 rows, one range of tiles per XCD
// and more workgroups all measure the same within 3%.
constexpr int JT_THREADS = 256;
constexpr int JT_ROWS = 64, JT_DIAGS = 32;          // a tile
constexpr int JT_SHORT = 8;                         // rows of at most this many entries go by lanes
constexpr int JT_STEPS = JT_ROWS * JT_DIAGS / JT_THREADS;
constexpr int JT_PITCH = JT_DIAGS + 1;

__device__ __forceinline__ int32_t diag_len(const int32_t *__restrict__ jp, int32_t d) { return jp[d + 1] - jp[d]; }

// rows of more than JT_SHORT entries
__device__ __forceinline__ int32_t jt_long_rows(const int32_t *__restrict__ jp, int32_t ndiag)
{
    return ndiag > JT_SHORT ? diag_len(jp, JT_SHORT) : 0;
}

// Tiles of 32 diagonals in groups: group k covers 2^q tiles of each of the
// row sets that reach its first diagonal, q as small as keeps the table of
// group sizes in one workgroup (q = 0 up to 65,504 diagonals; a workgroup
// that walks 4 to 16 tiles of one row set is 1-4% slower).
constexpr int JT_GROUPS = SCAN_TILE;
struct JtGroups {
    int32_t K;                  // groups over the diagonals
    int q;
};

static JtGroups jt_groups(int32_t ndiag)
{
    JtGroups g{1, 0};
    while ((g.K = (int32_t)ceil_div(ndiag > 0 ? ndiag : 1, (int64_t)JT_DIAGS << g.q)) > JT_GROUPS - 1) ++g.q;
    return g;
}

// prefix[k], k <= K: before group k.  C == 0: sets of JT_ROWS rows of more
// than JT_SHORT entries; C > 0: tiles of BT_ROWS rows, whole slices of C rows.
constexpr int BT_ROWS = 256;
__global__ __launch_bounds__(SCAN_THREADS) void jt_table_kernel(const int32_t *__restrict__ jp, int32_t ndiag,
                                                                int32_t C, JtGroups g,
                                                                int32_t *__restrict__ prefix)
{
    __shared__ int32_t wt[SCAN_THREADS / WAVE];
    const int32_t cut = jt_long_rows(jp, ndiag);
    int32_t v[SCAN_ITEMS], sum = 0;
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) {
        const int32_t k = (int32_t)threadIdx.x * SCAN_ITEMS + j;
        v[j] = 0;
        if (k < g.K && (int64_t)(k << g.q) * JT_DIAGS < ndiag) {       // jp ends with entry ndiag
            const int64_t reach = diag_len(jp, (k << g.q) * JT_DIAGS);
            const int64_t sets = C == 0 ? (min((int64_t)cut, reach) + JT_ROWS - 1) / JT_ROWS
                                        : ((reach + C - 1) / C * C + BT_ROWS - 1) / BT_ROWS;
            v[j] = (int32_t)sets << (C == 0 ? 0 : g.q);
        }
        sum += v[j];
    }
    int32_t total;
    int32_t run = block_exclusive_scan<int32_t>(sum, wt, &total);
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) {
        const int32_t k = (int32_t)threadIdx.x * SCAN_ITEMS + j;
        if (k < g.K) prefix[k] = run;
        run += v[j];
    }
    if (threadIdx.x == 0) prefix[g.K] = total;
}

// last k with prefix[k] <= b
__device__ __forceinline__ int32_t jt_group(const int32_t *__restrict__ prefix, int32_t groups, int32_t b)
{
    int32_t lo = 0, hi = groups - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (prefix[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

struct JtArgs {
    const int32_t *rp;          // CRS row pointer
    const int32_t *perm, *iperm;
    const int32_t *jp;
    int32_t n, ndiag;
    JtGroups g;
    const int32_t *prefix;      // K + 1 entries
    int symperm;
};

template <bool TO_JDS, typename T>
__global__ __launch_bounds__(JT_THREADS) void jds_transpose_kernel(JtArgs a, const int32_t *__restrict__ col_in,
                                                                   const T *__restrict__ val_in,
                                                                   int32_t *__restrict__ col_out,
                                                                   T *__restrict__ val_out)
{
    __shared__ int32_t cs[JT_ROWS * JT_PITCH];
    __shared__ T vs[JT_ROWS * JT_PITCH];
    __shared__ int32_t at[JT_ROWS], len[JT_ROWS], jd[JT_DIAGS];
    const int t = (int)threadIdx.x, lane = lane_id(), w = t / WAVE;
    const int32_t sets = a.prefix[a.g.K], cut = jt_long_rows(a.jp, a.ndiag);
    for (int32_t b = (int32_t)blockIdx.x; b < sets; b += (int32_t)gridDim.x) {
        const int32_t k = jt_group(a.prefix, a.g.K, b);
        const int32_t r0 = (b - a.prefix[k]) * JT_ROWS, nr = min(JT_ROWS, cut - r0);
        const int64_t d_first = (int64_t)k * JT_DIAGS << a.g.q;
        const int64_t d_end = min((int64_t)a.ndiag, d_first + (JT_DIAGS << a.g.q));
        for (int64_t d0 = d_first; d0 < d_end; d0 += JT_DIAGS) {
            __syncthreads();                                 // the tile before has been written
            if (t < nr) {
                const int32_t row = a.perm[r0 + t], s = a.rp[row];
                at[t] = s + (int32_t)d0;
                len[t] = min(a.rp[row + 1] - s - (int32_t)d0, JT_DIAGS);
            }
            if (t < JT_DIAGS) jd[t] = d0 + t < a.ndiag ? a.jp[d0 + t] + r0 : 0;
            __syncthreads();
            const int32_t depth = len[0];                    // rows by decreasing length
            if (depth <= 0) break;
            // side of the rows: 2^wlog lanes per row; side of the diagonals: a
            // lane per row, a diagonal per wavefront
            int wlog = 0;
            while (1 << wlog < depth) ++wlog;
            const int32_t step = JT_THREADS >> wlog, e = t & ((1 << wlog) - 1);
            int32_t c[JT_STEPS];
            T v[JT_STEPS];
#pragma unroll
            for (int j = 0; j < JT_STEPS; ++j) {
                const int32_t i = TO_JDS ? (t >> wlog) + j * step : lane, d = TO_JDS ? e : w + j * (JT_THREADS / WAVE);
                if (i < nr && d < len[i]) {
                    const int64_t from = TO_JDS ? at[i] + d : jd[d] + i;
                    c[j] = col_in[from];
                    v[j] = val_in[from];
                }
            }
#pragma unroll
            for (int j = 0; j < JT_STEPS; ++j) {
                const int32_t i = TO_JDS ? (t >> wlog) + j * step : lane, d = TO_JDS ? e : w + j * (JT_THREADS / WAVE);
                if (i < nr && d < len[i]) {
                    cs[i * JT_PITCH + d] = c[j];
                    vs[i * JT_PITCH + d] = v[j];
                }
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < JT_STEPS; ++j) {
                const int32_t i = TO_JDS ? lane : (t >> wlog) + j * step, d = TO_JDS ? w + j * (JT_THREADS / WAVE) : e;
                if (i < nr && d < len[i]) {
                    const int64_t to = TO_JDS ? jd[d] + i : at[i] + d;
                    const int32_t cc = cs[i * JT_PITCH + d];
                    col_out[to] = !a.symperm ? cc : TO_JDS ? a.iperm[cc] : a.perm[cc];
                    val_out[to] = vs[i * JT_PITCH + d];
                }
            }
        }
    }
}

template <bool TO_JDS, typename T>
__global__ __launch_bounds__(JT_THREADS) void jds_short_rows_kernel(JtArgs a, const int32_t *__restrict__ col_in,
                                                                    const T *__restrict__ val_in,
                                                                    int32_t *__restrict__ col_out,
                                                                    T *__restrict__ val_out)
{
    const int64_t row = xcd_remap(blockIdx.x, gridDim.x) * JT_THREADS + threadIdx.x;
    if (row >= a.n) return;
    const int32_t s = a.rp[row], len = a.rp[row + 1] - s, r = a.iperm[row];
    if (len > JT_SHORT) return;
    int32_t c[JT_SHORT];
    T v[JT_SHORT];
#pragma unroll
    for (int d = 0; d < JT_SHORT; ++d)
        if (d < len) {
            const int64_t from = TO_JDS ? s + d : a.jp[d] + r;
            c[d] = col_in[from];
            v[d] = val_in[from];
        }
#pragma unroll
    for (int d = 0; d < JT_SHORT; ++d)
        if (d < len) {
            const int64_t to = TO_JDS ? a.jp[d] + r : s + d;
            col_out[to] = !a.symperm ? c[d] : TO_JDS ? a.iperm[c[d]] : a.perm[c[d]];
            val_out[to] = v[d];
        }
}

static size_t jt_ws_bytes() { return align_up(sizeof(int32_t) * (JT_GROUPS + 1), 256) + 256; }

template <bool TO_JDS, typename T>
static spmv_status jds_transpose(JtArgs a, const int32_t *col_in, const void *val_in, int32_t *col_out, void *val_out,
                                 WsCarver &wc, hipStream_t s)
{
    a.g = jt_groups(a.ndiag);
    int32_t *prefix = wc.take<int32_t>(JT_GROUPS + 1);
    if (!wc.ok()) return fail(SPMV_ERR_INVALID_ARG, "CRS <-> JDS: workspace too small");
    jt_table_kernel<<<1, SCAN_THREADS, 0, s>>>(a.jp, a.ndiag, 0, a.g, prefix);
    SPMV_CHECK_LAUNCH("jds tiles");
    a.prefix = prefix;
    if (a.ndiag > JT_SHORT) {
        jds_transpose_kernel<TO_JDS, T><<<(unsigned)(device_cus() * 5), JT_THREADS, 0, s>>>(
            a, col_in, (const T *)val_in, col_out, (T *)val_out);
        SPMV_CHECK_LAUNCH("jds transpose");
    }
    jds_short_rows_kernel<TO_JDS, T><<<(unsigned)ceil_div(a.n, JT_THREADS), JT_THREADS, 0, s>>>(
        a, col_in, (const T *)val_in, col_out, (T *)val_out);
    SPMV_CHECK_LAUNCH("jds short rows");
    return SPMV_OK;
}

template <bool TO_JDS>
static spmv_status jds_transpose_dt(spmv_dtype dt, const JtArgs &a, const int32_t *col_in, const void *val_in,
                                    int32_t *col_out, void *val_out, WsCarver &wc, hipStream_t s)
{
    if (dt == SPMV_F64) return jds_transpose<TO_JDS, uint64_t>(a, col_in, val_in, col_out, val_out, wc, s);
    if (dt == SPMV_BF16) return jds_transpose<TO_JDS, uint16_t>(a, col_in, val_in, col_out, val_out, wc, s);
    return jds_transpose<TO_JDS, uint32_t>(a, col_in, val_in, col_out, val_out, wc, s);
}

// length of permuted row r from the diagonal lengths
__device__ __forceinline__ int32_t jds_len_of(const int32_t *__restrict__ jp, int32_t ndiag, int64_t r)
{
    int32_t lo = 0, hi = ndiag;
    while (lo < hi) {
        int32_t mid = (lo + hi) >> 1;
        if ((int64_t)(jp[mid + 1] - jp[mid]) > r) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__global__ void jds_row_len_kernel(const int32_t *__restrict__ jp, int32_t ndiag, const int32_t *__restrict__ perm,
                                   int32_t n, int32_t *__restrict__ len)
{
    GRID_LOOP(r, (int64_t)n) len[perm[r]] = jds_len_of(jp, ndiag, r);
}

__global__ void slice_nd_kernel(const int32_t *__restrict__ jp, int32_t ndiag, int32_t C, int32_t n_slices,
                                int32_t *__restrict__ nd, int64_t *__restrict__ sz)
{
    GRID_LOOP(s, (int64_t)n_slices)
    {
        int32_t l = jds_len_of(jp, ndiag, s * (int64_t)C);
        nd[s] = l;
        sz[s] = (int64_t)l * C;
    }
}

// JDS -> blocked JDS: both sides lie along the rows.  A wavefront copies 64
// rows of up to 32 diagonals, eight at a time; slots that their row does not
// reach become padding.  Tiles of 256 rows x 32 diagonals.  Bound: the copy rate (449 ->
// 142 us for 30 M entries with FP64 values).
constexpr int BT_U = 8;

template <typename T>
__global__ __launch_bounds__(BT_ROWS) void blocked_fill_kernel(const int32_t *__restrict__ jp, int32_t ndiag,
                                                               const int32_t *__restrict__ jd_col,
                                                               const T *__restrict__ jd_val, int32_t n_slices,
                                                               int32_t C, const int64_t *__restrict__ slice_ptr,
                                                               const int32_t *__restrict__ slice_nd, JtGroups g,
                                                               const int32_t *__restrict__ prefix,
                                                               int32_t *__restrict__ bl_col, T *__restrict__ bl_val)
{
    const int32_t tiles = prefix[g.K];
    for (int32_t b = (int32_t)blockIdx.x; b < tiles; b += (int32_t)gridDim.x) {
        const int32_t k = jt_group(prefix, g.K, b), i0 = b - prefix[k];
        const int64_t first = (((int64_t)k << g.q) + (i0 & ((1 << g.q) - 1))) * JT_DIAGS;
        if (first >= ndiag) continue;
        const int32_t d0 = (int32_t)first;
        // C is a multiple of 64: a wavefront's rows are in one slice
        const int64_t row0 = (int64_t)(i0 >> g.q) * BT_ROWS + (threadIdx.x & ~(WAVE - 1));
        const int64_t sl = __builtin_amdgcn_readfirstlane((int)(row0 / C));
        if (sl >= n_slices) continue;
        const int32_t last = (int32_t)min((int64_t)slice_nd[sl], first + JT_DIAGS);
        const int64_t r = row0 + lane_id(), dst0 = slice_ptr[sl] + (r - sl * C);
        for (int32_t d = d0; d < last; d += BT_U) {
            int32_t c[BT_U];
            T v[BT_U];
#pragma unroll
            for (int u = 0; u < BT_U; ++u) {
                const int32_t dd = min(d + u, ndiag - 1), from = jp[dd];
                c[u] = -1;
                v[u] = T{};
                if (d + u < last && r < jp[dd + 1] - from) {
                    c[u] = ld_stream(jd_col + from + r);
                    v[u] = ld_stream(jd_val + from + r);
                }
            }
#pragma unroll
            for (int u = 0; u < BT_U; ++u)
                if (d + u < last) {
                    bl_col[dst0 + (int64_t)(d + u) * C] = c[u];
                    bl_val[dst0 + (int64_t)(d + u) * C] = v[u];
                }
        }
    }
}

// Windowed RBJDS (rows sorted by length inside windows of sigma rows):
// window of the row each permuted position holds, the sort key of the
// second, stable pass.
__global__ void window_key_kernel(const int32_t *__restrict__ perm, int32_t n, int32_t sigma,
                                  uint32_t *__restrict__ key)
{
    GRID_LOOP(r, (int64_t)n) key[r] = (uint32_t)(perm[r] / sigma);
}

// slice s's depth = length of its first row (the longest: slices never span
// two windows and rows are sorted inside a window)
__global__ void window_slice_nd_kernel(const int32_t *__restrict__ rp, const int32_t *__restrict__ perm,
                                       int32_t C, int32_t n_slices, int32_t *__restrict__ nd,
                                       int64_t *__restrict__ sz)
{
    GRID_LOOP(s, (int64_t)n_slices)
    {
        const int32_t row = perm[s * (int64_t)C];
        const int32_t l = rp[row + 1] - rp[row];
        nd[s] = l;
        sz[s] = (int64_t)l * C;
    }
}

// slices of C rows in row order: depth = the slice's longest row
// One workgroup per window of SPMV_REM_WINDOW rows: each row's rank in the
// window's decreasing-length order (ties: lower row first) by counting over
// the window's lengths in LDS; the sorted position's window-local row (uint8)
// and global row (for the fill), and the depth of every slice of
// SPMV_REM_SLICE positions (its first row's length).
__global__ __launch_bounds__(SPMV_REM_WINDOW) void rem_order_kernel(const int32_t *__restrict__ rp, int32_t n,
                                                                     uint8_t *__restrict__ slot_row,
                                                                     int32_t *__restrict__ perm,
                                                                     int32_t *__restrict__ nd, int64_t *__restrict__ sz)
{
    __shared__ int32_t len[SPMV_REM_WINDOW];
    __shared__ int32_t at[SPMV_REM_WINDOW];
    const int64_t base = (int64_t)blockIdx.x * SPMV_REM_WINDOW;
    const int t = threadIdx.x;
    const int cnt = n - base < SPMV_REM_WINDOW ? (int)(n - base) : SPMV_REM_WINDOW;
    len[t] = t < cnt ? rp[base + t + 1] - rp[base + t] : -1;
    __syncthreads();
    if (t < cnt) {
        const int32_t l = len[t];
        int rank = 0;
        for (int j = 0; j < cnt; ++j) {
            const int32_t lj = len[j];
            rank += (lj > l) | ((lj == l) & (j < t));
        }
        at[rank] = t;
        slot_row[base + rank] = (uint8_t)t;
        perm[base + rank] = (int32_t)(base + t);
    }
    __syncthreads();
    if (t < cnt && t % SPMV_REM_SLICE == 0) {
        const int64_t sl = (base + t) / SPMV_REM_SLICE;
        const int32_t d = len[at[t]];
        nd[sl] = d;
        sz[sl] = (int64_t)d * SPMV_REM_SLICE;
    }
}

// slot k of the padded storage: entry d of permuted row r, taken from CRS in
// its row order, or padding (col = -1, value 0)
template <typename T>
__global__ void window_fill_kernel(const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
                                   const T *__restrict__ val, const int32_t *__restrict__ perm, int32_t n, int32_t C,
                                   const int64_t *__restrict__ slice_ptr, int32_t n_slices, int64_t total,
                                   int32_t *__restrict__ bl_col, T *__restrict__ bl_val)
{
    GRID_LOOP(k, total)
    {
        int32_t lo = 0, hi = n_slices - 1;
        while (lo < hi) {
            int32_t mid = (lo + hi + 1) >> 1;
            if (slice_ptr[mid] <= k) lo = mid;
            else hi = mid - 1;
        }
        const int64_t local = k - slice_ptr[lo];
        const int32_t d = (int32_t)(local / C);
        const int32_t rl = (int32_t)(local - (int64_t)d * C);
        const int64_t r = (int64_t)lo * C + rl;
        int32_t e = -1;
        if (r < n) {
            const int32_t row = perm[r];
            if (d < rp[row + 1] - rp[row]) e = rp[row] + d;
        }
        if (e >= 0) {
            bl_col[k] = col[e];
            bl_val[k] = val[e];
        } else {
            bl_col[k] = -1;
            bl_val[k] = T{};
        }
    }
}

// SOJDS: one thread per slice re-assigns each row's entries to diagonal slots
// (first row keeps CRS order; later rows take, slot by slot, the unused entry
// whose column is nearest to the previous row's column in that slot plus one,
// the smaller column on a tie).  `taken` holds one bit per entry of a row.
// A row whose columns strictly increase (CRS order of a matrix built by
// spmv_csr_from_coo) finds that entry in O(log L) loads: a binary search for
// the target column, then the nearest clear bit of `taken` on either side;
// any other row compares all of its unused entries.

// first clear bit at index >= from, or -1 if none below len
__device__ __forceinline__ int32_t next_clear(const uint32_t *taken, int32_t from, int32_t len)
{
    if (from >= len) return -1;
    int32_t w = from >> 5;
    uint32_t m = ~taken[w] & (0xffffffffu << (from & 31));
    const int32_t last = (len - 1) >> 5;
    while (m == 0) {
        if (++w > last) return -1;
        m = ~taken[w];
    }
    const int32_t e = (w << 5) + __ffs(m) - 1;
    return e < len ? e : -1;
}

// last clear bit at index < below, or -1 if none
__device__ __forceinline__ int32_t prev_clear(const uint32_t *taken, int32_t below)
{
    if (below <= 0) return -1;
    int32_t w = (below - 1) >> 5;
    uint32_t m = ~taken[w] & (0xffffffffu >> (31 - ((below - 1) & 31)));
    while (m == 0) {
        if (--w < 0) return -1;
        m = ~taken[w];
    }
    return (w << 5) + 31 - __clz(m);
}

// The same greedy rule with one wavefront per slice, for slices whose first
// row has at most SOJDS_LDS_CAP entries: the current row's columns (placed
// entries overwritten by a marker) and the previous row's slot columns live
// in LDS; for each slot the 64 lanes scan the row's unused entries (lane l:
// entries l, l+64, ...) for the one nearest to (previous row's column in that
// slot) + 1, smaller column on a tie, and a fixed shuffle tree picks the
// wavefront's best.  Columns of a row are distinct, so the pick is unique and
// matches the serial search whatever the entries' order.
constexpr int SOJDS_LDS_CAP = 4096;
constexpr int32_t SOJDS_TAKEN = INT32_MAX;    // no column reaches it (columns < n_cols <= INT32_MAX)

template <typename T>
__global__ __launch_bounds__(WAVE) void sojds_wave_kernel(const int32_t *__restrict__ jp, int32_t ndiag,
                                                          const int32_t *__restrict__ jd_col,
                                                          const T *__restrict__ jd_val, int32_t n, int32_t C,
                                                          const int64_t *__restrict__ slice_ptr,
                                                          int32_t *__restrict__ bl_col, T *__restrict__ bl_val)
{
    __shared__ int32_t cur[SOJDS_LDS_CAP];        // the row's columns; SOJDS_TAKEN once placed
    __shared__ int32_t prv[SOJDS_LDS_CAP];        // the previous row's column in each slot
    __shared__ int32_t pick[SOJDS_LDS_CAP];       // entry placed in each slot
    const int l = (int)threadIdx.x;
    const int64_t s = blockIdx.x;
    const int64_t r0 = s * (int64_t)C;
    const int32_t len0 = jds_len_of(jp, ndiag, r0);
    if (len0 > SOJDS_LDS_CAP || len0 == 0) return;       // whole wavefront: serial kernel's slice, or nothing to do
    const int64_t sp = slice_ptr[s];
    for (int32_t d = l; d < len0; d += WAVE) prv[d] = bl_col[sp + (int64_t)d * C];   // first row, CRS order
    __syncthreads();
    for (int32_t rl = 1; rl < C; ++rl) {
        const int64_t r = r0 + rl;
        if (r >= n) break;
        const int32_t len = jds_len_of(jp, ndiag, r);     // <= the previous row's length
        if (len == 0) break;                              // rows of the slice are sorted by length
        for (int32_t e = l; e < len; e += WAVE) cur[e] = jd_col[jp[e] + r];
        __syncthreads();
        for (int32_t d = 0; d < len; ++d) {
            // key = distance << 32 | column: the smallest key is the nearest
            // entry, the smaller column on a tie
            const uint32_t want = (uint32_t)prv[d] + 1u;
            uint64_t best = UINT64_MAX;
            int32_t be = -1;
            for (int32_t e = l; e < len; e += WAVE) {
                const int32_t c = cur[e];
                if (c == SOJDS_TAKEN) continue;
                const uint32_t uc = (uint32_t)c;
                const uint64_t key = ((uint64_t)(uc > want ? uc - want : want - uc) << 32) | uc;
                if (key < best) {
                    best = key;
                    be = e;
                }
            }
#pragma unroll
            for (int off = WAVE / 2; off > 0; off >>= 1) {
                const uint64_t ok = __shfl_xor(best, off, WAVE);
                const int32_t oe = __shfl_xor(be, off, WAVE);
                if (ok < best) {
                    best = ok;
                    be = oe;
                }
            }
            if (l == 0) {
                cur[be] = SOJDS_TAKEN;
                pick[d] = be;
                prv[d] = (int32_t)(uint32_t)best;        // the next row's target in this slot
            }
            __syncthreads();
        }
        for (int32_t d = l; d < len; d += WAVE) {
            const int32_t e = pick[d];
            bl_col[sp + (int64_t)d * C + rl] = prv[d];
            bl_val[sp + (int64_t)d * C + rl] = jd_val[jp[e] + r];
        }
        __syncthreads();
    }
}

template <typename T>
__global__ void sojds_kernel(const int32_t *__restrict__ jp, int32_t ndiag, const int32_t *__restrict__ jd_col,
                             const T *__restrict__ jd_val, int32_t n, int32_t C, const int64_t *__restrict__ slice_ptr,
                             int32_t n_slices, int32_t words, uint32_t *__restrict__ taken_all,
                             int32_t *__restrict__ bl_col, T *__restrict__ bl_val, int32_t min_len)
{
    GRID_LOOP(s, (int64_t)n_slices)
    {
        if (jds_len_of(jp, ndiag, s * (int64_t)C) <= min_len) continue;   // sojds_wave_kernel's slice
        uint32_t *taken = taken_all + s * (int64_t)words;
        const int64_t sp = slice_ptr[s];
        for (int32_t rl = 1; rl < C; ++rl) {
            const int64_t r = s * (int64_t)C + rl;
            if (r >= n) break;
            const int32_t len = jds_len_of(jp, ndiag, r);
            for (int32_t q = 0; q < (len + 31) / 32; ++q) taken[q] = 0;
            auto col_of = [&](int32_t e) -> int64_t { return jd_col[jp[e] + r]; };
            bool sorted = true;
            for (int32_t e = 1; e < len && sorted; ++e) sorted = col_of(e) > col_of(e - 1);
            for (int32_t d = 0; d < len; ++d) {
                const int64_t want = (int64_t)bl_col[sp + (int64_t)d * C + rl - 1] + 1;
                int32_t pick = -1;
                if (sorted) {
                    int32_t lo = 0, hi = len;                  // first entry with column >= want
                    while (lo < hi) {
                        const int32_t mid = (lo + hi) >> 1;
                        if (col_of(mid) < want) lo = mid + 1;
                        else hi = mid;
                    }
                    const int32_t right = next_clear(taken, lo, len), left = prev_clear(taken, lo);
                    if (left < 0) pick = right;
                    else if (right < 0) pick = left;
                    else pick = (col_of(right) - want < want - col_of(left)) ? right : left;   // tie: smaller column
                } else {
                    int64_t best = 0, bestc = 0;
                    for (int32_t e = 0; e < len; ++e) {
                        if (taken[e >> 5] & (1u << (e & 31))) continue;
                        const int64_t c = col_of(e);
                        const int64_t dist = c > want ? c - want : want - c;
                        if (pick < 0 || dist < best || (dist == best && c < bestc)) {
                            pick = e;
                            best = dist;
                            bestc = c;
                        }
                    }
                }
                taken[pick >> 5] |= 1u << (pick & 31);
                bl_col[sp + (int64_t)d * C + rl] = jd_col[jp[pick] + r];
                bl_val[sp + (int64_t)d * C + rl] = jd_val[jp[pick] + r];
            }
        }
    }
}

// ---- DIA + CRS hybrid: diagonals (offset col - row) stored densely, the rest in CRS

__global__ void diag_hist_kernel(const int32_t *__restrict__ rp, int32_t n_rows, const int32_t *__restrict__ col,
                                 int32_t *__restrict__ hist)
{
    GRID_LOOP(i, (int64_t)n_rows)
    {
        for (int32_t e = rp[i]; e < rp[i + 1]; ++e) atomicAdd(hist + ((int64_t)col[e] - i + n_rows - 1), 1);
    }
}

struct DiaOffsets {
    int32_t n;
    int32_t off[SPMV_DIA_MAX];
};

__global__ void dia_index_kernel(int64_t m, int32_t *__restrict__ oidx)
{
    GRID_LOOP(t, m) oidx[t] = -1;
}

// stored diagonal k: oidx = k; with `sym`, its mirror -off (off > 0) gets
// SPMV_DIA_MAX + k: covered by the stored diagonal, kept out of the remainder
__global__ void dia_index_set_kernel(int32_t n_rows, DiaOffsets D, int sym, int32_t *__restrict__ oidx)
{
    const int k = (int)threadIdx.x;
    if (k >= D.n) return;
    oidx[(int64_t)D.off[k] + n_rows - 1] = k;
    if (sym && D.off[k] > 0) oidx[(int64_t)n_rows - 1 - D.off[k]] = SPMV_DIA_MAX + k;
}

template <typename T>
__global__ void dia_zero_kernel(int64_t m, T *__restrict__ out)
{
    GRID_LOOP(t, m) out[t] = T{};
}

// entries on a stored diagonal go to dia[k * n_rows + row]; the others are
// counted per row for the remainder CRS
template <typename T>
__global__ void dia_scatter_kernel(const int32_t *__restrict__ rp, int32_t n_rows, const int32_t *__restrict__ col,
                                   const T *__restrict__ val, const int32_t *__restrict__ oidx, T *__restrict__ dia,
                                   int32_t *__restrict__ rem_cnt)
{
    GRID_LOOP(i, (int64_t)n_rows)
    {
        int32_t cnt = 0;
        for (int32_t e = rp[i]; e < rp[i + 1]; ++e) {
            const int32_t k = oidx[(int64_t)col[e] - i + n_rows - 1];
            if (k < 0) ++cnt;
            else if (k < SPMV_DIA_MAX) dia[(int64_t)k * n_rows + i] = val[e];
        }
        rem_cnt[i] = cnt;
    }
}

// remainder entries of each row, in CRS order
template <typename T>
__global__ void dia_rem_kernel(const int32_t *__restrict__ rp, int32_t n_rows, const int32_t *__restrict__ col,
                               const T *__restrict__ val, const int32_t *__restrict__ oidx,
                               const int32_t *__restrict__ rem_rp, int32_t *__restrict__ rem_col,
                               T *__restrict__ rem_val)
{
    GRID_LOOP(i, (int64_t)n_rows)
    {
        int32_t p = rem_rp[i];
        for (int32_t e = rp[i]; e < rp[i + 1]; ++e) {
            if (oidx[(int64_t)col[e] - i + n_rows - 1] >= 0) continue;
            rem_col[p] = col[e];
            rem_val[p] = val[e];
            ++p;
        }
    }
}

// ---- row split: part k = rows [b_k, b_{k+1}), cut so each holds about nnz/8 entries

__global__ void row_bounds_kernel(const int32_t *__restrict__ rp, int32_t n_rows, int64_t nnz,
                                  int64_t *__restrict__ bounds, int64_t *__restrict__ entry_bounds)
{
    const int k = (int)threadIdx.x;
    if (k > SPLIT_PARTS) return;
    int64_t b;
    if (k == 0) b = 0;
    else if (k == SPLIT_PARTS) b = n_rows;
    else if (nnz == 0) b = (int64_t)k * n_rows / SPLIT_PARTS;
    else b = lower_bound_dev(rp, (int64_t)n_rows + 1, (k * nnz + SPLIT_PARTS - 1) / SPLIT_PARTS);
    if (b > n_rows) b = n_rows;     // only if row_ptr[n_rows] < nnz, which the host reports
    bounds[k] = b;
    entry_bounds[k] = rp[b];
}

// part k's rebased row pointer at row_ptr_parts[b_k + k .. b_{k+1} + k]
__global__ void row_split_ptr_kernel(const int32_t *__restrict__ rp, int32_t n_rows,
                                     const int64_t *__restrict__ bounds, int32_t *__restrict__ out)
{
    GRID_LOOP(j, (int64_t)n_rows + SPLIT_PARTS)
    {
        int k = 0;
        while (k < SPLIT_PARTS - 1 && j > bounds[k + 1] + k) ++k;
        const int64_t row = bounds[k] + (j - bounds[k] - k);
        out[j] = rp[row] - rp[bounds[k]];
    }
}

// ---- column split: part k = entries whose column lies in [k*width, (k+1)*width)

__global__ void row_of_entries_kernel(const int32_t *__restrict__ rp, int32_t n, int64_t nnz, int32_t *__restrict__ rowid)
{
    GRID_LOOP(j, nnz) rowid[j] = row_of(rp, n, j);
}

__global__ void part_key_kernel(const int32_t *__restrict__ col, int64_t nnz, int32_t width, uint32_t *__restrict__ key)
{
    GRID_LOOP(j, nnz) key[j] = (uint32_t)(col[j] / width);
}

template <typename T>
__global__ void gather_split_kernel(const int32_t *__restrict__ perm, int64_t nnz, const int32_t *__restrict__ col,
                                    const T *__restrict__ val, const int32_t *__restrict__ rowid,
                                    int32_t *__restrict__ col_out, T *__restrict__ val_out,
                                    int32_t *__restrict__ rowid_out)
{
    GRID_LOOP(i, nnz)
    {
        const int32_t j = perm[i];
        col_out[i] = col[j];
        val_out[i] = val[j];
        rowid_out[i] = rowid[j];
    }
}

__global__ void part_bounds_kernel(const uint32_t *__restrict__ skey, int64_t nnz, int64_t *__restrict__ bounds)
{
    GRID_LOOP(p, (int64_t)SPLIT_PARTS + 1) bounds[p] = lower_bound_dev(skey, nnz, (int64_t)p);
}

// Compressed rows: a part keeps only the rows holding at least one of its
// entries.  head[i] = 1 where entry i (part-major order) opens a (row, part)
// group; the exclusive scan of head numbers the compressed rows.
__global__ void split_head_kernel(const uint32_t *__restrict__ skey, const int32_t *__restrict__ rowid_s, int64_t nnz,
                                  int32_t *__restrict__ head)
{
    GRID_LOOP(i, nnz) head[i] = (i == 0 || skey[i] != skey[i - 1] || rowid_s[i] != rowid_s[i - 1]) ? 1 : 0;
}

// row pointer of each compressed row (relative to its part's first entry) and
// the parts present in each original row (bit k of mask[row])
__global__ void split_rows_kernel(const uint32_t *__restrict__ skey, const int32_t *__restrict__ rowid_s,
                                  const int32_t *__restrict__ head, const int32_t *__restrict__ qidx, int64_t nnz,
                                  const int64_t *__restrict__ bounds, int32_t *__restrict__ row_ptr_all,
                                  uint32_t *__restrict__ mask)
{
    GRID_LOOP(i, nnz)
    {
        if (!head[i]) continue;
        const uint32_t k = skey[i];
        row_ptr_all[qidx[i] + k] = (int32_t)(i - bounds[k]);
        atomicOr(mask + rowid_s[i], 1u << k);
    }
}

__global__ void split_terminators_kernel(const int64_t *__restrict__ bounds, const int32_t *__restrict__ qidx,
                                         int32_t *__restrict__ row_ptr_all, int64_t *__restrict__ row_off)
{
    const int k = (int)threadIdx.x;
    if (k <= SPLIT_PARTS) row_off[k] = qidx[bounds[k]];
    if (k < SPLIT_PARTS) row_ptr_all[qidx[bounds[k + 1]] + k] = (int32_t)(bounds[k + 1] - bounds[k]);
}

__global__ void popcount_kernel(const uint32_t *__restrict__ mask, int32_t n, int32_t *__restrict__ cnt)
{
    GRID_LOOP(i, (int64_t)n) cnt[i] = __popc(mask[i]);
}

// slot of compressed row (row, k): row's slots are ordered by part
__global__ void split_dest_kernel(const uint32_t *__restrict__ skey, const int32_t *__restrict__ rowid_s,
                                  const int32_t *__restrict__ head, const int32_t *__restrict__ qidx, int64_t nnz,
                                  const uint32_t *__restrict__ mask, const int32_t *__restrict__ slot_ptr,
                                  int32_t *__restrict__ dest_all)
{
    GRID_LOOP(i, nnz)
    {
        if (!head[i]) continue;
        const uint32_t k = skey[i];
        const int32_t r = rowid_s[i];
        dest_all[qidx[i]] = slot_ptr[r] + __popc(mask[r] & ((1u << k) - 1u));
    }
}

__global__ void transpose_cols_kernel(const int32_t *__restrict__ rp, int32_t n_rows, const int32_t *__restrict__ tmap,
                                      int64_t nnz, int32_t *__restrict__ colT)
{
    GRID_LOOP(t, nnz) colT[t] = row_of(rp, n_rows, tmap[t]);
}

// one round-to-nearest-even step from double to bfloat16
__device__ __forceinline__ uint16_t f64_to_bf16_rne(double d)
{
    const uint64_t b = (uint64_t)__double_as_longlong(d);
    const uint16_t sign = (uint16_t)((b >> 48) & 0x8000u);
    const uint64_t a = b & 0x7fffffffffffffffull;
    if (a > 0x7ff0000000000000ull) return (uint16_t)(sign | 0x7fc0u);        // NaN
    if (a == 0x7ff0000000000000ull) return (uint16_t)(sign | 0x7f80u);       // inf
    const int e = (int)(a >> 52) - 1023;
    if (e >= -126) {
        uint64_t q = a >> 45;                        // exponent + 7 mantissa bits
        const uint64_t rem = a & ((1ull << 45) - 1);
        const uint64_t half = 1ull << 44;
        if (rem > half || (rem == half && (q & 1))) ++q;
        int64_t bits = (int64_t)q - ((int64_t)(1023 - 127) << 7);
        if (bits >= 0x7f80) bits = 0x7f80;            // overflow to infinity
        return (uint16_t)(sign | (uint16_t)bits);
    }
    // below the smallest normal: multiples of 2^-133, ties to even
    const double m = rint(__longlong_as_double((long long)a) * 0x1p133);
    return (uint16_t)(sign | (uint16_t)m);
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    const uint32_t lsb = (u >> 16) & 1u;
    return (uint16_t)((u + 0x7fffu + lsb) >> 16);
}

__global__ void convert_kernel(int64_t n, const void *__restrict__ in, int in_dt, void *__restrict__ out, int out_dt)
{
    GRID_LOOP(i, n)
    {
        if (in_dt == SPMV_F64) {
            const double v = ((const double *)in)[i];
            if (out_dt == SPMV_F32) ((float *)out)[i] = (float)v;
            else if (out_dt == SPMV_BF16) ((uint16_t *)out)[i] = f64_to_bf16_rne(v);
            else ((double *)out)[i] = v;
        } else if (in_dt == SPMV_F32) {
            const float v = ((const float *)in)[i];
            if (out_dt == SPMV_F64) ((double *)out)[i] = (double)v;
            else if (out_dt == SPMV_BF16) ((uint16_t *)out)[i] = f32_to_bf16_rne(v);
            else ((float *)out)[i] = v;
        } else {
            const float v = __uint_as_float((uint32_t)((const uint16_t *)in)[i] << 16);
            if (out_dt == SPMV_F64) ((double *)out)[i] = (double)v;
            else if (out_dt == SPMV_F32) ((float *)out)[i] = v;
            else ((uint16_t *)out)[i] = ((const uint16_t *)in)[i];
        }
    }
}

template <typename T>
__global__ void permute_kernel(int32_t n, const int32_t *__restrict__ perm, const T *__restrict__ in,
                               T *__restrict__ out, int inverse)
{
    GRID_LOOP(r, (int64_t)n)
    {
        if (inverse) out[perm[r]] = in[r];
        else out[r] = in[perm[r]];
    }
}

template <typename T>
__global__ void gather_kernel(int64_t n, const int32_t *__restrict__ map, const T *__restrict__ in, T *__restrict__ out)
{
    GRID_LOOP(i, n) out[i] = in[map[i]];
}

// dtype-dispatched launch of a kernel templated on the element type
template <template <typename> class K>
struct DtDispatch;

// ============================================================ host helpers

}  // namespace spmv

using namespace spmv;

extern "C" {

size_t spmv_csr_validate_workspace_size(void) { return 256; }

spmv_status spmv_csr_validate(int32_t n_rows, int32_t n_cols, int64_t nnz, const int32_t *row_ptr,
                              const int32_t *col_idx, int32_t *h_ok, void *ws, size_t ws_bytes, void *stream)
{
    SPMV_REQUIRE(n_rows >= 0 && n_cols >= 0 && nnz >= 0, "spmv_csr_validate: negative size");
    SPMV_REQUIRE(h_ok && row_ptr && ws && ws_bytes >= 4, "spmv_csr_validate: null pointer");
    SPMV_REQUIRE(nnz == 0 || col_idx, "spmv_csr_validate: null col_idx");
    hipStream_t s = as_stream(stream);
    int32_t *bad = (int32_t *)ws;
    SPMV_HIP(hipMemsetAsync(bad, 0, sizeof(int32_t), s));
    if (n_rows > 0) validate_rows_kernel<<<grid_for(n_rows), 256, 0, s>>>(row_ptr, n_rows, nnz, bad);
    if (nnz > 0) validate_cols_kernel<<<grid_for(nnz), 256, 0, s>>>(col_idx, nnz, n_cols, bad);
    SPMV_CHECK_LAUNCH("spmv_csr_validate");
    int32_t b = 0;
    if (read_flag(bad, &b, s) != SPMV_OK) return SPMV_ERR_HIP;
    if (n_rows == 0) {
        int32_t first = 0;
        if (read_flag(row_ptr, &first, s) != SPMV_OK) return SPMV_ERR_HIP;
        if (first != 0 || nnz != 0) b |= 2;
    }
    *h_ok = b == 0 ? 1 : 0;
    return SPMV_OK;
}

size_t spmv_jds_from_csr_workspace_size(int32_t n, int64_t nnz)
{
    size_t m = (size_t)(n > 0 ? n : 1);
    size_t b = 0;
    b += 256;                                       // max length
    b += align_up(sizeof(int32_t) * m, 256);        // lengths
    b += align_up(sizeof(uint32_t) * m, 256);       // keys
    b += align_up(sizeof(int32_t) * scan_ws_elems((int64_t)(m > (size_t)nnz ? m : (size_t)nnz)), 256);
    b += radix_ws_bytes((int64_t)m) + jt_ws_bytes();
    return b + 1024;
}

spmv_status spmv_jds_from_csr(int32_t n, int64_t nnz, const int32_t *row_ptr, const int32_t *col_idx,
                              const void *val, spmv_dtype dt, unsigned flags, int32_t *perm, int32_t *iperm,
                              int32_t *jd_ptr, int32_t jd_ptr_cap, int32_t *jd_col, void *jd_val, int32_t *h_ndiag,
                              int32_t *h_jd_ptr, void *ws, size_t ws_bytes, void *stream)
{
    SPMV_REQUIRE(n >= 0 && nnz >= 0, "spmv_jds_from_csr: negative size");
    if (nnz >= ((int64_t)1 << 31)) return fail(SPMV_ERR_UNSUPPORTED, "spmv_jds_from_csr: nnz >= 2^31");
    SPMV_REQUIRE(valid_payload_dtype(dt), "spmv_jds_from_csr: bad dtype");
    SPMV_REQUIRE((flags & ~SPMV_SYMPERM) == 0, "spmv_jds_from_csr: unknown flag");
    SPMV_REQUIRE(h_ndiag && row_ptr && (jd_ptr || jd_ptr_cap == 0), "spmv_jds_from_csr: null pointer");
    SPMV_REQUIRE(n == 0 || (perm && iperm), "spmv_jds_from_csr: null perm");
    SPMV_REQUIRE(nnz == 0 || (col_idx && val && jd_col && jd_val), "spmv_jds_from_csr: null arrays");
    SPMV_REQUIRE(ws && ws_bytes >= spmv_jds_from_csr_workspace_size(n, nnz), "spmv_jds_from_csr: workspace too small");
    hipStream_t s = as_stream(stream);
    WsCarver wc(ws, ws_bytes);
    int32_t *maxlen = wc.take<int32_t>(1);
    int32_t *len = wc.take<int32_t>((size_t)(n > 0 ? n : 1));
    uint32_t *keys = wc.take<uint32_t>((size_t)(n > 0 ? n : 1));
    int32_t *sws = wc.take<int32_t>(scan_ws_elems((int64_t)n > nnz ? (int64_t)n : (nnz > 0 ? nnz : 1)));
    size_t rws_bytes = radix_ws_bytes(n);
    void *rws = wc.take<char>(rws_bytes);
    if (!wc.ok()) return fail(SPMV_ERR_INVALID_ARG, "spmv_jds_from_csr: workspace too small");

    int32_t ndiag = 0;
    if (n > 0) {
        SPMV_HIP(hipMemsetAsync(maxlen, 0, sizeof(int32_t), s));
        row_len_kernel<<<std::min(grid_for(n), 1024u), 256, 0, s>>>(row_ptr, n, len, maxlen);
        SPMV_CHECK_LAUNCH("jds lengths");
        if (read_flag(maxlen, &ndiag, s) != SPMV_OK) return SPMV_ERR_HIP;
    }
    *h_ndiag = ndiag;
    if (jd_ptr_cap < ndiag + 1) return fail(SPMV_ERR_CAPACITY, "spmv_jds_from_csr: jd_ptr capacity < ndiag+1");
    if (n == 0) {
        SPMV_HIP(hipMemsetAsync(jd_ptr, 0, sizeof(int32_t), s));
        SPMV_HIP(hipStreamSynchronize(s));
        if (h_jd_ptr) h_jd_ptr[0] = 0;
        return SPMV_OK;
    }
    // stable sort of the rows by decreasing length: key = ndiag - length
    uint32_t *skey = (uint32_t *)len;
    desc_key_kernel<<<grid_for(n), 256, 0, s>>>(len, n, ndiag, skey);
    SPMV_CHECK_LAUNCH("jds keys");
    spmv_status st = radix_sort_pairs(keys, perm, n, bits_for(ndiag), rws, rws_bytes, s, skey);
    if (st != SPMV_OK) return st;
    inverse_perm_kernel<<<grid_for(n), 256, 0, s>>>(perm, n, iperm);
    SPMV_CHECK_LAUNCH("jds iperm");
    if (ndiag > 0) {
        // diagonal lengths go into jd_ptr itself, then an in-place scan
        diag_count_kernel<<<grid_for(ndiag), 256, 0, s>>>(keys, n, ndiag, jd_ptr);
        SPMV_CHECK_LAUNCH("jds diagonal counts");
        st = exclusive_scan<int32_t, int32_t>(jd_ptr, ndiag, jd_ptr, sws, s);
        if (st != SPMV_OK) return st;
    } else {
        SPMV_HIP(hipMemsetAsync(jd_ptr, 0, sizeof(int32_t), s));
    }
    if (nnz > 0 && ndiag > 0) {          // row_ptr may hold no entries whatever nnz says
        JtArgs t{};
        t.rp = row_ptr;
        t.perm = perm;
        t.iperm = iperm;
        t.jp = jd_ptr;
        t.n = n;
        t.ndiag = ndiag;
        t.symperm = (flags & SPMV_SYMPERM) ? 1 : 0;
        st = jds_transpose_dt<true>(dt, t, col_idx, val, jd_col, jd_val, wc, s);
        if (st != SPMV_OK) return st;
    }
    if (h_jd_ptr)
        SPMV_HIP(hipMemcpyAsync(h_jd_ptr, jd_ptr, sizeof(int32_t) * ((size_t)ndiag + 1), hipMemcpyDeviceToHost, s));
    SPMV_HIP(hipStreamSynchronize(s));
    return SPMV_OK;
}

size_t spmv_jds_to_csr_workspace_size(int32_t n)
{
    size_t m = (size_t)(n > 0 ? n : 1);
    return align_up(sizeof(int32_t) * m, 256) + align_up(sizeof(int32_t) * scan_ws_elems((int64_t)m), 256) +
           jt_ws_bytes() + 512;
}

spmv_status spmv_jds_to_csr(int32_t n, const int32_t *perm, const int32_t *jd_ptr, int32_t ndiag, const int32_t *jd_col,
                            const void *jd_val, spmv_dtype dt, unsigned flags, int32_t *row_ptr, int32_t *col_idx,
                            void *val, void *ws, size_t ws_bytes, void *stream)
{
    SPMV_REQUIRE(n >= 0 && ndiag >= 0, "spmv_jds_to_csr: negative size");
    SPMV_REQUIRE(valid_payload_dtype(dt), "spmv_jds_to_csr: bad dtype");
    SPMV_REQUIRE((flags & ~SPMV_SYMPERM) == 0, "spmv_jds_to_csr: unknown flag");
    SPMV_REQUIRE(row_ptr && jd_ptr, "spmv_jds_to_csr: null pointer");
    SPMV_REQUIRE(ws && ws_bytes >= spmv_jds_to_csr_workspace_size(n), "spmv_jds_to_csr: workspace too small");
    hipStream_t s = as_stream(stream);
    WsCarver wc(ws, ws_bytes);
    int32_t *len = wc.take<int32_t>((size_t)(n > 0 ? n : 1));
    int32_t *sws = wc.take<int32_t>(scan_ws_elems(n > 0 ? n : 1));
    if (n == 0) {
        SPMV_HIP(hipMemsetAsync(row_ptr, 0, sizeof(int32_t), s));
        return SPMV_OK;
    }
    SPMV_REQUIRE(perm, "spmv_jds_to_csr: null perm");
    jds_row_len_kernel<<<std::min(grid_for(n), 1024u), 256, 0, s>>>(jd_ptr, ndiag, perm, n, len);
    SPMV_CHECK_LAUNCH("jds_to_csr lengths");
    spmv_status st = exclusive_scan<int32_t, int32_t>(len, n, row_ptr, sws, s);
    if (st != SPMV_OK) return st;
    if (ndiag == 0) return SPMV_OK;
    if (!(jd_col && jd_val && col_idx && val)) {         // only a matrix without entries needs no arrays
        int32_t nnz = 0;
        if (read_flag(row_ptr + n, &nnz, s) != SPMV_OK) return SPMV_ERR_HIP;
        SPMV_REQUIRE(nnz == 0, "spmv_jds_to_csr: null arrays");
        return SPMV_OK;
    }
    JtArgs t{};
    t.rp = row_ptr;
    t.perm = perm;
    t.iperm = len;                                       // the lengths are in row_ptr now
    inverse_perm_kernel<<<grid_for(n), 256, 0, s>>>(perm, n, len);
    SPMV_CHECK_LAUNCH("jds_to_csr iperm");
    t.jp = jd_ptr;
    t.n = n;
    t.ndiag = ndiag;
    t.symperm = (flags & SPMV_SYMPERM) ? 1 : 0;
    st = jds_transpose_dt<false>(dt, t, jd_col, jd_val, col_idx, val, wc, s);
    if (st != SPMV_OK) return st;
    return SPMV_OK;
}

size_t spmv_jds_blocked_windowed_workspace_size(int32_t n)
{
    size_t m = (size_t)(n > 0 ? n : 1);
    size_t b = 256;                                              // longest row
    b += align_up(sizeof(int32_t) * m, 256);                     // lengths
    b += align_up(sizeof(uint32_t) * m, 256);                    // sort keys
    b += radix_ws_bytes((int64_t)m);
    b += align_up(sizeof(int64_t) * m, 256);                     // slice sizes (at most n slices)
    b += align_up(sizeof(int64_t) * scan_ws_elems((int64_t)m), 256);
    return b + 1024;
}

size_t spmv_jds_blocked_workspace_size(int32_t n, int32_t ndiag, int32_t C, unsigned flags)
{
    if (C <= 0) return 0;
    size_t ns = (size_t)ceil_div(n > 0 ? n : 1, C);
    size_t b = align_up(sizeof(int64_t) * ns, 256) + align_up(sizeof(int64_t) * scan_ws_elems((int64_t)ns), 256);
    if (flags & SPMV_SOJDS) b += align_up(sizeof(uint32_t) * ns * (size_t)ceil_div(ndiag > 0 ? ndiag : 1, 32), 256);
    return b + jt_ws_bytes() + 1024;
}

spmv_status spmv_jds_blocked_from_jds(int32_t n, const int32_t *jd_ptr, int32_t ndiag, const int32_t *jd_col,
                                      const void *jd_val, spmv_dtype dt, int32_t C, unsigned flags, int64_t *slice_ptr,
                                      int32_t *slice_nd, int32_t *bl_col, void *bl_val, int64_t bl_cap,
                                      int64_t *h_padded, int32_t *h_slice_nd, void *ws, size_t ws_bytes, void *stream)
{
    SPMV_REQUIRE(n >= 0 && ndiag >= 0, "spmv_jds_blocked_from_jds: negative size");
    SPMV_REQUIRE(C > 0 && C % 64 == 0, "spmv_jds_blocked_from_jds: C must be a positive multiple of 64");
    SPMV_REQUIRE(valid_payload_dtype(dt), "spmv_jds_blocked_from_jds: bad dtype");
    SPMV_REQUIRE((flags & ~SPMV_SOJDS) == 0, "spmv_jds_blocked_from_jds: unknown flag");
    SPMV_REQUIRE(jd_ptr && slice_ptr && h_padded, "spmv_jds_blocked_from_jds: null pointer");
    SPMV_REQUIRE(ws && ws_bytes >= spmv_jds_blocked_workspace_size(n, ndiag, C, flags),
                 "spmv_jds_blocked_from_jds: workspace too small");
    hipStream_t s = as_stream(stream);
    const int32_t ns = (int32_t)ceil_div(n, C);
    WsCarver wc(ws, ws_bytes);
    int64_t *sz = wc.take<int64_t>((size_t)(ns > 0 ? ns : 1));
    int64_t *sws = wc.take<int64_t>(scan_ws_elems(ns > 0 ? ns : 1));
    uint32_t *taken = (flags & SPMV_SOJDS) ? wc.take<uint32_t>((size_t)(ns > 0 ? ns : 1) *
                                                               (size_t)ceil_div(ndiag > 0 ? ndiag : 1, 32))
                                           : nullptr;
    int32_t *prefix = wc.take<int32_t>(JT_GROUPS + 1);
    if (ns == 0) {
        SPMV_HIP(hipMemsetAsync(slice_ptr, 0, sizeof(int64_t), s));
        SPMV_HIP(hipStreamSynchronize(s));
        *h_padded = 0;
        return SPMV_OK;
    }
    SPMV_REQUIRE(slice_nd, "spmv_jds_blocked_from_jds: null slice_nd");
    slice_nd_kernel<<<grid_for(ns), 256, 0, s>>>(jd_ptr, ndiag, C, ns, slice_nd, sz);
    SPMV_CHECK_LAUNCH("blocked slice sizes");
    spmv_status st = exclusive_scan<int64_t, int64_t>(sz, ns, slice_ptr, sws, s);
    if (st != SPMV_OK) return st;
    int64_t total = 0;
    SPMV_HIP(hipMemcpyAsync(&total, slice_ptr + ns, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    if (h_slice_nd) SPMV_HIP(hipMemcpyAsync(h_slice_nd, slice_nd, sizeof(int32_t) * ns, hipMemcpyDeviceToHost, s));
    SPMV_HIP(hipStreamSynchronize(s));
    *h_padded = total;
    if (bl_cap < total) return fail(SPMV_ERR_CAPACITY, "spmv_jds_blocked_from_jds: capacity < padded size");
    if (total == 0) return SPMV_OK;
    SPMV_REQUIRE(jd_col && jd_val && bl_col && bl_val, "spmv_jds_blocked_from_jds: null arrays");
    const int32_t words = (int32_t)ceil_div(ndiag > 0 ? ndiag : 1, 32);
    const JtGroups g = jt_groups(ndiag);
    jt_table_kernel<<<1, SCAN_THREADS, 0, s>>>(jd_ptr, ndiag, C, g, prefix);
    SPMV_CHECK_LAUNCH("blocked tiles");
#define BLK_CASE(DT, T)                                                                                             \
    if (dt == DT) {                                                                                                 \
        blocked_fill_kernel<T><<<(unsigned)(device_cus() * 8), BT_ROWS, 0, s>>>(                                    \
            jd_ptr, ndiag, jd_col, (const T *)jd_val, ns, C, slice_ptr, slice_nd, g, prefix, bl_col, (T *)bl_val);  \
        SPMV_CHECK_LAUNCH("blocked fill");                                                                          \
        if (flags & SPMV_SOJDS) {                                                                                   \
            sojds_wave_kernel<T><<<(unsigned)ns, WAVE, 0, s>>>(jd_ptr, ndiag, jd_col, (const T *)jd_val, n, C,       \
                                                               slice_ptr, bl_col, (T *)bl_val);                     \
            SPMV_CHECK_LAUNCH("sojds (wavefront per slice)");                                                       \
            if (ndiag > SOJDS_LDS_CAP) {                                                                            \
                sojds_kernel<T><<<grid_for(ns), 64, 0, s>>>(jd_ptr, ndiag, jd_col, (const T *)jd_val, n, C,         \
                                                            slice_ptr, ns, words, taken, bl_col, (T *)bl_val,       \
                                                            SOJDS_LDS_CAP);                                         \
                SPMV_CHECK_LAUNCH("sojds (long rows)");                                                             \
            }                                                                                                       \
        }                                                                                                           \
    }
    BLK_CASE(SPMV_F64, uint64_t)
    BLK_CASE(SPMV_F32, uint32_t)
    BLK_CASE(SPMV_I32, uint32_t)
    BLK_CASE(SPMV_BF16, uint16_t)
#undef BLK_CASE
    SPMV_HIP(hipStreamSynchronize(s));
    return SPMV_OK;
}

spmv_status spmv_jds_blocked_windowed_from_csr(int32_t n, int64_t nnz, const int32_t *row_ptr, const int32_t *col_idx,
                                               const void *val, spmv_dtype dt, int32_t C, int32_t sigma,
                                               int32_t *perm, int64_t *slice_ptr, int32_t *slice_nd,
                                               int32_t *bl_col, void *bl_val, int64_t bl_cap, int64_t *h_padded,
                                               int32_t *h_slice_nd, void *ws, size_t ws_bytes, void *stream)
{
    SPMV_REQUIRE(n >= 0 && nnz >= 0, "spmv_jds_blocked_windowed_from_csr: negative size");
    if (nnz >= ((int64_t)1 << 31)) return fail(SPMV_ERR_UNSUPPORTED, "spmv_jds_blocked_windowed_from_csr: nnz >= 2^31");
    SPMV_REQUIRE(C > 0 && C % 64 == 0, "spmv_jds_blocked_windowed_from_csr: C must be a positive multiple of 64");
    SPMV_REQUIRE(sigma > 0 && sigma % C == 0, "spmv_jds_blocked_windowed_from_csr: sigma must be a positive multiple of C");
    SPMV_REQUIRE(valid_payload_dtype(dt), "spmv_jds_blocked_windowed_from_csr: bad dtype");
    SPMV_REQUIRE(row_ptr && slice_ptr && h_padded, "spmv_jds_blocked_windowed_from_csr: null pointer");
    SPMV_REQUIRE(ws && ws_bytes >= spmv_jds_blocked_windowed_workspace_size(n),
                 "spmv_jds_blocked_windowed_from_csr: workspace too small");
    hipStream_t s = as_stream(stream);
    const int32_t ns = (int32_t)ceil_div(n, C);
    if (ns == 0) {
        SPMV_HIP(hipMemsetAsync(slice_ptr, 0, sizeof(int64_t), s));
        SPMV_HIP(hipStreamSynchronize(s));
        *h_padded = 0;
        return SPMV_OK;
    }
    SPMV_REQUIRE(perm && slice_nd, "spmv_jds_blocked_windowed_from_csr: null perm or slice_nd");
    const size_t m = (size_t)n;
    WsCarver wc(ws, ws_bytes);
    int32_t *maxlen = wc.take<int32_t>(1);
    int32_t *len = wc.take<int32_t>(m);
    uint32_t *keys = wc.take<uint32_t>(m);
    const size_t rws_bytes = radix_ws_bytes((int64_t)m);
    void *rws = wc.take<char>(rws_bytes);
    int64_t *sz = wc.take<int64_t>(m);
    int64_t *sws = wc.take<int64_t>(scan_ws_elems((int64_t)m));
    if (!wc.ok()) return fail(SPMV_ERR_INVALID_ARG, "spmv_jds_blocked_windowed_from_csr: workspace too small");
    int32_t ndiag = 0;
    SPMV_HIP(hipMemsetAsync(maxlen, 0, sizeof(int32_t), s));
    row_len_kernel<<<std::min(grid_for(n), 1024u), 256, 0, s>>>(row_ptr, n, len, maxlen);
    SPMV_CHECK_LAUNCH("windowed lengths");
    if (read_flag(maxlen, &ndiag, s) != SPMV_OK) return SPMV_ERR_HIP;
    // rows by decreasing length (stable), then by window (stable): window-major,
    // longest first inside a window, ties in original order
    uint32_t *skey = (uint32_t *)len;
    desc_key_kernel<<<grid_for(n), 256, 0, s>>>(len, n, ndiag, skey);
    SPMV_CHECK_LAUNCH("windowed keys");
    spmv_status st = radix_sort_pairs(keys, perm, n, bits_for(ndiag), rws, rws_bytes, s, skey);
    if (st != SPMV_OK) return st;
    window_key_kernel<<<grid_for(n), 256, 0, s>>>(perm, n, sigma, keys);
    SPMV_CHECK_LAUNCH("windowed window keys");
    st = radix_sort_pairs(keys, perm, n, bits_for((int64_t)(n - 1) / sigma), rws, rws_bytes, s);
    if (st != SPMV_OK) return st;
    window_slice_nd_kernel<<<grid_for(ns), 256, 0, s>>>(row_ptr, perm, C, ns, slice_nd, sz);
    SPMV_CHECK_LAUNCH("windowed slice sizes");
    st = exclusive_scan<int64_t, int64_t>(sz, ns, slice_ptr, sws, s);
    if (st != SPMV_OK) return st;
    int64_t total = 0;
    SPMV_HIP(hipMemcpyAsync(&total, slice_ptr + ns, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    if (h_slice_nd) SPMV_HIP(hipMemcpyAsync(h_slice_nd, slice_nd, sizeof(int32_t) * ns, hipMemcpyDeviceToHost, s));
    SPMV_HIP(hipStreamSynchronize(s));
    *h_padded = total;
    if (bl_cap < total) return fail(SPMV_ERR_CAPACITY, "spmv_jds_blocked_windowed_from_csr: capacity < padded size");
    if (total == 0) return SPMV_OK;
    SPMV_REQUIRE(col_idx && val && bl_col && bl_val, "spmv_jds_blocked_windowed_from_csr: null arrays");
#define WFILL_CASE(T)                                                                                              \
    window_fill_kernel<T><<<grid_for(total), 256, 0, s>>>(row_ptr, col_idx, (const T *)val, perm, n, C, slice_ptr, \
                                                          ns, total, bl_col, (T *)bl_val)
    if (dt == SPMV_F64) WFILL_CASE(uint64_t);
    else if (dt == SPMV_F32 || dt == SPMV_I32) WFILL_CASE(uint32_t);
    else WFILL_CASE(uint16_t);
#undef WFILL_CASE
    SPMV_CHECK_LAUNCH("windowed fill");
    SPMV_HIP(hipStreamSynchronize(s));
    return SPMV_OK;
}

size_t spmv_csr_slices_workspace_size(int32_t n_rows)
{
    const int64_t n = n_rows > 0 ? n_rows : 1;
    const int64_t ns = ceil_div(n, SPMV_REM_SLICE);
    return align_up(sizeof(int32_t) * (size_t)n, 256) + align_up(sizeof(int64_t) * (size_t)ns, 256) +
           align_up(sizeof(int64_t) * scan_ws_elems(ns), 256) + 512;
}

spmv_status spmv_csr_to_slices(int32_t n_rows, const int32_t *row_ptr, const int32_t *col_idx, const void *val,
                               spmv_dtype dt, int64_t *slice_ptr, int32_t *slice_nd, uint8_t *slot_row,
                               int32_t *bl_col, void *bl_val, int64_t bl_cap, int64_t *h_padded, void *ws,
                               size_t ws_bytes, void *stream)
{
    SPMV_REQUIRE(n_rows >= 0, "spmv_csr_to_slices: n_rows < 0");
    SPMV_REQUIRE(valid_payload_dtype(dt), "spmv_csr_to_slices: bad dtype");
    SPMV_REQUIRE(slice_ptr && h_padded, "spmv_csr_to_slices: null pointer");
    SPMV_REQUIRE(ws && ws_bytes >= spmv_csr_slices_workspace_size(n_rows), "spmv_csr_to_slices: workspace too small");
    hipStream_t s = as_stream(stream);
    const int32_t ns = (int32_t)ceil_div(n_rows, SPMV_REM_SLICE);
    if (ns == 0) {
        SPMV_HIP(hipMemsetAsync(slice_ptr, 0, sizeof(int64_t), s));
        SPMV_HIP(hipStreamSynchronize(s));
        *h_padded = 0;
        return SPMV_OK;
    }
    SPMV_REQUIRE(row_ptr && slice_nd && slot_row, "spmv_csr_to_slices: null row_ptr, slice_nd or slot_row");
    WsCarver wc(ws, ws_bytes);
    int32_t *perm = wc.take<int32_t>((size_t)n_rows);
    int64_t *sz = wc.take<int64_t>((size_t)ns);
    int64_t *sws = wc.take<int64_t>(scan_ws_elems(ns));
    if (!wc.ok()) return fail(SPMV_ERR_INVALID_ARG, "spmv_csr_to_slices: workspace too small");
    rem_order_kernel<<<(unsigned)ceil_div(n_rows, SPMV_REM_WINDOW), SPMV_REM_WINDOW, 0, s>>>(row_ptr, n_rows,
                                                                                          slot_row, perm, slice_nd, sz);
    SPMV_CHECK_LAUNCH("slice order");
    spmv_status st = exclusive_scan<int64_t, int64_t>(sz, ns, slice_ptr, sws, s);
    if (st != SPMV_OK) return st;
    int64_t total = 0;
    SPMV_HIP(hipMemcpyAsync(&total, slice_ptr + ns, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    SPMV_HIP(hipStreamSynchronize(s));
    *h_padded = total;
    if (!bl_col) return SPMV_OK;                                   // sizes only
    if (bl_cap < total) return fail(SPMV_ERR_CAPACITY, "spmv_csr_to_slices: capacity < padded size");
    if (total == 0) return SPMV_OK;
    SPMV_REQUIRE(col_idx && val && bl_val, "spmv_csr_to_slices: null arrays");
#define SFILL_CASE(T)                                                                                                \
    window_fill_kernel<T><<<grid_for(total), 256, 0, s>>>(row_ptr, col_idx, (const T *)val, perm, n_rows,            \
                                                          SPMV_REM_SLICE, slice_ptr, ns, total, bl_col, (T *)bl_val)
    if (dt == SPMV_F64) SFILL_CASE(uint64_t);
    else if (dt == SPMV_F32 || dt == SPMV_I32) SFILL_CASE(uint32_t);
    else SFILL_CASE(uint16_t);
#undef SFILL_CASE
    SPMV_CHECK_LAUNCH("slice fill");
    SPMV_HIP(hipStreamSynchronize(s));
    return SPMV_OK;
}

size_t spmv_split_columns_workspace_size(int32_t n_rows, int64_t nnz)
{
    const size_t m = (size_t)(nnz > 0 ? nnz : 1);
    const size_t n = (size_t)(n_rows > 0 ? n_rows : 1);
    const size_t sc = scan_ws_elems((int64_t)std::max(m + 1, n + 1));
    return 5 * align_up(sizeof(int32_t) * m, 256) + align_up(sizeof(int32_t) * (m + 1), 256) +
           2 * align_up(sizeof(int32_t) * n, 256) + 2 * align_up(sizeof(int64_t) * (SPLIT_PARTS + 1), 256) +
           align_up(sizeof(int32_t) * sc, 256) + radix_ws_bytes((int64_t)m) + 2048;
}

spmv_status spmv_split_columns(int32_t n_rows, int32_t n_cols, int64_t nnz, const int32_t *row_ptr,
                               const int32_t *col_idx, const void *val, spmv_dtype dt, int32_t width,
                               int32_t *row_ptr_all, int32_t *dest_all, int32_t *slot_ptr, int32_t *col_out,
                               void *val_out, int64_t *h_bounds, int64_t *h_row_off, void *ws, size_t ws_bytes,
                               void *stream)
{
    SPMV_REQUIRE(n_rows >= 0 && n_cols >= 0 && nnz >= 0, "spmv_split_columns: negative size");
    if (nnz >= ((int64_t)1 << 31)) return fail(SPMV_ERR_UNSUPPORTED, "spmv_split_columns: nnz >= 2^31");
    SPMV_REQUIRE(valid_dtype(dt), "spmv_split_columns: bad dtype");
    if (width == 0) width = (int32_t)(ceil_div(ceil_div(n_cols > 0 ? n_cols : 1, SPLIT_PARTS), 64) * 64);
    SPMV_REQUIRE(width > 0 && (int64_t)width * SPLIT_PARTS >= n_cols,
                 "spmv_split_columns: width * SPMV_SPLIT_PARTS must cover the columns");
    SPMV_REQUIRE(row_ptr && row_ptr_all && slot_ptr && h_bounds && h_row_off, "spmv_split_columns: null pointer");
    SPMV_REQUIRE(nnz == 0 || (col_idx && val && col_out && val_out && dest_all), "spmv_split_columns: null arrays");
    SPMV_REQUIRE(ws && ws_bytes >= spmv_split_columns_workspace_size(n_rows, nnz),
                 "spmv_split_columns: workspace too small");
    hipStream_t s = as_stream(stream);
    WsCarver wc(ws, ws_bytes);
    const size_t m = (size_t)(nnz > 0 ? nnz : 1);
    const size_t nn = (size_t)(n_rows > 0 ? n_rows : 1);
    int32_t *rowid = wc.take<int32_t>(m);
    int32_t *rowid_s = wc.take<int32_t>(m);
    uint32_t *keys = wc.take<uint32_t>(m);
    int32_t *perm = wc.take<int32_t>(m);
    int32_t *head = wc.take<int32_t>(m);
    int32_t *qidx = wc.take<int32_t>(m + 1);
    uint32_t *mask = wc.take<uint32_t>(nn);
    int32_t *cnt = wc.take<int32_t>(nn);
    int64_t *bounds = wc.take<int64_t>(SPLIT_PARTS + 1);
    int64_t *row_off = wc.take<int64_t>(SPLIT_PARTS + 1);
    int32_t *scan_ws = wc.take<int32_t>(scan_ws_elems((int64_t)std::max(m + 1, nn + 1)));
    const size_t rws_bytes = radix_ws_bytes((int64_t)m);
    void *rws = wc.take<char>(rws_bytes);
    if (!wc.ok()) return fail(SPMV_ERR_INVALID_ARG, "spmv_split_columns: workspace too small");
    if (n_rows > 0) SPMV_HIP(hipMemsetAsync(mask, 0, sizeof(uint32_t) * n_rows, s));
    if (nnz > 0) {
        row_of_entries_kernel<<<grid_for(nnz), 256, 0, s>>>(row_ptr, n_rows, nnz, rowid);
        uint32_t *pkey = (uint32_t *)head;       // free until the head flags are written
        part_key_kernel<<<grid_for(nnz), 256, 0, s>>>(col_idx, nnz, width, pkey);
        SPMV_CHECK_LAUNCH("split keys");
        // stable: each part keeps the row-major order of its entries
        spmv_status st = radix_sort_pairs(keys, perm, nnz, bits_for(SPLIT_PARTS - 1), rws, rws_bytes, s, pkey);
        if (st != SPMV_OK) return st;
        if (dt == SPMV_F64)
            gather_split_kernel<uint64_t><<<grid_for(nnz), 256, 0, s>>>(perm, nnz, col_idx, (const uint64_t *)val, rowid,
                                                                         col_out, (uint64_t *)val_out, rowid_s);
        else if (dt == SPMV_F32)
            gather_split_kernel<uint32_t><<<grid_for(nnz), 256, 0, s>>>(perm, nnz, col_idx, (const uint32_t *)val, rowid,
                                                                         col_out, (uint32_t *)val_out, rowid_s);
        else
            gather_split_kernel<uint16_t><<<grid_for(nnz), 256, 0, s>>>(perm, nnz, col_idx, (const uint16_t *)val, rowid,
                                                                         col_out, (uint16_t *)val_out, rowid_s);
        SPMV_CHECK_LAUNCH("split gather");
        split_head_kernel<<<grid_for(nnz), 256, 0, s>>>(keys, rowid_s, nnz, head);
        SPMV_CHECK_LAUNCH("split heads");
    }
    spmv_status st = exclusive_scan<int32_t, int32_t>(head, nnz, qidx, scan_ws, s);
    if (st != SPMV_OK) return st;
    part_bounds_kernel<<<1, 64, 0, s>>>(keys, nnz, bounds);
    SPMV_CHECK_LAUNCH("split bounds");
    if (nnz > 0) {
        split_rows_kernel<<<grid_for(nnz), 256, 0, s>>>(keys, rowid_s, head, qidx, nnz, bounds, row_ptr_all, mask);
        SPMV_CHECK_LAUNCH("split rows");
    }
    split_terminators_kernel<<<1, 64, 0, s>>>(bounds, qidx, row_ptr_all, row_off);
    popcount_kernel<<<grid_for(n_rows), 256, 0, s>>>(mask, n_rows, cnt);
    SPMV_CHECK_LAUNCH("split slots");
    st = exclusive_scan<int32_t, int32_t>(cnt, n_rows, slot_ptr, scan_ws, s);
    if (st != SPMV_OK) return st;
    if (nnz > 0) {
        split_dest_kernel<<<grid_for(nnz), 256, 0, s>>>(keys, rowid_s, head, qidx, nnz, mask, slot_ptr, dest_all);
        SPMV_CHECK_LAUNCH("split dest");
    }
    SPMV_HIP(hipMemcpyAsync(h_bounds, bounds, sizeof(int64_t) * (SPLIT_PARTS + 1), hipMemcpyDeviceToHost, s));
    SPMV_HIP(hipMemcpyAsync(h_row_off, row_off, sizeof(int64_t) * (SPLIT_PARTS + 1), hipMemcpyDeviceToHost, s));
    SPMV_HIP(hipStreamSynchronize(s));
    return SPMV_OK;
}

size_t spmv_dia_workspace_size(int32_t n_rows, int32_t n_cols)
{
    const int64_t m = (int64_t)(n_rows > 0 ? n_rows : 1) + (n_cols > 0 ? n_cols : 1) - 1;
    const size_t nn = (size_t)(n_rows > 0 ? n_rows : 1);
    return align_up(sizeof(int32_t) * (size_t)m, 256) + align_up(sizeof(int32_t) * nn, 256) +
           align_up(sizeof(int32_t) * scan_ws_elems((int64_t)nn), 256) + 1024;
}

}  // extern "C"

namespace spmv {
// ---- upper triangle of a symmetric matrix: entries with col >= row

__global__ void upper_count_kernel(const int32_t *__restrict__ rp, int32_t n, const int32_t *__restrict__ col,
                                   int32_t *__restrict__ cnt)
{
    GRID_LOOP(i, (int64_t)n)
    {
        int32_t c = 0;
        for (int32_t e = rp[i]; e < rp[i + 1]; ++e) c += col[e] >= i;
        cnt[i] = c;
    }
}

template <typename T>
__global__ void upper_fill_kernel(const int32_t *__restrict__ rp, int32_t n, const int32_t *__restrict__ col,
                                  const T *__restrict__ val, const int32_t *__restrict__ up_rp,
                                  int32_t *__restrict__ up_col, T *__restrict__ up_val)
{
    GRID_LOOP(i, (int64_t)n)
    {
        int32_t p = up_rp[i];
        for (int32_t e = rp[i]; e < rp[i + 1]; ++e) {
            if (col[e] < i) continue;
            up_col[p] = col[e];
            up_val[p] = val[e];
            ++p;
        }
    }
}

static spmv_status dia_from_csr_impl(bool sym, int32_t n_rows, int32_t n_cols, int64_t nnz, const int32_t *row_ptr,
                                     const int32_t *col_idx, const void *val, spmv_dtype dt, int32_t max_diags,
                                     int32_t *h_offsets, int32_t *h_ndia, int64_t *h_rem_nnz, void *dia_val,
                                     int32_t *rem_row_ptr, int32_t *rem_col, void *rem_val, void *ws, size_t ws_bytes,
                                     void *stream)
{
    SPMV_REQUIRE(n_rows >= 0 && n_cols >= 0 && nnz >= 0, "spmv_dia[_sym]_from_csr: negative size");
    if (nnz >= ((int64_t)1 << 31)) return fail(SPMV_ERR_UNSUPPORTED, "spmv_dia[_sym]_from_csr: nnz >= 2^31");
    SPMV_REQUIRE(valid_dtype(dt), "spmv_dia[_sym]_from_csr: bad dtype");
    if (max_diags == 0) max_diags = SPMV_DIA_MAX;
    SPMV_REQUIRE(max_diags > 0 && max_diags <= SPMV_DIA_MAX, "spmv_dia[_sym]_from_csr: max_diags must be 0..SPMV_DIA_MAX");
    SPMV_REQUIRE(h_offsets && h_ndia && h_rem_nnz, "spmv_dia[_sym]_from_csr: null host output");
    SPMV_REQUIRE(n_rows == 0 || row_ptr, "spmv_dia[_sym]_from_csr: null row_ptr");
    SPMV_REQUIRE(nnz == 0 || (col_idx && val), "spmv_dia[_sym]_from_csr: null col_idx or val");
    SPMV_REQUIRE(ws && ws_bytes >= spmv_dia_workspace_size(n_rows, n_cols), "spmv_dia[_sym]_from_csr: workspace too small");
    hipStream_t s = as_stream(stream);
    const int64_t m = (int64_t)(n_rows > 0 ? n_rows : 1) + (n_cols > 0 ? n_cols : 1) - 1;
    const size_t nn = (size_t)(n_rows > 0 ? n_rows : 1);
    WsCarver wc(ws, ws_bytes);
    int32_t *hist = wc.take<int32_t>((size_t)m);           // later: offset -> stored diagonal index
    int32_t *cnt = wc.take<int32_t>(nn);
    int32_t *scan_ws = wc.take<int32_t>(scan_ws_elems((int64_t)nn));
    if (!wc.ok()) return fail(SPMV_ERR_INVALID_ARG, "spmv_dia[_sym]_from_csr: workspace too small");

    // entries per offset
    std::vector<int32_t> h_hist((size_t)m, 0);
    if (nnz > 0 && n_rows > 0) {
        SPMV_HIP(hipMemsetAsync(hist, 0, sizeof(int32_t) * (size_t)m, s));
        diag_hist_kernel<<<grid_for(n_rows), 256, 0, s>>>(row_ptr, n_rows, col_idx, hist);
        SPMV_CHECK_LAUNCH("dia histogram");
        SPMV_HIP(hipMemcpyAsync(h_hist.data(), hist, sizeof(int32_t) * (size_t)m, hipMemcpyDeviceToHost, s));
        SPMV_HIP(hipStreamSynchronize(s));
    }
    // a diagonal is stored densely when its dense span costs no more bytes
    // than its entries do in CRS (value + 4-byte index); the fullest first.
    // Symmetric: only offsets >= 0 are stored, each also serving its mirror,
    // so its entries are those of offset o and -o
    const int64_t sv = (int64_t)dtype_size(dt);
    std::vector<std::pair<int32_t, int64_t>> cand;            // (count, offset)
    for (int64_t t = 0; t < m; ++t) {
        const int64_t o = t - (n_rows - 1);
        if (sym && o < 0) continue;
        int64_t c = h_hist[(size_t)t];
        if (sym && o > 0) c += h_hist[(size_t)(n_rows - 1 - o)];
        if (c == 0) continue;
        const int64_t span = std::min<int64_t>(n_rows, (int64_t)n_cols - o) - std::max<int64_t>(0, -o);
        if (c * (sv + 4) >= span * sv) cand.push_back({(int32_t)c, o});
    }
    std::sort(cand.begin(), cand.end(), [](const std::pair<int32_t, int64_t> &a, const std::pair<int32_t, int64_t> &b) {
        return a.first != b.first ? a.first > b.first : a.second < b.second;
    });
    if ((int64_t)cand.size() > max_diags) cand.resize((size_t)max_diags);
    DiaOffsets D{};
    D.n = (int32_t)cand.size();
    int64_t on_dia = 0;
    for (int k = 0; k < D.n; ++k) {
        D.off[k] = (int32_t)cand[(size_t)k].second;
        on_dia += cand[(size_t)k].first;
    }
    std::sort(D.off, D.off + D.n);
    *h_ndia = D.n;
    for (int k = 0; k < D.n; ++k) h_offsets[k] = D.off[k];
    *h_rem_nnz = nnz - on_dia;
    if (!dia_val) return SPMV_OK;                            // sizes only

    SPMV_REQUIRE(rem_row_ptr && (*h_rem_nnz == 0 || (rem_col && rem_val)), "spmv_dia[_sym]_from_csr: null output");
    if (n_rows > 0) {
        dia_index_kernel<<<grid_for(m), 256, 0, s>>>(m, hist);
        dia_index_set_kernel<<<1, SPMV_DIA_MAX, 0, s>>>(n_rows, D, sym ? 1 : 0, hist);
        SPMV_CHECK_LAUNCH("dia index");
    }
    const int64_t ndv = (int64_t)D.n * n_rows;
#define DIA_CASE(DT, T)                                                                                          \
    if (dt == DT) {                                                                                              \
        if (ndv > 0) dia_zero_kernel<T><<<grid_for(ndv), 256, 0, s>>>(ndv, (T *)dia_val);                       \
        if (n_rows > 0)                                                                                          \
            dia_scatter_kernel<T><<<grid_for(n_rows), 256, 0, s>>>(row_ptr, n_rows, col_idx, (const T *)val,     \
                                                                   hist, (T *)dia_val, cnt);                    \
        SPMV_CHECK_LAUNCH("dia scatter");                                                                        \
        spmv_status st = exclusive_scan<int32_t, int32_t>(cnt, n_rows, rem_row_ptr, scan_ws, s);                \
        if (st != SPMV_OK) return st;                                                                            \
        if (*h_rem_nnz > 0)                                                                                      \
            dia_rem_kernel<T><<<grid_for(n_rows), 256, 0, s>>>(row_ptr, n_rows, col_idx, (const T *)val, hist,  \
                                                               rem_row_ptr, rem_col, (T *)rem_val);             \
        SPMV_CHECK_LAUNCH("dia remainder");                                                                      \
    }
    DIA_CASE(SPMV_F64, uint64_t)
    DIA_CASE(SPMV_F32, uint32_t)
    DIA_CASE(SPMV_BF16, uint16_t)
#undef DIA_CASE
    SPMV_HIP(hipStreamSynchronize(s));
    return SPMV_OK;
}

}  // namespace spmv

extern "C" {

spmv_status spmv_dia_from_csr(int32_t n_rows, int32_t n_cols, int64_t nnz, const int32_t *row_ptr,
                              const int32_t *col_idx, const void *val, spmv_dtype dt, int32_t max_diags,
                              int32_t *h_offsets, int32_t *h_ndia, int64_t *h_rem_nnz, void *dia_val,
                              int32_t *rem_row_ptr, int32_t *rem_col, void *rem_val, void *ws, size_t ws_bytes,
                              void *stream)
{
    return dia_from_csr_impl(false, n_rows, n_cols, nnz, row_ptr, col_idx, val, dt, max_diags, h_offsets, h_ndia,
                             h_rem_nnz, dia_val, rem_row_ptr, rem_col, rem_val, ws, ws_bytes, stream);
}

spmv_status spmv_dia_sym_from_csr(int32_t n, int64_t nnz, const int32_t *row_ptr, const int32_t *col_idx,
                                  const void *val, spmv_dtype dt, int32_t max_diags, int32_t *h_offsets,
                                  int32_t *h_ndia, int64_t *h_rem_nnz, void *dia_val, int32_t *rem_row_ptr,
                                  int32_t *rem_col, void *rem_val, void *ws, size_t ws_bytes, void *stream)
{
    return dia_from_csr_impl(true, n, n, nnz, row_ptr, col_idx, val, dt, max_diags, h_offsets, h_ndia, h_rem_nnz,
                             dia_val, rem_row_ptr, rem_col, rem_val, ws, ws_bytes, stream);
}

size_t spmv_csr_upper_workspace_size(int32_t n)
{
    const size_t nn = (size_t)(n > 0 ? n : 1);
    return align_up(sizeof(int32_t) * nn, 256) + align_up(sizeof(int32_t) * (nn + 1), 256) +
           align_up(sizeof(int32_t) * scan_ws_elems((int64_t)nn), 256) + 512;
}

spmv_status spmv_csr_upper_from_csr(int32_t n, int64_t nnz, const int32_t *row_ptr, const int32_t *col_idx,
                                    const void *val, spmv_dtype dt, int64_t *h_nnz_upper, int32_t *up_row_ptr,
                                    int32_t *up_col, void *up_val, void *ws, size_t ws_bytes, void *stream)
{
    SPMV_REQUIRE(n >= 0 && nnz >= 0, "spmv_csr_upper_from_csr: negative size");
    if (nnz >= ((int64_t)1 << 31)) return fail(SPMV_ERR_UNSUPPORTED, "spmv_csr_upper_from_csr: nnz >= 2^31");
    SPMV_REQUIRE(valid_payload_dtype(dt), "spmv_csr_upper_from_csr: bad dtype");
    SPMV_REQUIRE(h_nnz_upper, "spmv_csr_upper_from_csr: null h_nnz_upper");
    SPMV_REQUIRE(n == 0 || row_ptr, "spmv_csr_upper_from_csr: null row_ptr");
    SPMV_REQUIRE(nnz == 0 || (col_idx && val), "spmv_csr_upper_from_csr: null col_idx or val");
    SPMV_REQUIRE(ws && ws_bytes >= spmv_csr_upper_workspace_size(n), "spmv_csr_upper_from_csr: workspace too small");
    hipStream_t s = as_stream(stream);
    const size_t nn = (size_t)(n > 0 ? n : 1);
    WsCarver wc(ws, ws_bytes);
    int32_t *cnt = wc.take<int32_t>(nn);
    int32_t *rp = wc.take<int32_t>(nn + 1);
    int32_t *sws = wc.take<int32_t>(scan_ws_elems((int64_t)nn));
    if (!wc.ok()) return fail(SPMV_ERR_INVALID_ARG, "spmv_csr_upper_from_csr: workspace too small");
    int32_t total = 0;
    if (n > 0) {
        upper_count_kernel<<<grid_for(n), 256, 0, s>>>(row_ptr, n, col_idx, cnt);
        SPMV_CHECK_LAUNCH("upper count");
        spmv_status st = exclusive_scan<int32_t, int32_t>(cnt, n, rp, sws, s);
        if (st != SPMV_OK) return st;
        SPMV_HIP(hipMemcpyAsync(&total, rp + n, sizeof(int32_t), hipMemcpyDeviceToHost, s));
        SPMV_HIP(hipStreamSynchronize(s));
    }
    *h_nnz_upper = total;
    if (!up_row_ptr) return SPMV_OK;                          // size only
    SPMV_REQUIRE(total == 0 || (up_col && up_val), "spmv_csr_upper_from_csr: null output");
    if (n == 0) {
        SPMV_HIP(hipMemsetAsync(up_row_ptr, 0, sizeof(int32_t), s));
        SPMV_HIP(hipStreamSynchronize(s));
        return SPMV_OK;
    }
    SPMV_HIP(hipMemcpyAsync(up_row_ptr, rp, sizeof(int32_t) * ((size_t)n + 1), hipMemcpyDeviceToDevice, s));
    if (total > 0) {
#define UP_CASE(DT, T)                                                                                          \
        if (dt == DT)                                                                                           \
            upper_fill_kernel<T><<<grid_for(n), 256, 0, s>>>(row_ptr, n, col_idx, (const T *)val, rp, up_col,   \
                                                             (T *)up_val);
        UP_CASE(SPMV_F64, uint64_t)
        UP_CASE(SPMV_F32, uint32_t)
        UP_CASE(SPMV_BF16, uint16_t)
        UP_CASE(SPMV_I32, uint32_t)
#undef UP_CASE
        SPMV_CHECK_LAUNCH("upper fill");
    }
    SPMV_HIP(hipStreamSynchronize(s));
    return SPMV_OK;
}

size_t spmv_split_rows_workspace_size(void) { return 2 * align_up(sizeof(int64_t) * (SPLIT_PARTS + 1), 256); }

spmv_status spmv_split_rows(int32_t n_rows, int64_t nnz, const int32_t *row_ptr, int32_t *row_ptr_parts,
                            int64_t *h_bounds, int64_t *h_entry_bounds, void *ws, size_t ws_bytes, void *stream)
{
    SPMV_REQUIRE(n_rows >= 0 && nnz >= 0, "spmv_split_rows: negative size");
    if (nnz >= ((int64_t)1 << 31)) return fail(SPMV_ERR_UNSUPPORTED, "spmv_split_rows: nnz >= 2^31");
    SPMV_REQUIRE(row_ptr && row_ptr_parts && h_bounds && h_entry_bounds, "spmv_split_rows: null pointer");
    SPMV_REQUIRE(ws && ws_bytes >= spmv_split_rows_workspace_size(), "spmv_split_rows: workspace too small");
    hipStream_t s = as_stream(stream);
    WsCarver wc(ws, ws_bytes);
    int64_t *bounds = wc.take<int64_t>(SPLIT_PARTS + 1);
    int64_t *entry_bounds = wc.take<int64_t>(SPLIT_PARTS + 1);
    row_bounds_kernel<<<1, 64, 0, s>>>(row_ptr, n_rows, nnz, bounds, entry_bounds);
    row_split_ptr_kernel<<<grid_for((int64_t)n_rows + SPLIT_PARTS), 256, 0, s>>>(row_ptr, n_rows, bounds,
                                                                                 row_ptr_parts);
    SPMV_CHECK_LAUNCH("spmv_split_rows");
    SPMV_HIP(hipMemcpyAsync(h_bounds, bounds, sizeof(int64_t) * (SPLIT_PARTS + 1), hipMemcpyDeviceToHost, s));
    SPMV_HIP(hipMemcpyAsync(h_entry_bounds, entry_bounds, sizeof(int64_t) * (SPLIT_PARTS + 1), hipMemcpyDeviceToHost,
                            s));
    SPMV_HIP(hipStreamSynchronize(s));
    if (h_entry_bounds[SPLIT_PARTS] != nnz)
        return fail(SPMV_ERR_BAD_FORMAT, "spmv_split_rows: row_ptr[n_rows] != nnz");
    return SPMV_OK;
}

size_t spmv_transpose_workspace_size(int32_t n_rows, int32_t n_cols, int64_t nnz)
{
    (void)n_rows;
    (void)n_cols;
    size_t n = (size_t)(nnz > 0 ? nnz : 1);
    return align_up(sizeof(uint32_t) * n, 256) + radix_ws_bytes((int64_t)n) + 512;
}

spmv_status spmv_transpose_csr(int32_t n_rows, int32_t n_cols, int64_t nnz, const int32_t *row_ptr,
                               const int32_t *col_idx, int32_t *rowT_ptr, int32_t *colT, int32_t *tmap, void *ws,
                               size_t ws_bytes, void *stream)
{
    SPMV_REQUIRE(n_rows >= 0 && n_cols >= 0 && nnz >= 0, "spmv_transpose_csr: negative size");
    if (nnz >= ((int64_t)1 << 31)) return fail(SPMV_ERR_UNSUPPORTED, "spmv_transpose_csr: nnz >= 2^31");
    SPMV_REQUIRE(rowT_ptr && row_ptr, "spmv_transpose_csr: null pointer");
    SPMV_REQUIRE(nnz == 0 || (col_idx && colT && tmap), "spmv_transpose_csr: null arrays");
    SPMV_REQUIRE(ws && ws_bytes >= spmv_transpose_workspace_size(n_rows, n_cols, nnz),
                 "spmv_transpose_csr: workspace too small");
    hipStream_t s = as_stream(stream);
    WsCarver wc(ws, ws_bytes);
    uint32_t *keys = wc.take<uint32_t>((size_t)(nnz > 0 ? nnz : 1));
    size_t rws_bytes = radix_ws_bytes(nnz);
    void *rws = wc.take<char>(rws_bytes);
    if (nnz == 0) {
        SPMV_HIP(hipMemsetAsync(rowT_ptr, 0, sizeof(int32_t) * ((size_t)n_cols + 1), s));
        SPMV_HIP(hipStreamSynchronize(s));
        return SPMV_OK;
    }
    // entries are in row order, so a stable sort by column lists each column's
    // entries by ascending row
    spmv_status st = radix_sort_pairs(keys, tmap, nnz, bits_for(n_cols > 0 ? n_cols - 1 : 0), rws, rws_bytes, s,
                                      (const uint32_t *)col_idx);
    if (st != SPMV_OK) return st;
    transpose_cols_kernel<<<grid_for(nnz), 256, 0, s>>>(row_ptr, n_rows, tmap, nnz, colT);
    ptr_from_sorted_kernel<uint32_t><<<grid_for((int64_t)n_cols + 1), 256, 0, s>>>(keys, nnz, n_cols, rowT_ptr);
    SPMV_CHECK_LAUNCH("transpose structure");
    SPMV_HIP(hipStreamSynchronize(s));
    return SPMV_OK;
}

spmv_status spmv_convert_values(int64_t n, const void *in, spmv_dtype in_dt, void *out, spmv_dtype out_dt, void *stream)
{
    SPMV_REQUIRE(n >= 0, "spmv_convert_values: n < 0");
    SPMV_REQUIRE(valid_dtype(in_dt) && valid_dtype(out_dt), "spmv_convert_values: bad dtype");
    if (n == 0) return SPMV_OK;
    SPMV_REQUIRE(in && out, "spmv_convert_values: null pointer");
    convert_kernel<<<grid_for(n), 256, 0, as_stream(stream)>>>(n, in, (int)in_dt, out, (int)out_dt);
    SPMV_CHECK_LAUNCH("spmv_convert_values");
    return SPMV_OK;
}

spmv_status spmv_permute_vec(int32_t n, const int32_t *perm, const void *in, void *out, spmv_dtype dt, int inverse,
                             void *stream)
{
    SPMV_REQUIRE(n >= 0, "spmv_permute_vec: n < 0");
    SPMV_REQUIRE(valid_vec_dtype(dt) || dt == SPMV_I32, "spmv_permute_vec: dtype must be F64, F32 or I32");
    if (n == 0) return SPMV_OK;
    SPMV_REQUIRE(perm && in && out && in != out, "spmv_permute_vec: null or aliased pointer");
    hipStream_t s = as_stream(stream);
    if (dt == SPMV_F64)
        permute_kernel<uint64_t><<<grid_for(n), 256, 0, s>>>(n, perm, (const uint64_t *)in, (uint64_t *)out, inverse);
    else
        permute_kernel<uint32_t><<<grid_for(n), 256, 0, s>>>(n, perm, (const uint32_t *)in, (uint32_t *)out, inverse);
    SPMV_CHECK_LAUNCH("spmv_permute_vec");
    return SPMV_OK;
}

spmv_status spmv_gather_values(int64_t n, const int32_t *map, const void *in, void *out, spmv_dtype dt, void *stream)
{
    SPMV_REQUIRE(n >= 0, "spmv_gather_values: n < 0");
    SPMV_REQUIRE(valid_payload_dtype(dt), "spmv_gather_values: bad dtype");
    if (n == 0) return SPMV_OK;
    SPMV_REQUIRE(map && in && out && in != out, "spmv_gather_values: null or aliased pointer");
    hipStream_t s = as_stream(stream);
    if (dt == SPMV_F64)
        gather_kernel<uint64_t><<<grid_for(n), 256, 0, s>>>(n, map, (const uint64_t *)in, (uint64_t *)out);
    else if (dt == SPMV_F32 || dt == SPMV_I32)
        gather_kernel<uint32_t><<<grid_for(n), 256, 0, s>>>(n, map, (const uint32_t *)in, (uint32_t *)out);
    else
        gather_kernel<uint16_t><<<grid_for(n), 256, 0, s>>>(n, map, (const uint16_t *)in, (uint16_t *)out);
    SPMV_CHECK_LAUNCH("spmv_gather_values");
    return SPMV_OK;
}

}  // extern "C"
