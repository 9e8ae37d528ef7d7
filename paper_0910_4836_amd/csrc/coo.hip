// COO -> CRS (paper Section 2, the CRS arrays): entries by (row, column),
// duplicates summed in input order.
//
// Two ways to the same result:
//   * buckets: the entries (row, column and value together) go through one to
//     three stable radix passes over the high bits of the row, which leaves
//     them in buckets of 2^s consecutive rows, about 1024 entries each; then
//     one workgroup per bucket sorts by (row, column) in LDS, adds up
//     duplicates and writes the bucket compactly, and a last pass closes the
//     gaps that duplicates left.  Every array is streamed once per pass; no
//     access goes by a random index.  Input that is already in bucket order
//     skips the radix passes.
//   * keys and indices: stable radix sorts by column and by row of (key,
//     index) pairs, then gathers of columns and values by index.  Twice the
//     passes, and three random gathers of 4-8 bytes, a 128-byte line each.
// 31.3 M shuffled triplets (5% duplicates, FP64 values, 2 M rows): 1.6 ms by
// buckets (radix passes 0.57, sorts 0.63, closing 0.14, check 0.07), 3.8 ms by
// indices; the bound, every triplet read and every entry written once, is
// 0.18 ms at the copy rate.
#include "common.hpp"
#include "sort.hpp"

namespace spmv {

// ---------------------------------------------------------------- by buckets

constexpr int CB_TARGET = 1024;       // entries wanted per bucket
constexpr int CB_SMALL_THREADS = 256;
constexpr int CB_ITEMS = 8;           // per lane: buckets of up to 2048 entries
constexpr int CB_MID_THREADS = 512;   // up to 4096: at 31 M entries the few thousand of these take
constexpr int CB_BIG_THREADS = 1024;  // 60 us less than in workgroups of 1024 lanes;
                                      // up to 8192: what the largest workgroup sorts
constexpr int CB_LIST_GRID = 2048;
constexpr int32_t CB_MAX = CB_BIG_THREADS * CB_ITEMS;   // entries of a bucket
constexpr int CB_MAX_ROW_BITS = 13;   // rows per bucket
constexpr int CB_DIGIT = 7;           // bits per pass in LDS (6 the same, 8 4% slower)
constexpr int CB_BINS = 1 << CB_DIGIT;

struct CooSplit {
    bool use;           // whether the buckets fit
    int row_bits;       // a bucket holds 2^row_bits rows
    int col_bits;
    int passes;         // radix passes over the bucket number
    int32_t buckets;
};

// About CB_TARGET entries per bucket (twice that where it saves a pass).
// Buckets of more than 2^13 rows (a matrix of mostly empty rows) would spend
// their time on the row pointer: such input, and a bucket of more entries
// than a workgroup sorts, goes by indices.  What was done by then is lost, so
// such a bucket is looked for early:
//   * more entries than all buckets hold are seen here;
//   * where one pass orders the entries, the check has counted every bucket by
//     the time that its result is waited for;
//   * up to COO_FINE buckets, the check sees whether some tile of unordered
//     entries holds more of a bucket than its part of a bucket that fits, and
//     the buckets are counted if so (coo_count_kernel);
//   * beyond that the kernels after the passes return at once.
// One row of 9 k entries more among rows of 15 (FP64, shuffled): 16 k rows 303 us
// without all this, 215 with; 50 k 375 and 284; 400 k 1194 and 1072.
static CooSplit coo_split(int32_t n_rows, int32_t n_cols, int64_t nnz)
{
    CooSplit c{};
    if (n_rows <= 0 || n_cols <= 0 || nnz <= 0) return c;
    const int rb = bits_for(n_rows - 1);
    int w = bits_for((nnz - 1) / CB_TARGET);
    if (w > 8 && w % 8 == 1) --w;
    if (w > rb) w = rb;
    if (w > 24) return c;
    c.row_bits = rb - w;
    c.col_bits = bits_for(n_cols - 1);
    c.passes = (w + 7) / 8;
    c.buckets = ((n_rows - 1) >> c.row_bits) + 1;
    c.use = c.row_bits <= CB_MAX_ROW_BITS && nnz <= (int64_t)c.buckets * CB_MAX;
    return c;
}

// flags[0]: an index is out of range; flags[1]: rows out of bucket order.
// Also the first radix pass's digit counts (skipped if counts is null), and
// their totals over the tiles (skipped if totals is null; flags[7] if one is
// more than a bucket may hold).  FINE: flags[5] if a
// tile out of bucket order holds more than `most` entries of one of COO_FINE
// buckets.
constexpr int COO_FINE = 2048;
template <bool FINE>
__global__ __launch_bounds__(RS_THREADS) void coo_check_kernel(const int32_t *__restrict__ row,
                                                               const int32_t *__restrict__ col, int64_t n,
                                                               int32_t n_rows, int32_t n_cols, int row_bits,
                                                               int32_t *__restrict__ counts, int64_t ntiles,
                                                               int32_t *__restrict__ totals, int32_t most,
                                                               int32_t *__restrict__ flags)
{
    __shared__ int32_t h[RS_BINS];
    __shared__ int32_t fine[FINE ? COO_FINE : 1];
    for (int i = threadIdx.x; i < RS_BINS; i += RS_THREADS) h[i] = 0;
    if (FINE)
        for (int i = threadIdx.x; i < COO_FINE; i += RS_THREADS) fine[i] = 0;
    __syncthreads();
    const int64_t tile = xcd_remap(blockIdx.x, ntiles);
    const int64_t base = tile * RS_TILE;
    int32_t r[RS_ITEMS], c[RS_ITEMS], before[RS_ITEMS];
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const int64_t i = base + (int64_t)j * RS_THREADS + threadIdx.x;
        const bool in = i < n;
        r[j] = in ? row[i] : 0;
        c[j] = in ? col[i] : 0;
        before[j] = in && i > 0 ? row[i - 1] : 0;
    }
    bool bad = false, mixed = false;
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const int64_t i = base + (int64_t)j * RS_THREADS + threadIdx.x;
        if (i < n) {
            bad |= r[j] < 0 || r[j] >= n_rows || c[j] < 0 || c[j] >= n_cols;
            mixed |= (before[j] >> row_bits) > (r[j] >> row_bits);
            if (counts) atomicAdd(&h[((uint32_t)r[j] >> row_bits) & (RS_BINS - 1)], 1);
        }
    }
    // plain stores of one value: an atomic per wavefront would queue at the
    // one line (362 us instead of 75 at 31 M shuffled triplets)
    bad = __syncthreads_or(bad);
    mixed = __syncthreads_or(mixed);
    if (threadIdx.x == 0 && bad) flags[0] = 1;
    if (threadIdx.x == 0 && mixed) flags[1] = 1;
    if (FINE && mixed) {                    // ordered entries are all in a few buckets
        bool crowded = false;
#pragma unroll
        for (int j = 0; j < RS_ITEMS; ++j)
            if (base + (int64_t)j * RS_THREADS + threadIdx.x < n)
                atomicAdd(&fine[((uint32_t)r[j] >> row_bits) & (COO_FINE - 1)], 1);
        __syncthreads();
        for (int i = threadIdx.x; i < COO_FINE; i += RS_THREADS) crowded |= fine[i] > most;
        crowded = __syncthreads_or(crowded);
        if (threadIdx.x == 0 && crowded) flags[5] = 1;
    }
    if (!counts) return;
    for (int i = threadIdx.x; i < RS_BINS; i += RS_THREADS) {
        counts[(int64_t)i * ntiles + tile] = h[i];
        // whoever adds last sees the whole bucket
        if (totals && h[i] && atomicAdd(totals + i, h[i]) + h[i] > CB_MAX) flags[7] = 1;
    }
}

// sizes[b] (zero before): entries of bucket b, of at most COO_FINE buckets; the
// largest goes to *largest.  Rows are in range.
__global__ __launch_bounds__(RS_THREADS) void coo_count_kernel(const int32_t *__restrict__ row, int64_t n, int row_bits,
                                                               int32_t *__restrict__ sizes,
                                                               int32_t *__restrict__ largest)
{
    __shared__ int32_t h[COO_FINE];
    for (int i = threadIdx.x; i < COO_FINE; i += RS_THREADS) h[i] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * RS_TILE;
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const int64_t i = base + (int64_t)j * RS_THREADS + threadIdx.x;
        if (i < n) atomicAdd(&h[((uint32_t)row[i] >> row_bits) & (COO_FINE - 1)], 1);
    }
    __syncthreads();
    int32_t most = 0;
    for (int i = threadIdx.x; i < COO_FINE; i += RS_THREADS)
        if (h[i]) most = max(most, atomicAdd(sizes + i, h[i]) + h[i]);
    for (int off = WAVE / 2; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off, WAVE));
    if (lane_id() == 0 && most > CB_MAX) atomicMax(largest, most);
}

// start[b]: first entry of bucket b, from the rows in bucket order; buckets
// too large for the small sort are listed in big (their number in n_big), and
// the largest size goes to n_big[1].
__global__ __launch_bounds__(256) void coo_bounds_kernel(const uint32_t *__restrict__ row, int64_t n, int row_bits,
                                                         int32_t buckets, int32_t *__restrict__ start,
                                                         int32_t *__restrict__ ucount, int32_t *__restrict__ big,
                                                         int32_t *__restrict__ n_big)
{
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (b > buckets) return;
    int64_t at[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int64_t key = (b + q) << row_bits;
        at[q] = b + q >= buckets ? n : lower_bound_dev(row, n, key);
    }
    start[b] = (int32_t)at[0];
    if (b == buckets) return;
    ucount[b] = 0;                      // stays so in a bucket that no kernel sorts
    const int32_t size = (int32_t)(at[1] - at[0]);
    if (size > CB_SMALL_THREADS * CB_ITEMS) {
        big[atomicAdd(n_big, 1)] = (int32_t)b;
        atomicMax(n_big + 1, size);
    }
}

// Sorts one bucket by (row, column) in LDS with a stable radix sort of
// (key, index in the bucket) pairs, sums duplicates in input order and writes
// the distinct entries to the front of the bucket's place in (col_out,
// val_out), their number to ucount and each row's first one, counted from the
// bucket's, to row_ptr.  K holds row and column bits together.
template <int TH, int ITEMS, typename K, typename T>
__device__ __forceinline__ void coo_sort_bucket(int32_t b, const uint32_t *__restrict__ row,
                                                const int32_t *__restrict__ col, const T *__restrict__ val,
                                                int32_t start, int32_t size, CooSplit C, int32_t n_rows,
                                                int32_t *__restrict__ col_out, T *__restrict__ val_out,
                                                int32_t *__restrict__ ucount, int32_t *__restrict__ row_ptr, K *kb,
                                                uint16_t *ib, int32_t (*cnt)[CB_BINS], int32_t *wtot)
{
    constexpr int WAVES = TH / WAVE;
    const int t = (int)threadIdx.x, w = t / WAVE, lane = lane_id();
    const int rounds = (size + TH - 1) / TH;              // <= ITEMS
    const int32_t lw = w * WAVE * rounds + lane;         // wave w owns `rounds` rounds of 64 in order
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (WAVE - lane));
    const K row0 = (K)b << C.row_bits;
    K k[ITEMS];
    int32_t id[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int32_t i = lw + j * WAVE;
        const bool in = j < rounds && i < size;
        const uint32_t r = in ? row[start + i] : 0u;
        const uint32_t c = in ? (uint32_t)col[start + i] : 0u;
        k[j] = in ? (((K)r - row0) << C.col_bits) | (K)c : (K)0;
        id[j] = i;
    }
    const int bits = C.row_bits + C.col_bits;
    const int passes = (bits + CB_DIGIT - 1) / CB_DIGIT;
    constexpr uint32_t mask = CB_BINS - 1;
    for (int p = 0; p < passes; ++p) {
        const int shift = p * CB_DIGIT;
        for (int i = t; i < WAVES * CB_BINS; i += TH) (&cnt[0][0])[i] = 0;
        __syncthreads();
        int32_t rank[ITEMS];
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            if (j < rounds) {
                const bool in = lw + j * WAVE < size;
                const uint32_t dg = (uint32_t)(k[j] >> shift) & mask;
                uint64_t peers = __ballot(in);
#pragma unroll
                for (int q = 0; q < CB_DIGIT; ++q) {
                    const uint64_t m = __ballot((dg >> q) & 1u);
                    peers &= ((dg >> q) & 1u) ? m : ~m;
                }
                const int before = __popcll(peers & lt_mask);
                const int32_t s0 = cnt[w][dg];
                rank[j] = s0 + before;
                if (in && before == 0) cnt[w][dg] = s0 + __popcll(peers);
                __builtin_amdgcn_wave_barrier();
            }
        }
        __syncthreads();
        int32_t run = 0, inc = 0;
        if (t < CB_BINS) {
#pragma unroll
            for (int q = 0; q < WAVES; ++q) {
                const int32_t c = cnt[q][t];
                cnt[q][t] = run;
                run += c;
            }
            inc = run;
            for (int off = 1; off < WAVE; off <<= 1) {
                const int32_t o = __shfl_up(inc, off, WAVE);
                if (lane >= off) inc += o;
            }
            if (lane == WAVE - 1) wtot[w] = inc;
        }
        __syncthreads();
        if (t < CB_BINS) {
            int32_t ds = inc - run;
            for (int q = 0; q < w; ++q) ds += wtot[q];
#pragma unroll
            for (int q = 0; q < WAVES; ++q) cnt[q][t] += ds;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            if (j < rounds && lw + j * WAVE < size) {
                const int32_t to = rank[j] + cnt[w][(uint32_t)(k[j] >> shift) & mask];
                kb[to] = k[j];
                ib[to] = (uint16_t)id[j];
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int32_t i = lw + j * WAVE;
            if (j < rounds && i < size) {
                k[j] = kb[i];
                id[j] = ib[i];
            }
        }
        __syncthreads();
    }
    if (passes == 0) {                                    // one row and one column
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int32_t i = lw + j * WAVE;
            if (j < rounds && i < size) {
                kb[i] = k[j];
                ib[i] = (uint16_t)i;
            }
        }
        __syncthreads();
    }
    // heads of the runs of equal keys, numbered in order
    int32_t u[ITEMS], heads = 0;
    uint32_t is_head = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int32_t i = lw + j * WAVE;
        const bool in = j < rounds && i < size;
        const bool head = in && (i == 0 || kb[i - 1] != k[j]);
        const uint64_t m = __ballot(head);
        u[j] = heads + __popcll(m & lt_mask);
        heads += __popcll(m);
        if (head) is_head |= 1u << j;
    }
    if (lane == 0) wtot[w] = heads;
    __syncthreads();
    int32_t base = 0, total = 0;
    for (int q = 0; q < WAVES; ++q) {
        if (q < w) base += wtot[q];
        total += wtot[q];
    }
    const K cmask = ((K)1 << C.col_bits) - 1;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        if (is_head >> j & 1u) {
            const int32_t i = lw + j * WAVE;
            T s = val[start + id[j]];
            for (int32_t q = i + 1; q < size && kb[q] == k[j]; ++q) s = s + val[start + ib[q]];
            col_out[start + base + u[j]] = (int32_t)(k[j] & cmask);
            val_out[start + base + u[j]] = s;
        }
    }
    __syncthreads();
    // ib[i]: number of the head at sorted place i
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        if (is_head >> j & 1u) ib[lw + j * WAVE] = (uint16_t)(base + u[j]);
    __syncthreads();
    const int64_t r0 = (int64_t)b << C.row_bits;
    const int32_t rows = n_rows - r0 < ((int64_t)1 << C.row_bits) ? (int32_t)(n_rows - r0) : 1 << C.row_bits;
    for (int32_t r = t; r < rows; r += TH) {
        const K key = (K)r << C.col_bits;
        int32_t lo = 0, hi = size;
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if (kb[mid] < key) lo = mid + 1;
            else hi = mid;
        }
        row_ptr[r0 + r] = lo < size ? ib[lo] : total;
    }
    if (t == 0) ucount[b] = total;
    __syncthreads();
}

// One workgroup per bucket (list == nullptr), or a fixed grid over the listed
// buckets; sorts those of more than `over` and at most TH * ITEMS entries.
// n_list[0]: buckets listed; nothing is done if the largest, n_list[1], fits
// no workgroup.
template <int TH, int ITEMS, typename K, typename T>
__global__ __launch_bounds__(TH) void coo_bucket_kernel(const uint32_t *__restrict__ row,
                                                        const int32_t *__restrict__ col, const T *__restrict__ val,
                                                        const int32_t *__restrict__ start, CooSplit C, int32_t n_rows,
                                                        const int32_t *__restrict__ list,
                                                        const int32_t *__restrict__ n_list,
                                                        int32_t *__restrict__ col_out, T *__restrict__ val_out,
                                                        int32_t *__restrict__ ucount, int32_t *__restrict__ row_ptr,
                                                        int32_t over)
{
    __shared__ K kb[TH * ITEMS];
    __shared__ uint16_t ib[TH * ITEMS];
    __shared__ int32_t cnt[TH / WAVE][CB_BINS];
    __shared__ int32_t wtot[TH / WAVE];
    if (n_list[1] > CB_MAX) return;
    const int32_t count = list ? n_list[0] : C.buckets;
    for (int32_t i = (int32_t)blockIdx.x; i < count; i += (int32_t)gridDim.x) {
        const int32_t b = list ? list[i] : (int32_t)xcd_remap(i, count);
        const int32_t s0 = start[b], size = start[b + 1] - s0;
        if (size > TH * ITEMS || size <= over) continue;
        coo_sort_bucket<TH, ITEMS, K, T>(b, row, col, val, s0, size, C, n_rows, col_out, val_out, ucount, row_ptr, kb,
                                         ib, cnt, wtot);
    }
}

// Closes the gaps: bucket b's entries move to ubase[b], its row pointers too.
template <typename T>
__global__ __launch_bounds__(256) void coo_close_kernel(const int32_t *__restrict__ start,
                                                        const int32_t *__restrict__ ubase, CooSplit C, int32_t n_rows,
                                                        const int32_t *__restrict__ col, const T *__restrict__ val,
                                                        int32_t *__restrict__ col_out, T *__restrict__ val_out,
                                                        int32_t *__restrict__ row_ptr, int32_t *__restrict__ total,
                                                        const int32_t *__restrict__ largest)
{
    if (*largest > CB_MAX) return;
    const int32_t b = (int32_t)xcd_remap(blockIdx.x, C.buckets);
    const int32_t from = start[b], to = ubase[b], size = ubase[b + 1] - to;
    const int t = (int)threadIdx.x;
    constexpr int U = 4;
    for (int32_t i0 = 0; i0 < size; i0 += U * 256) {
        int32_t c[U];
        T v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t i = i0 + u * 256 + t;
            if (i < size) {
                c[u] = col[from + i];
                v[u] = val[from + i];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t i = i0 + u * 256 + t;
            if (i < size) {
                col_out[to + i] = c[u];
                val_out[to + i] = v[u];
            }
        }
    }
    const int64_t r0 = (int64_t)b << C.row_bits;
    const int32_t rows = n_rows - r0 < ((int64_t)1 << C.row_bits) ? (int32_t)(n_rows - r0) : 1 << C.row_bits;
    for (int32_t r = t; r < rows; r += 256) row_ptr[r0 + r] += to;
    if (b == C.buckets - 1 && t == 0) {
        row_ptr[n_rows] = to + size;
        *total = to + size;
    }
}

struct CooArrays {
    uint32_t *row;
    int32_t *col;
    void *val;
};

static size_t coo_bucket_ws_bytes(const CooSplit &C, int64_t nnz)
{
    if (!C.use) return 0;
    const size_t n = (size_t)nnz, nb = (size_t)C.buckets;
    size_t b = 2 * align_up(sizeof(uint32_t) * n, 256);            // rows, twice
    b += align_up(sizeof(int32_t) * n, 256);                       // columns
    b += align_up(sizeof(uint64_t) * n, 256);                      // values
    b += radix_table_bytes(nnz);
    b += 4 * align_up(sizeof(int32_t) * (nb + 2), 256);             // starts, list, counts, bases
    b += align_up(sizeof(int32_t) * scan_ws_elems((int64_t)nb), 256);
    return b + 1024;
}

// flags[2]: number of large buckets, [3]: the largest, [4]: entries out.  The
// outputs (col_idx, val_out) serve as the second set of arrays of the passes.
template <typename T, typename B>
static spmv_status coo_by_buckets(const CooSplit &C, int32_t n_rows, int64_t nnz, const int32_t *row,
                                  const int32_t *col, const T *val, bool ordered, const RadixTables &R, int32_t *flags,
                                  int32_t *row_ptr, int32_t *col_idx, T *val_out, WsCarver &wc, hipStream_t s)
{
    const size_t n = (size_t)nnz;
    uint32_t *row_a = wc.take<uint32_t>(n), *row_b = wc.take<uint32_t>(n);
    int32_t *col_b = wc.take<int32_t>(n);
    T *val_b = (T *)wc.take<uint64_t>(n);
    int32_t *start = wc.take<int32_t>((size_t)C.buckets + 1), *big = wc.take<int32_t>((size_t)C.buckets);
    int32_t *ucount = wc.take<int32_t>((size_t)C.buckets), *ubase = wc.take<int32_t>((size_t)C.buckets + 1);
    int32_t *sws = wc.take<int32_t>(scan_ws_elems(C.buckets));
    if (!wc.ok()) return fail(SPMV_ERR_INVALID_ARG, "spmv_csr_from_coo: workspace too small");
    const uint32_t *rows = (const uint32_t *)row;
    const int32_t *cols = col;
    const T *vals = val;
    const int passes = ordered ? 0 : C.passes;
    for (int p = 0; p < passes; ++p) {
        const bool out = ((passes - 1 - p) & 1) == 0;               // the last pass lands in the output arrays
        uint32_t *rn = out ? row_a : row_b;
        int32_t *cn = out ? col_idx : col_b;
        T *vn = out ? val_out : val_b;
        spmv_status st = radix_pass<int32_t, B>(rows, cols, (const B *)vals, nnz, C.row_bits + 8 * p, rn, cn, (B *)vn, R,
                                                s, p == 0);
        if (st != SPMV_OK) return st;
        rows = rn;
        cols = cn;
        vals = vn;
    }
    coo_bounds_kernel<<<(unsigned)ceil_div((int64_t)C.buckets + 1, 256), 256, 0, s>>>(rows, nnz, C.row_bits, C.buckets,
                                                                                      start, ucount, big, flags + 2);
    SPMV_CHECK_LAUNCH("coo bounds");
    const unsigned grid = (unsigned)C.buckets, list_grid = std::min<unsigned>(grid, CB_LIST_GRID);
#define COO_SORT_CLASS(K, TH, GRID, LIST, OVER)                                                                        \
    coo_bucket_kernel<TH, CB_ITEMS, K, T><<<GRID, TH, 0, s>>>(rows, cols, vals, start, C, n_rows, LIST, flags + 2,     \
                                                              col_b, val_b, ucount, row_ptr, OVER);                    \
    SPMV_CHECK_LAUNCH("coo buckets")
#define COO_SORT(K)                                                                                                    \
    COO_SORT_CLASS(K, CB_SMALL_THREADS, grid, nullptr, -1);                                                            \
    COO_SORT_CLASS(K, CB_MID_THREADS, list_grid, big, -1);                                                             \
    COO_SORT_CLASS(K, CB_BIG_THREADS, list_grid, big, CB_MID_THREADS *CB_ITEMS)
    if (C.row_bits + C.col_bits <= 32) {
        COO_SORT(uint32_t);
    } else {
        COO_SORT(uint64_t);
    }
#undef COO_SORT
#undef COO_SORT_CLASS
    spmv_status st = exclusive_scan<int32_t, int32_t>(ucount, C.buckets, ubase, sws, s);
    if (st != SPMV_OK) return st;
    coo_close_kernel<T><<<grid, 256, 0, s>>>(start, ubase, C, n_rows, col_b, val_b, col_idx, val_out, row_ptr, flags + 4,
                                           flags + 3);
    SPMV_CHECK_LAUNCH("coo close");
    return SPMV_OK;
}

// ---------------------------------------------------------------- by indices

__global__ void gather_u32_kernel(const int32_t *__restrict__ src, const int32_t *__restrict__ idx,
                                  uint32_t *__restrict__ out, int64_t n)
{
    GRID_LOOP(i, n) out[i] = (uint32_t)src[idx[i]];
}

// sorted (row, col) pairs -> 1 where a new (row, col) starts
__global__ void head_flags_kernel(const uint32_t *__restrict__ rk, const int32_t *__restrict__ idx,
                                  const int32_t *__restrict__ col, int64_t n, int32_t *__restrict__ flag)
{
    GRID_LOOP(i, n)
    {
        int32_t f = 1;
        if (i > 0 && rk[i] == rk[i - 1] && col[idx[i]] == col[idx[i - 1]]) f = 0;
        flag[i] = f;
    }
}

// one thread per run of equal (row, col): sums the run's values in input order
template <typename T>
__global__ void compact_kernel(const uint32_t *__restrict__ rk, const int32_t *__restrict__ idx,
                               const int32_t *__restrict__ col, const T *__restrict__ val,
                               const int32_t *__restrict__ flag, const int32_t *__restrict__ pos, int64_t n,
                               int32_t *__restrict__ col_out, T *__restrict__ val_out, int32_t *__restrict__ row_u)
{
    GRID_LOOP(i, n)
    {
        if (!flag[i]) continue;
        const int32_t p = pos[i];
        T s = val[idx[i]];
        for (int64_t j = i + 1; j < n && !flag[j]; ++j) s = s + val[idx[j]];
        col_out[p] = col[idx[i]];
        val_out[p] = s;
        row_u[p] = (int32_t)rk[i];
    }
}

static size_t coo_index_ws_bytes(int64_t nnz)
{
    const size_t n = (size_t)nnz;
    size_t b = 4 * align_up(sizeof(uint32_t) * n, 256);  // keys, indices, head flags, unique rows
    b += align_up(sizeof(int32_t) * (n + 1), 256);       // positions
    b += align_up(sizeof(int32_t) * scan_ws_elems((int64_t)n), 256);
    return b + radix_ws_bytes(nnz) + 1024;
}

template <typename T>
static spmv_status coo_by_indices(int32_t n_rows, int32_t n_cols, int64_t nnz, const int32_t *row, const int32_t *col,
                                  const T *val, int32_t *row_ptr, int32_t *col_idx, T *val_out, int64_t *h_nnz_out,
                                  WsCarver &wc, hipStream_t s)
{
    uint32_t *keys = wc.take<uint32_t>((size_t)nnz);
    int32_t *idx = wc.take<int32_t>((size_t)nnz);
    int32_t *head = wc.take<int32_t>((size_t)nnz);
    int32_t *pos = wc.take<int32_t>((size_t)nnz + 1);
    int32_t *row_u = wc.take<int32_t>((size_t)nnz);
    int32_t *sws = wc.take<int32_t>(scan_ws_elems(nnz));
    const size_t rws_bytes = radix_ws_bytes(nnz);
    void *rws = wc.take<char>(rws_bytes);
    if (!wc.ok()) return fail(SPMV_ERR_INVALID_ARG, "spmv_csr_from_coo: workspace too small");
    // stable sort by column, then stably by row: order (row, col, input index);
    // the rows in column order go where the head flags come later
    spmv_status st = radix_sort_pairs(keys, idx, nnz, bits_for(n_cols - 1), rws, rws_bytes, s, (const uint32_t *)col);
    if (st != SPMV_OK) return st;
    gather_u32_kernel<<<grid_for(nnz), 256, 0, s>>>(row, idx, keys, nnz);
    SPMV_CHECK_LAUNCH("coo gather rows");
    st = radix_sort_pairs(keys, idx, nnz, bits_for(n_rows - 1), rws, rws_bytes, s);
    if (st != SPMV_OK) return st;
    head_flags_kernel<<<grid_for(nnz), 256, 0, s>>>(keys, idx, col, nnz, head);
    SPMV_CHECK_LAUNCH("coo heads");
    st = exclusive_scan<int32_t, int32_t>(head, nnz, pos, sws, s);
    if (st != SPMV_OK) return st;
    int32_t nout = 0;
    if (read_flag(pos + nnz, &nout, s) != SPMV_OK) return SPMV_ERR_HIP;
    compact_kernel<T><<<grid_for(nnz), 256, 0, s>>>(keys, idx, col, val, head, pos, nnz, col_idx, val_out, row_u);
    SPMV_CHECK_LAUNCH("coo compact");
    ptr_from_sorted_kernel<int32_t><<<grid_for((int64_t)n_rows + 1), 256, 0, s>>>(row_u, nout, n_rows, row_ptr);
    SPMV_CHECK_LAUNCH("coo row_ptr");
    SPMV_HIP(hipStreamSynchronize(s));
    *h_nnz_out = nout;
    return SPMV_OK;
}

constexpr int COO_TOTALS = 8;                        // the flags, then the buckets' sizes
constexpr int COO_FLAGS = COO_TOTALS + RS_BINS;

static size_t coo_ws_bytes(int32_t n_rows, int32_t n_cols, int64_t nnz)
{
    const int64_t n = nnz > 0 ? nnz : 1;
    return align_up(sizeof(int32_t) * COO_FLAGS, 256) +
           std::max(coo_bucket_ws_bytes(coo_split(n_rows, n_cols, n), n), coo_index_ws_bytes(n));
}

}  // namespace spmv

using namespace spmv;

extern "C" {

size_t spmv_csr_from_coo_workspace_size(int32_t n_rows, int32_t n_cols, int64_t nnz)
{
    return coo_ws_bytes(n_rows, n_cols, nnz);
}

spmv_status spmv_csr_from_coo(int32_t n_rows, int32_t n_cols, int64_t nnz, const int32_t *row, const int32_t *col,
                              const void *val, spmv_dtype dt, int32_t *row_ptr, int32_t *col_idx, void *val_out,
                              int64_t *h_nnz_out, void *ws, size_t ws_bytes, void *stream)
{
    SPMV_REQUIRE(n_rows >= 0 && n_cols >= 0 && nnz >= 0, "spmv_csr_from_coo: negative size");
    if (nnz >= ((int64_t)1 << 31)) return fail(SPMV_ERR_UNSUPPORTED, "spmv_csr_from_coo: nnz >= 2^31");
    SPMV_REQUIRE(dt == SPMV_F64 || dt == SPMV_F32, "spmv_csr_from_coo: dtype must be F64 or F32");
    SPMV_REQUIRE(row_ptr && h_nnz_out, "spmv_csr_from_coo: null row_ptr or h_nnz_out");
    SPMV_REQUIRE(nnz == 0 || (row && col && val && col_idx && val_out), "spmv_csr_from_coo: null pointer");
    SPMV_REQUIRE(ws && ws_bytes >= coo_ws_bytes(n_rows, n_cols, nnz), "spmv_csr_from_coo: workspace too small");
    hipStream_t s = as_stream(stream);
    if (nnz == 0) {
        SPMV_HIP(hipMemsetAsync(row_ptr, 0, sizeof(int32_t) * ((size_t)n_rows + 1), s));
        SPMV_HIP(hipStreamSynchronize(s));
        *h_nnz_out = 0;
        return SPMV_OK;
    }
    WsCarver wc(ws, ws_bytes);
    int32_t *flags = wc.take<int32_t>(COO_FLAGS);
    const WsCarver after_flags = wc;
    const CooSplit C = coo_split(n_rows, n_cols, nnz);
    const size_t tb = radix_table_bytes(nnz);
    const RadixTables R(nnz, wc.take<char>(tb), tb);
    int32_t h[COO_TOTALS] = {0};
    SPMV_HIP(hipMemsetAsync(flags, 0, sizeof(int32_t) * (C.passes == 1 ? COO_FLAGS : COO_TOTALS), s));
    int32_t *counts = C.use && C.passes > 0 ? R.counts : nullptr;
    int32_t *totals = C.passes == 1 ? flags + COO_TOTALS : nullptr;
    const unsigned tiles = (unsigned)R.ntiles;
    // a tile's part of a bucket of CB_MAX entries in random order, 32 to 128: half
    // the tiles hold more of it if it has more
    const int32_t most = (int32_t)((int64_t)CB_MAX * RS_TILE / nnz);
    const bool fine = C.use && C.passes > 1 && C.buckets <= COO_FINE;
    if (fine)
        coo_check_kernel<true><<<tiles, RS_THREADS, 0, s>>>(row, col, nnz, n_rows, n_cols, C.row_bits, counts, R.ntiles,
                                                            totals, most, flags);
    else
        coo_check_kernel<false><<<tiles, RS_THREADS, 0, s>>>(row, col, nnz, n_rows, n_cols, C.row_bits, counts,
                                                             R.ntiles, totals, 0, flags);
    SPMV_CHECK_LAUNCH("coo check");
    SPMV_HIP(hipMemcpyAsync(h, flags, sizeof(h), hipMemcpyDeviceToHost, s));
    SPMV_HIP(hipStreamSynchronize(s));
    if (h[0]) return fail(SPMV_ERR_BAD_FORMAT, "spmv_csr_from_coo: row or column index out of range");

    bool fits = C.use && h[7] == 0;
    if (fits && fine && h[1] && h[5]) {
        WsCarver tmp = wc;
        int32_t *sizes = tmp.take<int32_t>(COO_FINE);
        SPMV_HIP(hipMemsetAsync(sizes, 0, sizeof(int32_t) * COO_FINE, s));
        coo_count_kernel<<<tiles, RS_THREADS, 0, s>>>(row, nnz, C.row_bits, sizes, flags + 6);
        SPMV_CHECK_LAUNCH("coo count");
        SPMV_HIP(hipMemcpyAsync(h, flags, sizeof(h), hipMemcpyDeviceToHost, s));
        SPMV_HIP(hipStreamSynchronize(s));
        fits = h[6] <= CB_MAX;
    }
    if (fits) {
        const bool ordered = h[1] == 0;
        spmv_status st =
            dt == SPMV_F64
                ? coo_by_buckets<double, uint64_t>(C, n_rows, nnz, row, col, (const double *)val, ordered, R, flags,
                                                   row_ptr, col_idx, (double *)val_out, wc, s)
                : coo_by_buckets<float, uint32_t>(C, n_rows, nnz, row, col, (const float *)val, ordered, R, flags,
                                                  row_ptr, col_idx, (float *)val_out, wc, s);
        if (st != SPMV_OK) return st;
        SPMV_HIP(hipMemcpyAsync(h, flags, sizeof(h), hipMemcpyDeviceToHost, s));
        SPMV_HIP(hipStreamSynchronize(s));
        if (h[3] <= CB_MAX) {
            *h_nnz_out = h[4];
            return SPMV_OK;
        }
    }
    wc = after_flags;
    return dt == SPMV_F64 ? coo_by_indices<double>(n_rows, n_cols, nnz, row, col, (const double *)val, row_ptr, col_idx,
                                                   (double *)val_out, h_nnz_out, wc, s)
                          : coo_by_indices<float>(n_rows, n_cols, nnz, row, col, (const float *)val, row_ptr, col_idx,
                                                  (float *)val_out, h_nnz_out, wc, s);
}

}  // extern "C"
