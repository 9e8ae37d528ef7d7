// Prefix sums and the stable radix sort that the conversions share.
#pragma once

#include <algorithm>

#include "common.hpp"

namespace spmv {

#define GRID_LOOP(i, n) \
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n); i += (int64_t)gridDim.x * blockDim.x)

static inline unsigned grid_for(int64_t n)
{
    int64_t g = ceil_div(n, 256);
    if (g > 65536) g = 65536;
    return (unsigned)(g < 1 ? 1 : g);
}

// ======================================================================= scan
// Exclusive prefix sum out[i] = sum_{j<i} in[j], out[n] = total.  Three
// phases: tile sums, (recursive) scan of the tile sums, tile scans.

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;

template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, T *wave_tot, T *total)
{
    const int lane = lane_id(), w = (int)threadIdx.x / WAVE;
    T inc = v;
    for (int off = 1; off < WAVE; off <<= 1) {
        T o = __shfl_up(inc, off, WAVE);
        if (lane >= off) inc += o;
    }
    if (lane == WAVE - 1) wave_tot[w] = inc;
    __syncthreads();
    T wbase = 0, all = 0;
    for (int i = 0; i < SCAN_THREADS / WAVE; ++i) {
        if (i < w) wbase += wave_tot[i];
        all += wave_tot[i];
    }
    if (total) *total = all;
    __syncthreads();
    return wbase + inc - v;
}

template <typename TI, typename TO>
__global__ __launch_bounds__(SCAN_THREADS) void scan_tile_sums(const TI *__restrict__ in, int64_t n,
                                                               TO *__restrict__ sums)
{
    __shared__ TO wt[SCAN_THREADS / WAVE];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    TO s = 0;
    for (int j = 0; j < SCAN_ITEMS; ++j) {
        int64_t i = base + (int64_t)j * SCAN_THREADS + threadIdx.x;
        if (i < n) s += (TO)in[i];
    }
    TO tot;
    block_exclusive_scan<TO>(s, wt, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

template <typename TI, typename TO>
__global__ __launch_bounds__(SCAN_THREADS) void scan_tiles(const TI *__restrict__ in, int64_t n,
                                                           const TO *__restrict__ tile_base, TO *__restrict__ out,
                                                           bool write_total)
{
    __shared__ TO wt[SCAN_THREADS / WAVE];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    TO v[SCAN_ITEMS];
    TO s = 0;
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) {
        int64_t i = base + j;
        v[j] = i < n ? (TO)in[i] : (TO)0;
        s += v[j];
    }
    TO tot;
    TO run = block_exclusive_scan<TO>(s, wt, &tot) + (tile_base ? tile_base[blockIdx.x] : (TO)0);
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) {
        int64_t i = base + j;
        if (i < n) out[i] = run;
        run += v[j];
    }
    if (write_total && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
        out[n] = (tile_base ? tile_base[blockIdx.x] : (TO)0) + tot;
}

static inline size_t scan_ws_elems(int64_t n)
{
    size_t total = 0;
    int64_t tiles = ceil_div(n, SCAN_TILE);
    while (tiles > 1) {
        total += (size_t)tiles + 1;
        tiles = ceil_div(tiles, SCAN_TILE);
    }
    return total + 1;
}

// out has n+1 entries; ws holds scan_ws_elems(n) TO values.
template <typename TI, typename TO>
static spmv_status exclusive_scan(const TI *in, int64_t n, TO *out, TO *ws, hipStream_t s)
{
    if (n == 0) {
        SPMV_HIP(hipMemsetAsync(out, 0, sizeof(TO), s));
        return SPMV_OK;
    }
    int64_t tiles = ceil_div(n, SCAN_TILE);
    if (tiles == 1) {
        scan_tiles<TI, TO><<<1, SCAN_THREADS, 0, s>>>(in, n, (const TO *)nullptr, out, true);
        SPMV_CHECK_LAUNCH("scan");
        return SPMV_OK;
    }
    TO *sums = ws;                    // tiles + 1 entries
    TO *rest = ws + tiles + 1;
    scan_tile_sums<TI, TO><<<(unsigned)tiles, SCAN_THREADS, 0, s>>>(in, n, sums);
    SPMV_CHECK_LAUNCH("scan tile sums");
    spmv_status st = exclusive_scan<TO, TO>(sums, tiles, sums, rest, s);   // in place is safe per tile
    if (st != SPMV_OK) return st;
    scan_tiles<TI, TO><<<(unsigned)tiles, SCAN_THREADS, 0, s>>>(in, n, sums, out, true);
    SPMV_CHECK_LAUNCH("scan tiles");
    return SPMV_OK;
}

// ================================================================ radix sort
// Stable LSD radix sort of uint32 keys with one or two payload arrays, 8 bits
// per pass.  A pass reads and writes every item once, so its bound is the
// copy rate; three kernels: per-tile digit counts, their scan (digit-major),
// and the scatter.  The scatter orders its tile by digit in LDS first, so
// that a digit's items leave as one run (8192 items / 256 digits: 128 bytes
// of 4-byte items on average) instead of one 4-byte store per line, and it
// issues all of a lane's loads before the first rank is taken.  Tiles are
// dealt to the XCDs in contiguous ranges: neighbouring tiles append to the
// same lines of every digit's run.
constexpr int RS_THREADS = 512;
constexpr int RS_WAVES = RS_THREADS / WAVE;
constexpr int RS_ITEMS = 16;                       // per lane
constexpr int RS_TILE = RS_THREADS * RS_ITEMS;     // 8192 items per tile
constexpr int RS_BINS = 256;

struct NoPayload {};

template <typename V>
struct PayloadSize { static constexpr size_t value = sizeof(V); };
template <>
struct PayloadSize<NoPayload> { static constexpr size_t value = 0; };

static __global__ __launch_bounds__(RS_THREADS) void radix_hist_kernel(const uint32_t *__restrict__ keys, int64_t n,
                                                                int shift, int32_t *__restrict__ counts,
                                                                int64_t ntiles)
{
    __shared__ int32_t h[RS_BINS];
    for (int i = threadIdx.x; i < RS_BINS; i += RS_THREADS) h[i] = 0;
    __syncthreads();
    const int64_t tile = xcd_remap(blockIdx.x, ntiles);
    const int64_t base = tile * RS_TILE;
    uint32_t k[RS_ITEMS];
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const int64_t i = base + (int64_t)j * RS_THREADS + threadIdx.x;
        k[j] = i < n ? keys[i] : 0u;
    }
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const int64_t i = base + (int64_t)j * RS_THREADS + threadIdx.x;
        if (i < n) atomicAdd(&h[((k[j] >> shift) & (RS_BINS - 1))], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < RS_BINS; i += RS_THREADS) counts[(int64_t)i * ntiles + tile] = h[i];
}

// offs[d * ntiles + tile]: where tile's items of digit d start.  A first
// payload of nullptr stands for the item's index.
template <typename V1, typename V2>
__global__ __launch_bounds__(RS_THREADS) void radix_scatter_kernel(const uint32_t *__restrict__ kin,
                                                                   const V1 *__restrict__ vin,
                                                                   const V2 *__restrict__ win, int64_t n, int shift,
                                                                   const int32_t *__restrict__ offs, int64_t ntiles,
                                                                   uint32_t *__restrict__ kout,
                                                                   V1 *__restrict__ vout, V2 *__restrict__ wout)
{
    constexpr bool TWO = PayloadSize<V2>::value != 0;
    constexpr size_t ITEM = PayloadSize<V1>::value > PayloadSize<V2>::value ? PayloadSize<V1>::value
                                                                              : PayloadSize<V2>::value;
    constexpr size_t SLOT = ITEM > sizeof(uint32_t) ? ITEM : sizeof(uint32_t);
    __shared__ double buf[RS_TILE * SLOT / sizeof(double)];
    __shared__ int32_t cnt[RS_WAVES][RS_BINS];
    __shared__ int32_t gofs[RS_BINS];
    __shared__ int32_t wtot[RS_BINS / WAVE];
    const int t = (int)threadIdx.x, w = t / WAVE, lane = lane_id();
    const int64_t tile = xcd_remap(blockIdx.x, ntiles);
    const int64_t base = tile * RS_TILE;
    const int32_t n_in = n - base < RS_TILE ? (int32_t)(n - base) : RS_TILE;
    const int32_t first = t < RS_BINS ? offs[(int64_t)t * ntiles + tile] : 0;
    // wave w owns items [1024 w, 1024 (w + 1)) of the tile, in rounds of 64 in order
    const int32_t lw = w * WAVE * RS_ITEMS + lane;
    uint32_t k[RS_ITEMS];
    V1 v[RS_ITEMS];
    V2 x[RS_ITEMS];
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const int32_t i = lw + j * WAVE;
        k[j] = i < n_in ? kin[base + i] : 0u;
    }
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const int32_t i = lw + j * WAVE;
        if (vin) v[j] = i < n_in ? vin[base + i] : V1(0);
        else v[j] = (V1)(base + i);
        if constexpr (TWO) x[j] = i < n_in ? win[base + i] : V2(0);
    }
    for (int i = t; i < RS_WAVES * RS_BINS; i += RS_THREADS) (&cnt[0][0])[i] = 0;
    __syncthreads();
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (WAVE - lane));
    int32_t rank[RS_ITEMS];
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const bool in = lw + j * WAVE < n_in;
        const uint32_t dg = ((k[j] >> shift) & (RS_BINS - 1));
        uint64_t peers = __ballot(in);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t m = __ballot((dg >> b) & 1u);
            peers &= ((dg >> b) & 1u) ? m : ~m;
        }
        const int before = __popcll(peers & lt_mask);
        const int32_t start = cnt[w][dg];
        rank[j] = start + before;
        // the first lane of each digit group advances the wave's counter
        if (in && before == 0) cnt[w][dg] = start + __popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // per digit: exclusive prefix over the waves (tile order = wave order),
    // then over the digits
    int32_t run = 0, inc = 0;
    if (t < RS_BINS) {
#pragma unroll
        for (int q = 0; q < RS_WAVES; ++q) {
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
    if (t < RS_BINS) {
        int32_t ds = inc - run;
        for (int q = 0; q < w; ++q) ds += wtot[q];
#pragma unroll
        for (int q = 0; q < RS_WAVES; ++q) cnt[q][t] += ds;
        gofs[t] = first - ds;
    }
    __syncthreads();
    // through LDS into digit order: keys, then each payload
    uint32_t *kb = reinterpret_cast<uint32_t *>(buf);
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        rank[j] += cnt[w][((k[j] >> shift) & (RS_BINS - 1))];
        if (lw + j * WAVE < n_in) kb[rank[j]] = k[j];
    }
    __syncthreads();
    int32_t pos[RS_ITEMS];
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const int32_t i = j * RS_THREADS + t;
        if (i < n_in) {
            const uint32_t key = kb[i];
            pos[j] = gofs[((key >> shift) & (RS_BINS - 1))] + i;
            kout[pos[j]] = key;
        }
    }
    __syncthreads();
    V1 *vb = reinterpret_cast<V1 *>(buf);
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j)
        if (lw + j * WAVE < n_in) vb[rank[j]] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < RS_ITEMS; ++j) {
        const int32_t i = j * RS_THREADS + t;
        if (i < n_in) vout[pos[j]] = vb[i];
    }
    if constexpr (TWO) {
        __syncthreads();
        V2 *xb = reinterpret_cast<V2 *>(buf);
#pragma unroll
        for (int j = 0; j < RS_ITEMS; ++j)
            if (lw + j * WAVE < n_in) xb[rank[j]] = x[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < RS_ITEMS; ++j) {
            const int32_t i = j * RS_THREADS + t;
            if (i < n_in) wout[pos[j]] = xb[i];
        }
    }
}

static inline size_t radix_cells(int64_t n) { return (size_t)(n > 0 ? ceil_div(n, RS_TILE) : 1) * RS_BINS; }

// counts, offsets and scan scratch of a pass
static inline size_t radix_table_bytes(int64_t n)
{
    const size_t cells = radix_cells(n);
    return align_up(sizeof(int32_t) * cells, 256) + align_up(sizeof(int32_t) * (cells + 1), 256) +
           align_up(sizeof(int32_t) * scan_ws_elems((int64_t)cells), 256) + 256;
}

static inline size_t radix_ws_bytes(int64_t n)
{
    return radix_table_bytes(n) + 2 * align_up(sizeof(uint32_t) * (size_t)(n > 0 ? n : 1), 256) + 256;   // ping-pong
}

// Tables of a pass, carved out of radix_table_bytes(n).
struct RadixTables {
    int64_t ntiles;
    int32_t *counts, *offs, *sws;
    bool ok;
    RadixTables(int64_t n, void *ws, size_t ws_bytes) : ntiles(ceil_div(n, RS_TILE))
    {
        const size_t cells = radix_cells(n);
        WsCarver wc(ws, ws_bytes);
        counts = wc.take<int32_t>(cells);
        offs = wc.take<int32_t>(cells + 1);
        sws = wc.take<int32_t>(scan_ws_elems((int64_t)cells));
        ok = wc.ok();
    }
};

// One pass over the 8 bits from `shift`; `counted`: the tables already hold
// the tiles' digit counts.
template <typename V1, typename V2>
static spmv_status radix_pass(const uint32_t *kin, const V1 *vin, const V2 *win, int64_t n, int shift, uint32_t *kout,
                              V1 *vout, V2 *wout, const RadixTables &R, hipStream_t s, bool counted = false)
{
    if (!R.ok) return fail(SPMV_ERR_INVALID_ARG, "radix sort: workspace too small");
    if (!counted) {
        radix_hist_kernel<<<(unsigned)R.ntiles, RS_THREADS, 0, s>>>(kin, n, shift, R.counts, R.ntiles);
        SPMV_CHECK_LAUNCH("radix hist");
    }
    spmv_status st = exclusive_scan<int32_t, int32_t>(R.counts, (int64_t)radix_cells(n), R.offs, R.sws, s);
    if (st != SPMV_OK) return st;
    radix_scatter_kernel<V1, V2><<<(unsigned)R.ntiles, RS_THREADS, 0, s>>>(kin, vin, win, n, shift, R.offs, R.ntiles,
                                                                           kout, vout, wout);
    SPMV_CHECK_LAUNCH("radix scatter");
    return SPMV_OK;
}

static __global__ void radix_init_kernel(const uint32_t *__restrict__ src, int64_t n, uint32_t *__restrict__ keys,
                                  int32_t *__restrict__ vals)
{
    GRID_LOOP(i, n)
    {
        keys[i] = src[i];
        vals[i] = (int32_t)i;
    }
}

// Sorts by the low `bits` bits of the keys, stably; the result is left in
// (keys, vals), ws provides the ping-pong buffers.  src == nullptr: sorts
// (keys, vals) in place (an odd number of passes copies back at the end).
// Otherwise the keys come from src, which stays as it is and is none of the
// other arrays, and the values are the indices 0 .. n-1.
static inline spmv_status radix_sort_pairs(uint32_t *keys, int32_t *vals, int64_t n, int bits, void *ws, size_t ws_bytes,
                                    hipStream_t s, const uint32_t *src = nullptr)
{
    if (n <= 0) return SPMV_OK;
    const int passes = n > 1 && bits > 0 ? (bits + 7) / 8 : 0;
    if (passes == 0) {
        if (src) {
            radix_init_kernel<<<(unsigned)std::min<int64_t>(ceil_div(n, 256), 65536), 256, 0, s>>>(src, n, keys, vals);
            SPMV_CHECK_LAUNCH("radix init");
        }
        return SPMV_OK;
    }
    WsCarver wc(ws, ws_bytes);
    const size_t tb = radix_table_bytes(n);
    void *tws = wc.take<char>(tb);
    uint32_t *k2 = wc.take<uint32_t>((size_t)n);
    int32_t *v2 = wc.take<int32_t>((size_t)n);
    if (!wc.ok()) return fail(SPMV_ERR_INVALID_ARG, "radix sort: workspace too small");
    const RadixTables R(n, tws, tb);
    const uint32_t *ka = src ? src : keys;
    const int32_t *va = src ? nullptr : vals;
    for (int p = 0; p < passes; ++p) {
        // from src the last pass lands in (keys, vals); in place the first leaves them
        const bool home = src ? ((passes - 1 - p) & 1) == 0 : (p & 1) != 0;
        uint32_t *kb = home ? keys : k2;
        int32_t *vb = home ? vals : v2;
        spmv_status st = radix_pass<int32_t, NoPayload>(ka, va, nullptr, n, 8 * p, kb, vb, nullptr, R, s);
        if (st != SPMV_OK) return st;
        ka = kb;
        va = vb;
    }
    if (ka != keys) {
        SPMV_HIP(hipMemcpyAsync(keys, ka, sizeof(uint32_t) * n, hipMemcpyDeviceToDevice, s));
        SPMV_HIP(hipMemcpyAsync(vals, va, sizeof(int32_t) * n, hipMemcpyDeviceToDevice, s));
    }
    return SPMV_OK;
}

static inline int bits_for(int64_t maxval)
{
    int b = 0;
    while (b < 32 && ((int64_t)1 << b) <= maxval) ++b;
    return b;
}

// first index in sorted a[0..n) with a[idx] >= key
template <typename T, typename K>
__device__ __forceinline__ int64_t lower_bound_dev(const T *a, int64_t n, K key)
{
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if ((K)a[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

template <typename T>
__global__ void ptr_from_sorted_kernel(const T *__restrict__ sorted, int64_t n, int32_t nseg,
                                       int32_t *__restrict__ ptr)
{
    GRID_LOOP(r, (int64_t)nseg + 1) ptr[r] = (int32_t)lower_bound_dev(sorted, n, (int64_t)r);
}

static inline spmv_status read_flag(const int32_t *dev, int32_t *host, hipStream_t s)
{
    SPMV_HIP(hipMemcpyAsync(host, dev, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    SPMV_HIP(hipStreamSynchronize(s));
    return SPMV_OK;
}

}  // namespace spmv
