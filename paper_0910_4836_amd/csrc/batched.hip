// Many independent SpMVs y_m = A_m x_m in one persistent launch.
//
// Every matrix is in blocked-JDS storage (its own slice height C_m) inside
// shared arrays.  The host cuts all matrices into tiles of R consecutive
// permuted rows and writes a tile table: matrices largest first, each
// matrix's tiles together and in row order.  A grid sized to the GPU walks
// the table: each XCD takes one contiguous eighth of it and its wavefronts
// step through that range with a fixed stride (the staged form below: its
// workgroups, eight tiles at a time).  No atomics, no queue to
// reset, so the result does not depend on timing and the launch can be
// captured in a HIP graph and replayed.  This is the paper's
// static-versus-dynamic scheduling question (Section 5) answered for a GPU:
// static assignment, as the paper found best, with locality (one matrix's x
// per L2 at a time) taking the place of first-touch page placement.
#include <algorithm>
#include <numeric>
#include <vector>

#include "common.hpp"

namespace spmv {

struct BTile {
    int64_t base;      // bl_col/bl_val offset of the tile's first row, diagonal 0
    int64_t row_base;  // matrix offset into y and perm
    int64_t col_base;  // matrix offset into x
    int32_t r0;        // first local (permuted) row of the tile
    int32_t nrows;     // valid rows (<= R)
    int32_t C;         // slice height: stride between diagonals
    int32_t nd;        // diagonals of the tile's slice
    int32_t rlog;      // R = 1 << rlog rows per wavefront
    int32_t pad;
};
static_assert(sizeof(BTile) == SPMV_BATCHED_PLAN_WORDS * sizeof(int32_t), "tile record size");

constexpr int B_THREADS = 256;
constexpr int B_WAVES = B_THREADS / WAVE;

template <int U, bool WIDE>
__device__ __forceinline__ typename Acc<WIDE>::T batched_lane_sum(const BTile &T, const int32_t *__restrict__ col,
                                                                  const float *__restrict__ val,
                                                                  const float *__restrict__ x, int rl, int kk, int G,
                                                                  bool r_ok)
{
    typename Acc<WIDE>::T s = 0;
    for (int32_t base = 0; base < T.nd; base += G * U) {
        int32_t c[U];
        float v[U];
        bool act[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t dd = base + kk + u * G;
            act[u] = false;
            if (r_ok && dd < T.nd) {
                const int64_t e = T.base + (int64_t)dd * T.C + rl;
                c[u] = ld_stream(col + e);
                v[u] = ld_stream(val + e);
                act[u] = c[u] >= 0;
            }
        }
        float xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (act[u]) xv[u] = x[T.col_base + c[u]];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (act[u]) s = Acc<WIDE>::mac(s, v[u], xv[u]);
    }
    return s;
}

template <int U>
__device__ __forceinline__ void batched_tile(const BTile &T, const int32_t *__restrict__ perm,
                                             const int32_t *__restrict__ col, const float *__restrict__ val,
                                             const float *__restrict__ x, float *__restrict__ y)
{
    const int lane = lane_id();
    const int R = 1 << T.rlog, G = WAVE >> T.rlog;
    const int rl = lane & (R - 1), kk = lane >> T.rlog;
    const bool r_ok = rl < T.nrows;
    double td;
    if (T.nd > SPMV_WIDE_ROW_NNZ) {
        double s = batched_lane_sum<U, true>(T, col, val, x, rl, kk, G, r_ok);
        for (int off = 32; off >= R; off >>= 1) s += __shfl_xor(s, off, WAVE);
        td = s;
    } else {
        float s = batched_lane_sum<U, false>(T, col, val, x, rl, kk, G, r_ok);
        for (int off = 32; off >= R; off >>= 1) s += __shfl_xor(s, off, WAVE);
        td = (double)s;
    }
    if (r_ok && kk == 0) {
        const int64_t pr = T.row_base + T.r0 + rl;
        y[T.row_base + perm[pr]] = (float)td;
    }
}

template <int U>
__global__ __launch_bounds__(B_THREADS) void batched_kernel(int64_t n_tiles, const BTile *__restrict__ tiles,
                                                            const int32_t *__restrict__ perm,
                                                            const int32_t *__restrict__ col,
                                                            const float *__restrict__ val,
                                                            const float *__restrict__ x, float *__restrict__ y)
{
    // Workgroups are dealt to the 8 XCDs round-robin (the host launches a
    // multiple of 8).  Each XCD owns one contiguous eighth of the tile table, so
    // its L2 holds the x of the one or two matrices it is working on; inside
    // that range its wavefronts take tiles with a fixed stride.
    constexpr int NX = 8;
    const int w = (int)threadIdx.x / WAVE;
    const int xcd = (int)(blockIdx.x % NX);
    const int64_t local = blockIdx.x / NX;
    const int64_t waves_per_xcd = (int64_t)(gridDim.x / NX) * B_WAVES;
    const int64_t t_begin = n_tiles * xcd / NX, t_end = n_tiles * (xcd + 1) / NX;
    for (int64_t t = t_begin + local * B_WAVES + w; t < t_end; t += waves_per_xcd) {
        batched_tile<U>(tiles[t], perm, col, val, x, y);
    }
}

// The staged form, for tiles of 64 rows: a workgroup takes BS_WAVES tiles,
// holds their entries in registers and gathers x from LDS.
//
// What bounds the plain form is the L2's rate of lines: every gathered x is a
// 128-byte line of its own (128 matrices of 1,000 to 200,000 rows, 91 M
// entries: 573 us, 20 TB/s out of the L2s, against 0.73 GB of entries).  Here
// the x that a group of tiles reads, the columns from its smallest to its
// largest, passes through LDS once per group, in pieces of 40 KB (the next on
// its way, by direct loads, while one is read) or 80 KB where that holds all
// of it: 300 us for the same matrices, 203 against 344 for 100 matrices of
// 30,000 to 39,000 rows, 10.5 against 20 for four of 1,000 to 4,000.
//
// 512 lanes and 80 KB: two workgroups per compute unit, one streaming entries
// while the other gathers (1,024 lanes and 160 KB: 317 us; 768 and 160: 334;
// 320 and 53: 369, more rows share a piece the larger the group).  ND = 40
// entries of a row per pass, in 80 registers (32: 307, 48: 328); every load of
// a pass is in flight at once.  Rows beyond 40 entries take several passes.
constexpr int BS_THREADS = 512;
constexpr int BS_WAVES = BS_THREADS / WAVE;
constexpr int BS_PER_CU = 2;
constexpr int BS_HALF = 9984;           // floats of a piece, with room for the alignment and the zero slot
constexpr int BS_ND = 40;
// Staged where the span has fewer than this many columns per entry: 4 bytes a
// column then cost less than 128 a gathered line would, by more than the
// barriers (2 to 4 alike, 8: 20 matrices up to 200,000 rows 58 us for 50).
constexpr int BS_SPAN = 4;
constexpr int32_t BS_MAX_C = 1 << 23;

constexpr int BUFFER_RAW = 0x27000;     // word 3 of a descriptor: 32-bit data, no swizzle
constexpr int BUFFER_NT = 2;            // non-temporal

struct BSpan {          // what one wavefront's entries read
    int64_t mat;        // its matrix's offset into x
    int32_t lo, hi;     // smallest and largest column (lo > hi: no entry)
    int32_t n;          // stored slots; negative: a value is not finite
};

// n floats of x to xs + skew, straight to LDS in 16-byte pieces; x - skew and
// xs are aligned to 16 bytes, the ragged ends go one float per lane.  xs[skew +
// m], past the piece's m columns, becomes 0.
__device__ __forceinline__ void batched_stage(const float *__restrict__ x, int32_t n, int32_t m, int32_t skew, float *xs,
                                              int w)
{
    const int lane = lane_id();
    const int32_t head = min(skew ? 4 - skew : 0, n);
    const int32_t quads = (n - head) / 4, tail = head + 4 * quads;
    for (int32_t i = w * WAVE; i < quads; i += BS_THREADS)
        if (i + lane < quads)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void *)(x + head + 4 * (i + lane)),
                (__attribute__((address_space(3))) void *)(xs + skew + head + 4 * i), 16, 0, 0);
    if (w == BS_WAVES - 1) {
        if (lane < head) xs[skew + lane] = x[lane];
        if (lane < n - tail) xs[skew + tail + lane] = x[tail + lane];
        if (lane == 0) xs[skew + m] = 0.0f;
    }
}

// Up to ND entries per row, from diagonal s0 on, of the workgroup's tiles (T:
// the wavefront's, if live; spare: where a tile that has entries stores its
// first), added to s.  An entry outside the piece at hand multiplies the zero
// slot, which leaves s as it is if the value is finite; a group with other
// values, with tiles of several matrices or with a wide span gathers directly.
template <int ND>
__device__ __forceinline__ void batched_group(const BTile &T, bool live, int64_t spare, int32_t s0,
                                              const int32_t *__restrict__ col, const float *__restrict__ val,
                                              const float *__restrict__ x, float *xs, BSpan *span, int w, float &s)
{
    const int lane = lane_id();
    const int32_t steps = live ? T.nd : 0;
    // a wavefront without entries here reads the first ones of the deepest tile
    const bool some = s0 < steps;
    const int64_t base = some ? T.base + (int64_t)s0 * T.C : spare;
    const int32_t last = some ? steps - 1 - s0 : 0;
    const int32_t row_mask = some && lane < T.nrows ? 0 : -1;
    int32_t c[ND];
    float v[ND];
    // one descriptor per array, diagonals as 32-bit offsets from it (ND *
    // BS_MAX_C * 4 < 2^31): the loads in flight need no address registers
    const auto cr = __builtin_amdgcn_make_buffer_rsrc((void *)(col + base), 0, -1, BUFFER_RAW);
    const auto vr = __builtin_amdgcn_make_buffer_rsrc((void *)(val + base), 0, -1, BUFFER_RAW);
    auto at = [&](int d) { return (uint32_t)min(d, last) * (uint32_t)T.C * 4; };
#pragma unroll
    for (int d = 0; d < ND; ++d) c[d] = __builtin_amdgcn_raw_buffer_load_b32(cr, lane * 4, at(d), BUFFER_NT);
#pragma unroll
    for (int d = 0; d < ND; ++d)
        v[d] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(vr, lane * 4, at(d), BUFFER_NT));
    __builtin_amdgcn_sched_barrier(0);                        // else the compiler spills
    int32_t lo = INT32_MAX, hi = -1;
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        c[d] |= row_mask | (d <= last ? 0 : -1);
        hi = max(hi, c[d]);
        lo = (int32_t)min((uint32_t)lo, (uint32_t)c[d]);      // -1 is the largest
    }
    int32_t n = max(0, min(steps - s0, ND)) * T.nrows;
    float bad = 0.0f;                                         // NaN if a value is NaN or infinite
#pragma unroll
    for (int d = 0; d < ND; ++d) bad = fmaf(v[d], 0.0f, bad);
    if (__any(bad != bad)) n = -BS_THREADS * ND * ND;
    for (int o = 32; o; o >>= 1) {
        lo = min(lo, __shfl_xor(lo, o, WAVE));
        hi = max(hi, __shfl_xor(hi, o, WAVE));
    }
    if (lane == 0) span[w] = BSpan{T.col_base, lo, hi, n};
    __syncthreads();
    const BSpan S = span[min(lane, BS_WAVES - 1)];
    int32_t glo = S.lo, ghi = S.hi, gn = lane < BS_WAVES ? S.n : 0;
    for (int o = 32; o; o >>= 1) {
        glo = min(glo, __shfl_xor(glo, o, WAVE));
        ghi = max(ghi, __shfl_xor(ghi, o, WAVE));
        gn += __shfl_xor(gn, o, WAVE);
    }
    glo = __builtin_amdgcn_readfirstlane(glo);
    ghi = __builtin_amdgcn_readfirstlane(ghi);
    gn = __builtin_amdgcn_readfirstlane(gn);
    const bool staged = __all(S.mat == T.col_base && S.n >= 0) && ghi >= 0 && (ghi - glo) / BS_SPAN < gn;
    const float *xm = x + T.col_base;
    if (!staged) {
#pragma unroll
        for (int q = 0; q < ND; q += 8) {
            if (s0 + q >= steps || hi < 0) break;
            float xv[8];
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                // the address is made here and not ahead of all batches, which
                // costs registers (the 128 matrices above: 371 us, 300 so)
                asm volatile("" : "+v"(c[q + d]));
                xv[d] = xm[c[q + d] >= 0 ? c[q + d] : lo];
            }
#pragma unroll
            for (int d = 0; d < 8; ++d) s = c[q + d] >= 0 ? Acc<false>::mac(s, v[q + d], xv[d]) : s;
        }
        __syncthreads();                                      // span may be written again
        return;
    }
    // byte offsets in the span; no entry: past every chunk
#pragma unroll
    for (int d = 0; d < ND; ++d) c[d] = c[d] < 0 ? INT32_MIN : (c[d] - glo) * 4;
    const int32_t skew = (int32_t)((uintptr_t)(xm + glo) / sizeof(float) % 4);
    const int32_t m = ghi - glo < 2 * BS_HALF - 4 ? 2 * BS_HALF - 4 : BS_HALF - 4;
    batched_stage(xm + glo, min(m, ghi - glo + 1), m, skew, xs, w);
    uint32_t from = 0;                                        // first byte of the chunk in the span
    for (int32_t left = ghi - glo + 1, k = 0; left > 0; left -= m, ++k) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const char *xc = (const char *)(xs + (k & 1) * BS_HALF + skew);
        if (left > m) batched_stage(xm + glo + from / 4 + m, min(m, left - m), m, skew, xs + (~k & 1) * BS_HALF, w);
#pragma unroll
        for (int q = 0; q < ND; q += 8) {
            if (s0 + q >= steps) break;
            float xv[8];
#pragma unroll
            for (int d = 0; d < 8; ++d)
                xv[d] = *(const float *)(xc + min((uint32_t)c[q + d] - from, (uint32_t)m * 4));
#pragma unroll
            for (int d = 0; d < 8; ++d) s = Acc<false>::mac(s, v[q + d], xv[d]);
        }
        from += (uint32_t)m * 4;
    }
    __syncthreads();                                          // xs and span may be written again
}

__global__ __launch_bounds__(BS_THREADS, 4) void batched_staged_kernel(int64_t n_tiles, const BTile *__restrict__ tiles,
                                                                    const int32_t *__restrict__ perm,
                                                                    const int32_t *__restrict__ col,
                                                                    const float *__restrict__ val,
                                                                    const float *__restrict__ x,
                                                                    float *__restrict__ y)
{
    __shared__ __attribute__((aligned(16))) float xs[2 * BS_HALF];
    __shared__ BSpan span[BS_WAVES];
    constexpr int NX = 8;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE), lane = lane_id();
    const int xcd = (int)(blockIdx.x % NX);
    const int64_t local = blockIdx.x / NX;
    const int64_t step = (int64_t)(gridDim.x / NX) * BS_WAVES;
    const int64_t t_begin = n_tiles * xcd / NX, t_end = n_tiles * (xcd + 1) / NX;
    for (int64_t t0 = t_begin + local * BS_WAVES; t0 < t_end; t0 += step) {
        const int cnt = (int)min((int64_t)BS_WAVES, t_end - t0);
        const bool live = w < cnt;
        const BTile T = tiles[t0 + (live ? w : 0)];
        int32_t deep = 0;
        bool other = false;
        if (lane < cnt) {
            const BTile &q = tiles[t0 + lane];
            deep = q.nd;
            other = q.nd > SPMV_WIDE_ROW_NNZ || q.rlog != 6 || q.C > BS_MAX_C;
        }
        if (__any(other)) {
            if (live) batched_tile<8>(T, perm, col, val, x, y);
            continue;
        }
        const int32_t mine = deep;
        for (int o = 32; o; o >>= 1) deep = max(deep, __shfl_xor(deep, o, WAVE));
        deep = __builtin_amdgcn_readfirstlane(deep);
        const int64_t spare = tiles[t0 + __builtin_ctzll(__ballot(mine == deep))].base;
        const bool writes = live && lane < T.nrows;
        const int32_t yi = writes ? perm[T.row_base + T.r0 + lane] : 0;
        float s = 0.0f;
        for (int32_t s0 = 0; s0 < deep; s0 += BS_ND) {
            const int32_t left = deep - s0;
#define BATCHED_GROUP(ND) batched_group<ND>(T, live, spare, s0, col, val, x, xs, span, w, s)
            if (left <= 8) BATCHED_GROUP(8);
            else if (left <= 16) BATCHED_GROUP(16);
            else if (left <= 24) BATCHED_GROUP(24);
            else if (left <= 32) BATCHED_GROUP(32);
            else BATCHED_GROUP(BS_ND);
#undef BATCHED_GROUP
        }
        if (writes) y[T.row_base + yi] = s;
    }
}

}  // namespace spmv

using namespace spmv;

extern "C" {

spmv_status spmv_batched_plan(int32_t n_mat, const int32_t *h_n_rows, const int32_t *h_C, const int64_t *h_slice_base,
                              const int64_t *h_row_base, const int64_t *h_col_base, const int64_t *h_slice_ptr,
                              const int32_t *h_slice_nd, int32_t rows_per_wave, int32_t *plan, int64_t plan_cap,
                              int64_t *h_n_tiles, void *stream)
{
    SPMV_REQUIRE(n_mat >= 0, "spmv_batched_plan: n_mat < 0");
    SPMV_REQUIRE(h_n_tiles, "spmv_batched_plan: null h_n_tiles");
    if (rows_per_wave == 0) rows_per_wave = 64;
    SPMV_REQUIRE(rows_per_wave == 8 || rows_per_wave == 16 || rows_per_wave == 32 || rows_per_wave == 64,
                 "spmv_batched_plan: rows_per_wave must be 8, 16, 32 or 64");
    SPMV_REQUIRE(n_mat == 0 || (h_n_rows && h_C && h_slice_base && h_row_base && h_col_base && h_slice_ptr &&
                                h_slice_nd),
                 "spmv_batched_plan: null descriptor");
    int rlog = 0;
    while ((1 << rlog) < rows_per_wave) ++rlog;
    // matrices ordered by stored slots, largest first (stable); each matrix's
    // tiles stay together in row order so that the wavefronts working at one
    // time share that matrix's x in L2
    std::vector<int64_t> work(n_mat, 0);
    for (int32_t m = 0; m < n_mat; ++m) {
        const int32_t n = h_n_rows[m], C = h_C[m];
        SPMV_REQUIRE(n >= 0 && C > 0 && C % 64 == 0, "spmv_batched_plan: bad n_rows or C");
        for (int64_t s = 0; s < ceil_div(n, C); ++s) work[m] += (int64_t)h_slice_nd[h_slice_base[m] + s] * C;
    }
    std::vector<int32_t> order(n_mat);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return work[a] > work[b]; });
    std::vector<BTile> tiles;
    for (int32_t m : order) {
        const int32_t n = h_n_rows[m], C = h_C[m];
        const int64_t ns = ceil_div(n, C);
        for (int64_t s = 0; s < ns; ++s) {
            const int64_t sp = h_slice_ptr[h_slice_base[m] + s];
            const int32_t nd = h_slice_nd[h_slice_base[m] + s];
            for (int32_t g = 0; g < C; g += rows_per_wave) {
                const int64_t r0 = s * C + g;
                if (r0 >= n) break;
                BTile t{};
                t.base = sp + g;
                t.row_base = h_row_base[m];
                t.col_base = h_col_base[m];
                t.r0 = (int32_t)r0;
                t.nrows = (int32_t)std::min<int64_t>(rows_per_wave, n - r0);
                t.C = C;
                t.nd = nd;
                t.rlog = rlog;
                tiles.push_back(t);
            }
        }
    }
    *h_n_tiles = (int64_t)tiles.size();
    const int64_t words = (int64_t)tiles.size() * SPMV_BATCHED_PLAN_WORDS;
    if (!plan || plan_cap < words) return fail(SPMV_ERR_CAPACITY, "spmv_batched_plan: plan capacity too small");
    if (!tiles.empty()) {
        hipStream_t s = as_stream(stream);
        SPMV_HIP(hipMemcpyAsync(plan, tiles.data(), sizeof(BTile) * tiles.size(), hipMemcpyHostToDevice, s));
        SPMV_HIP(hipStreamSynchronize(s));
    }
    return SPMV_OK;
}

spmv_status spmv_batched(int64_t n_tiles, const int32_t *plan, const int32_t *perm, const int32_t *bl_col,
                         const float *bl_val, const float *x, float *y, int32_t unroll, int32_t n_workgroups,
                         void *stream)
{
    SPMV_REQUIRE(n_tiles >= 0 && n_workgroups >= 0, "spmv_batched: negative size");
    SPMV_REQUIRE(unroll == 0 || unroll == 2 || unroll == 4 || unroll == 8, "spmv_batched: unroll must be 0, 2, 4 or 8");
    if (n_tiles == 0) return SPMV_OK;
    SPMV_REQUIRE(plan && perm && bl_col && bl_val && x && y, "spmv_batched: null pointer");
    const BTile *tiles = reinterpret_cast<const BTile *>(plan);
    hipStream_t s = as_stream(stream);
    if (n_workgroups == 0 && unroll == 0) {
        // no form was asked for: staged (tiles of fewer than 64 rows, rows
        // beyond SPMV_WIDE_ROW_NNZ and huge slices take batched_tile there)
        int dev = 0, cus = 0;
        SPMV_HIP(hipGetDevice(&dev));
        SPMV_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        const int64_t groups = 8 * ceil_div(ceil_div(n_tiles, 8), BS_WAVES);
        const unsigned grid = (unsigned)std::min<int64_t>(groups, ceil_div(cus, 8) * 8 * BS_PER_CU);
        batched_staged_kernel<<<grid, BS_THREADS, 0, s>>>(n_tiles, tiles, perm, bl_col, bl_val, x, y);
        SPMV_CHECK_LAUNCH("spmv_batched");
        return SPMV_OK;
    }
    if (n_workgroups == 0) {
        int dev = 0, cus = 0;
        SPMV_HIP(hipGetDevice(&dev));
        SPMV_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        n_workgroups = cus * 8;
    }
    // a multiple of 8 workgroups: every XCD gets the same number
    const int64_t need = ceil_div(n_tiles, B_WAVES);
    int64_t g = std::min<int64_t>(n_workgroups, need);
    g = std::max<int64_t>(8, g / 8 * 8);
    const unsigned grid = (unsigned)g;
    switch (unroll) {
    case 2: batched_kernel<2><<<grid, B_THREADS, 0, s>>>(n_tiles, tiles, perm, bl_col, bl_val, x, y); break;
    case 8: batched_kernel<8><<<grid, B_THREADS, 0, s>>>(n_tiles, tiles, perm, bl_col, bl_val, x, y); break;
    default: batched_kernel<4><<<grid, B_THREADS, 0, s>>>(n_tiles, tiles, perm, bl_col, bl_val, x, y); break;
    }
    SPMV_CHECK_LAUNCH("spmv_batched");
    return SPMV_OK;
}

}  // extern "C"
