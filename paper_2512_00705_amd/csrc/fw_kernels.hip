// gfx950 kernels beside the walk itself: graph validation and layout, h_MAX / h_SUM, the edge
// index, the proposal records and label groups, the profiling kernels of the cost model and
// the random-read calibration.
#include <algorithm>

#include "fw_walk.h"

namespace fw {

__global__ void zero_kernel(unsigned long long *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// Many small copies at once, also between device and pinned host memory: a copy call of its own
// per piece costs 20 to 80 us of the calling thread (see the walk server, whose ticks move a few
// dozen pieces of some hundred KB).  blockIdx.y strides over the moves, blockIdx.x over a move.
__global__ void __launch_bounds__(kBlock) moves_kernel(const MoveDev *moves, int n)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock, t0 = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    for (int i = blockIdx.y; i < n; i += gridDim.y) {
        const MoveDev m = moves[i];
        int64_t from = 0;  // words moved 16 bytes at a time
        if (((reinterpret_cast<uintptr_t>(m.src) | reinterpret_cast<uintptr_t>(m.dst)) & 15) == 0) {
            from = m.words & ~(int64_t)3;
            const uint4 *src = reinterpret_cast<const uint4 *>(m.src);
            uint4 *dst = reinterpret_cast<uint4 *>(m.dst);
            for (int64_t k = t0; k < from / 4; k += stride) dst[k] = src ? src[k] : make_uint4(0, 0, 0, 0);
        }
        for (int64_t k = from + t0; k < m.words; k += stride) m.dst[k] = m.src ? m.src[k] : 0;
    }
}

// h_MAX and h_SUM per row (Section 4.2 preprocess()), one wave per row.  The sum is
// accumulated in double, so for float32 inputs of moderate range it is exact and the
// rounding to float32 does not depend on the summation order.
__global__ void __launch_bounds__(kBlock) preprocess_kernel(const int64_t *row_ptr, const float *h, int64_t nv,
                                                            uint4 *vrec)
{
    const int lane = lane_id();
    const int64_t nw = (int64_t)gridDim.x * (kBlock / kWave);
    for (int64_t v = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; v < nv; v += nw) {
        const int64_t b = row_ptr[v], e = row_ptr[v + 1];
        float mx = 0.0f;
        double sm = 0.0;
        for (int64_t k = b + lane; k < e; k += kWave) {
            const float x = h ? h[k] : 1.0f;
            mx = x > mx ? x : mx;
            sm += (double)x;
        }
        mx = wave_max(mx);
        sm = wave_sum_f64(sm);
        if (lane == 0) vrec[v] = make_uint4((uint32_t)b, (uint32_t)(e - b), __float_as_uint(mx), __float_as_uint((float)sm));
    }
}

// Device layout: {col, h} edge records and {start, degree, -, -} vertex records.
// 8-bit property weights: h = h_scale * code, one float32 product.
__global__ void dequantize_kernel(const uint8_t *code, float h_scale, int64_t ne, float *h)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < ne; k += stride)
        h[k] = (float)code[k] * h_scale;
}

// 8-bit property weights on graphs of at most 2^24 vertices: a 4-byte edge record.
__global__ void pack8_kernel(const int32_t *col, const uint8_t *code, int64_t ne, uint32_t *erec8)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < ne; k += stride)
        erec8[k] = (uint32_t)col[k] | ((uint32_t)code[k] << 24);
}

__global__ void layout_kernel(const int64_t *row_ptr, const int32_t *col, const float *h, int64_t nv, int64_t ne,
                              uint2 *edges, uint4 *vrec, uint32_t *start_hi)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (edges)
        for (int64_t k = t0; k < ne; k += stride)
            edges[k] = make_uint2((uint32_t)col[k], __float_as_uint(h ? h[k] : 1.0f));
    for (int64_t v = t0; v < nv; v += stride) {
        const int64_t b = row_ptr[v], e = row_ptr[v + 1];
        vrec[v] = make_uint4((uint32_t)b, (uint32_t)(e - b), 0u, 0u);
        if (start_hi) start_hi[v] = (uint32_t)((uint64_t)b >> 32);
    }
}

__global__ void validate_rows_kernel(const int64_t *row_ptr, int64_t nv, int64_t ne, int *err)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v <= nv; v += stride) {
        bool bad = false;
        if (v == 0 && row_ptr[0] != 0) bad = true;
        if (v == nv && row_ptr[nv] != ne) bad = true;
        if (v < nv && row_ptr[v] > row_ptr[v + 1]) bad = true;
        if (bad) atomicOr(err, 1);
    }
}

// Kernels over the graph's entries give every wave the same number of consecutive ones, not
// rows: with a wave per row the longest row sets the time (scale 20, 31 M entries, rows of up to
// 10^5: validation 3.6 ms, symmetry 6.3, index 7.6 of which the longest row's wave took most).
// EntrySpan: the entries [k, end) of this wave, a multiple of 64 from k on.
struct EntrySpan {
    int64_t k, end;
};

__device__ __forceinline__ EntrySpan entry_span(int64_t ne)
{
    const int64_t nw = (int64_t)gridDim.x * (kBlock / kWave);
    const int64_t each = ((ne + nw - 1) / nw + kWave - 1) / kWave * kWave;
    const int64_t k = ((int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave) * each;
    return EntrySpan{k, k + each < ne ? k + each : ne};
}

static unsigned entry_blocks(int64_t ne)
{
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(2048, (ne + kBlock - 1) / kBlock));
}

// The row of entry e, 0 <= e < row_ptr[nv]: the last v with row_ptr[v] <= e.  The whole wave
// searches 64 ways (every lane calls, with the same e).
__device__ __forceinline__ int64_t row_of_entry(const int64_t *row_ptr, int64_t nv, int64_t e)
{
    const int lane = lane_id();
    int64_t lo = 0, hi = nv;
    while (hi - lo > 1) {
        const int64_t step = (hi - lo + kWave) / (kWave + 1);
        const int64_t v = lo + (lane + 1) * step;
        const int c = __popcll(__ballot(v < hi && row_ptr[v] <= e));
        lo += c * step;
        hi = lo + step < hi ? lo + step : hi;
    }
    return lo;
}

// The rows of 64 consecutive entries k + lane (below `end`); r0 is the row of some entry at or
// before k (-1: not known yet) and becomes the row of the last one.  Every lane calls.
__device__ __forceinline__ int64_t rows_of_entries(const int64_t *row_ptr, int64_t nv, int64_t k, int64_t end,
                                                   int64_t &r0)
{
    const int lane = lane_id();
    const int64_t e = k + lane < end ? k + lane : end - 1;
    int64_t row = -1;
    if (r0 < 0) r0 = row_of_entry(row_ptr, nv, k);
    for (;;) {
        // the lane's row among the 64 from r0 on: count the row starts after r0 that are <= e
        const int64_t x = row_ptr[r0 + 1 + lane < nv ? r0 + 1 + lane : nv];
        int c = 0;
#pragma unroll
        for (int s = kWave / 2; s > 0; s >>= 1)
            if (__shfl((long long)x, c + s - 1, kWave) <= e) c += s;
        if (__shfl((long long)x, c, kWave) <= e) ++c;
        if (row < 0 && c < kWave) row = r0 + c;
        const uint64_t open = __ballot(row < 0);
        if (open == 0) break;
        r0 = row_of_entry(row_ptr, nv, k + (__ffsll((unsigned long long)open) - 1));  // many empty rows between
    }
    r0 = __shfl((long long)row, kWave - 1, kWave);
    return row;
}

// cnt[0] counts the entries that do not ascend from the entry before them, cnt[1] those of them
// that start a row: the rows are strictly ascending iff both are equal.  cnt[2] counts rows whose
// first entries (up to 64) all weigh 0.  Reads col and h once, in
// order (scale 20: 0.36 ms; with a wave per row 3.6).
__global__ void __launch_bounds__(kBlock) validate_edges_kernel(const int64_t *row_ptr, const int32_t *col,
                                                                const float *h, int64_t nv, int64_t ne, int *err,
                                                                unsigned long long *max_deg, unsigned long long *cnt)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock, t0 = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    unsigned long long falls = 0, row_falls = 0, zeros = 0, dmax = 0;
    bool bad = false;
    for (int64_t k = t0; k < ne; k += stride) {
        const int32_t c = col[k];
        if (c < 0 || (int64_t)c >= nv) bad = true;
        if (k > 0 && col[k - 1] >= c) ++falls;
        if (h) {
            const float x = h[k];
            if (!(x >= 0.0f) || isinf(x)) bad = true;
        }
    }
    for (int64_t v = t0; v < nv; v += stride) {
        const int64_t b = row_ptr[v], e = row_ptr[v + 1];
        dmax = (unsigned long long)(e - b) > dmax ? (unsigned long long)(e - b) : dmax;
        if (b > 0 && b < e && col[b - 1] >= col[b]) ++row_falls;
        if (h && b < e) {
            int64_t k = b;
            const int64_t to = e - b < kWave ? e : b + kWave;
            while (k < to && h[k] == 0.0f) ++k;
            if (k == to) ++zeros;
        }
    }
    falls = wave_sum_u64(falls);
    row_falls = wave_sum_u64(row_falls);
    zeros = wave_sum_u64(zeros);
    for (int d = kWave / 2; d > 0; d >>= 1) dmax = max(dmax, (unsigned long long)__shfl_xor((long long)dmax, d, kWave));
    if (__ballot(bad) != 0 && lane_id() == 0) atomicOr(err, 2);
    if (lane_id() == 0) {
        if (falls != 0) atomicAdd(cnt, falls);
        if (row_falls != 0) atomicAdd(cnt + 1, row_falls);
        if (zeros != 0) atomicAdd(cnt + 2, zeros);
        if (dmax > 0) atomicMax(max_deg, dmax);
    }
}

// Proposal records of h-proportional eRJS: Walker's alias table of each row's h, built
// with the sweeping construction of Huebschle-Schneider and Sanders (Parallel Weighted
// Random Sampling) in exact integer arithmetic, here in its parallel form.  Row v with n
// entries: q_k = floor(h_k / h_MAX * 2^32) (double quotient, one rounding; 2^32 when the
// row has no positive h or the graph is unweighted), Q = sum q_k, entry k brings
// a_k = q_k * n units to buckets of Q units; light entries (a_k < Q) have the deficit
// Q - a_k, heavy ones the surplus a_k - Q.  With D the deficits of the light entries
// before a given one and E the surplus of the heavy entries up to a given one (both in
// index order), the sequential sweep is equivalent to:
//   * light entry i keeps a_i and takes as alias the first heavy entry j with E_j >= D_i;
//   * heavy entry j keeps Q + E_j - D(n_j), where n_j counts the light entries with
//     D_i <= E_j and D(n_j) is their total deficit (the total of all deficits, which
//     equals the last E, when n_j covers them all); unless it keeps a full Q its alias is
//     the next heavy entry.
// Sums of up to 2^31 values below 2^63 need 128 bits; everything is an integer, so the
// result does not depend on the order of any sum.  A bucket keeping K units stores the
// threshold min(floor(K * 2^32 / Q), 2^32 - 1).
//
// Pass 1 (a wave per row, a block for the longest): Q, then each light entry's D and each heavy
// entry's E, the light entries' at the row's front in index order and the heavy ones' at its back
// in reverse order (val: the sum at its place and each entry's place, idx: the entry of a place),
// and {Q, light count} per row.  Pass 2 (a lane per entry): a search of the other sequence for
// each entry's partner, and its 64-byte record:
//   {col_k, bits(h_k), col_a, bits(h_a)}, {threshold, label_k | label_a << 8, a, 0},
//   vrec[col_k], vrec[col_a]   (a: the alias's offset in the row).
// Rows of up to 64 entries take both passes at once in registers.
using u128 = unsigned __int128;

// Rows of at most this many entries are built whole by alias_small_kernel.
constexpr int64_t kAliasSmallRow = kWave;
// The sums of a row of n entries stay below n * Q <= n^2 * 2^32 (every q_k <= 2^32).  Longer rows
// than this are scanned by alias_hub_scan_kernel, a block per row, with 128-bit sums; the others
// by a wave with sums of 64 bits, which rows of up to 2^15 entries need.
constexpr int64_t kAliasHubRow = 8192;

template <typename T>
__device__ __forceinline__ T shfl_up_t(T x, int d)
{
    if constexpr (sizeof(T) == 8) {
        return (T)__shfl_up((long long)x, d, kWave);
    } else {
        const uint64_t lo = (uint64_t)__shfl_up((long long)(uint64_t)x, d, kWave);
        const uint64_t hi = (uint64_t)__shfl_up((long long)(uint64_t)(x >> 64), d, kWave);
        return ((u128)hi << 64) | lo;
    }
}

template <typename T>
__device__ __forceinline__ T wave_incl_scan_t(T x)
{
    const int lane = lane_id();
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const T y = shfl_up_t(x, d);
        if (lane >= d) x += y;
    }
    return x;
}

// The scratch of a row that starts at entry b, 16 bytes per entry from val + b on: the sums at
// their places (64 bits, or 94 in three words), and each entry's place.
struct NarrowRow {
    using Sum = uint64_t;
    uint64_t *sums;
    uint32_t *places;
    __device__ NarrowRow(uint4 *val, int64_t b, int64_t n)
        : sums(reinterpret_cast<uint64_t *>(val + b)), places(reinterpret_cast<uint32_t *>(sums + n)) {}
    __device__ Sum sum(int64_t t) const { return sums[t]; }
    __device__ void put(int64_t t, Sum x) const { sums[t] = x; }
    __device__ uint32_t &place(int64_t k) const { return places[k]; }
};

struct WideRow {
    using Sum = u128;
    uint4 *v;
    __device__ WideRow(uint4 *val, int64_t b, int64_t) : v(val + b) {}
    __device__ Sum sum(int64_t t) const
    {
        const uint32_t *w = &v[t].x;
        return ((u128)w[2] << 64) | ((uint64_t)w[1] << 32) | w[0];
    }
    __device__ void put(int64_t t, Sum x) const
    {
        uint32_t *w = &v[t].x;
        w[0] = (uint32_t)x;
        w[1] = (uint32_t)((uint64_t)x >> 32);
        w[2] = (uint32_t)(x >> 64);
    }
    __device__ uint32_t &place(int64_t k) const { return v[k].w; }
};

// q_k of the construction: h_k relative to the row maximum in 32 fractional bits.
__device__ __forceinline__ uint64_t alias_q_of(float hk, float hmax)
{
    if (!(hmax > 0.0f)) return (uint64_t)1 << 32;
    return (uint64_t)floor(((double)hk / (double)hmax) * 4294967296.0);
}

__device__ __forceinline__ uint64_t alias_q(const float *h, int64_t k, float hmax)
{
    return h == nullptr ? (uint64_t)1 << 32 : alias_q_of(h[k], hmax);
}

// min(floor(keep * 2^32 / Q), 2^32 - 1), keep <= Q < 2^63.  The quotient in double is off by less
// than 2^-18, so its integer part by at most one, which the exact products decide.
__device__ __forceinline__ uint32_t alias_thr(uint64_t keep, uint64_t Q)
{
    if (keep >= Q) return 0xFFFFFFFFu;
    uint64_t t = (uint64_t)((double)keep / (double)Q * 4294967296.0);
    const u128 x = (u128)keep << 32, y = (u128)t * Q;
    if (y > x) --t;
    else if (x - y >= Q) ++t;
    return t >= 0xFFFFFFFFu ? 0xFFFFFFFFu : (uint32_t)t;
}

// Pass 1 on row [b, b + n) with maximum hmax.
__device__ __forceinline__ void alias_scan_row(const float *h, int64_t b, int64_t n, float hmax, uint4 *val,
                                               int32_t *idx, ulonglong2 *rowinfo_v)
{
    const int lane = lane_id();
    const NarrowRow row(val, b, n);
    const uint64_t below = lanes_below(lane);
    uint64_t qs = 0;
    for (int64_t k = lane; k < n; k += kWave) qs += alias_q(h, b + k, hmax);
    const uint64_t Q = wave_sum_u64(qs);
    uint64_t dcarry = 0, ecarry = 0;
    int64_t nl = 0, nh = 0;
    for (int64_t k0 = 0; k0 < n; k0 += kWave) {
        const int64_t k = k0 + lane;
        const bool valid = k < n;
        const uint64_t a = valid ? alias_q(h, b + k, hmax) * (uint64_t)n : 0;
        const bool light = valid && a < Q, heavy = valid && a >= Q;
        const uint64_t lm = __ballot(light), hm = __ballot(heavy);
        const uint64_t d = light ? Q - a : 0, e = heavy ? a - Q : 0;
        const uint64_t dinc = wave_incl_scan_t(d), einc = wave_incl_scan_t(e);
        if (light) {
            const int64_t pos = nl + __popcll(lm & below);
            row.put(pos, dcarry + dinc - d);  // deficits before this entry
            idx[b + pos] = (int32_t)k;
            row.place(k) = (uint32_t)pos;
        }
        if (heavy) {
            const int64_t pos = n - 1 - (nh + __popcll(hm & below));
            row.put(pos, ecarry + einc);  // surplus up to and including this entry
            idx[b + pos] = (int32_t)k;
            row.place(k) = (uint32_t)pos;
        }
        dcarry += (uint64_t)__shfl((long long)dinc, kWave - 1, kWave);
        ecarry += (uint64_t)__shfl((long long)einc, kWave - 1, kWave);
        nl += __popcll(lm);
        nh += __popcll(hm);
    }
    if (lane == 0) *rowinfo_v = make_ulonglong2((unsigned long long)Q, (unsigned long long)nl);
}

__global__ void __launch_bounds__(kBlock) alias_scan_kernel(const int64_t *row_ptr, const float *h, int64_t nv,
                                                            const uint4 *vrec, const float *rmax, uint4 *val,
                                                            int32_t *idx, ulonglong2 *rowinfo)
{
    const int64_t nw = (int64_t)gridDim.x * (kBlock / kWave);
    for (int64_t v = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; v < nv; v += nw) {
        const int64_t b = row_ptr[v];
        const int64_t n = row_ptr[v + 1] - b;
        if (n <= kAliasSmallRow || n > kAliasHubRow) continue;  // alias_small_kernel, alias_hub_scan_kernel
        const float hmax = rmax ? rmax[v] : __uint_as_float(vrec[v].z);
        alias_scan_row(h, b, n, hmax, val, idx, rowinfo + v);
    }
}

// Each lane with `valid` gives record r0..r3 for prop[4 * at]; four lanes write one together, since
// 16-byte pieces of 64 records per store are four times the requests (buf: 256 uint4 of LDS for
// the wave; the parts are swizzled over its banks).  Every lane calls.
__device__ __forceinline__ void write_records(uint4 *buf, bool valid, int64_t at, uint4 r0, uint4 r1, uint4 r2,
                                              uint4 r3, uint4 *prop)
{
    const int lane = lane_id();
    const uint64_t mask = __ballot(valid);
    uint4 *const mine = buf + lane * 4;
    const int sw = (lane >> 2) & 3;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the last records have been read
    mine[0 ^ sw] = r0;
    mine[1 ^ sw] = r1;
    mine[2 ^ sw] = r2;
    mine[3 ^ sw] = r3;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int rec = i * 16 + lane / 4, part = lane & 3;
        const int64_t k = (int64_t)__shfl((long long)at, rec, kWave);
        if ((mask >> rec) & 1) prop[(int64_t)kPropU4 * k + part] = buf[rec * 4 + (part ^ ((rec >> 2) & 3))];
    }
}

// Index of the first of the G lanes of the lane's group whose x (ascending over the lanes) is
// >= key (ge) or > key (!ge); G when there is none.
template <int G>
__device__ __forceinline__ int group_bound(uint64_t x, uint64_t key, bool ge)
{
    int c = 0;
#pragma unroll
    for (int s = G / 2; s > 0; s >>= 1) {
        const uint64_t y = (uint64_t)__shfl((long long)x, c + s - 1, G);
        if (ge ? (y < key) : (y <= key)) c += s;
    }
    const uint64_t y = (uint64_t)__shfl((long long)x, c, G);
    return (ge ? (y < key) : (y <= key)) ? c + 1 : c;
}

template <int G>
__device__ __forceinline__ uint64_t group_scan(uint64_t x)
{
    const int gl = lane_id() & (G - 1);
#pragma unroll
    for (int d = 1; d < G; d <<= 1) {
        const uint64_t y = (uint64_t)__shfl_up((long long)x, d, G);
        if (gl >= d) x += y;
    }
    return x;
}

// Both passes for rows of at most G entries, a lane per entry, 64 / G rows at once: `rows` are the
// lanes whose rows (b, n, hmax) are of this size.  The inclusive sums of the surplus and the
// exclusive ones of the deficits ascend over the lanes, so the merges are searches of the group's
// lanes.  A light entry with D > 0 finds the lane where the surplus reaches D, a heavy one; the
// first (D = 0) takes the first heavy one.  Heavy entry j's D(n_j) is the first deficit sum above
// E_j of any lane (lanes of heavy entries hold that of the next light one), or all of them.
template <int G>
__device__ __forceinline__ void alias_group_rows(uint64_t rows, const int32_t *col, const float *h,
                                                 const uint8_t *label, const uint4 *vrec, int64_t b, int32_t n,
                                                 float hmax, uint4 *buf, uint4 *prop)
{
    const int lane = lane_id(), k = lane & (G - 1), gi = lane / G;
    while (rows != 0) {
        int src = -1;
#pragma unroll
        for (int i = 0; i < kWave / G; ++i) {
            const int bit = rows != 0 ? __ffsll((unsigned long long)rows) - 1 : -1;
            if (gi == i) src = bit;
            rows &= rows - 1;  // (0 stays 0)
        }
        const int64_t rb = (int64_t)__shfl((long long)b, src < 0 ? 0 : src, kWave);
        const int32_t rn0 = __shfl(n, src < 0 ? 0 : src, kWave);
        const float rh = __shfl(hmax, src < 0 ? 0 : src, kWave);
        const int32_t rn = src < 0 ? 0 : rn0;
        const bool valid = k < rn;
        int32_t ck = 0;
        float hk = 1.0f;
        uint32_t lab = 0;
        uint4 vr = make_uint4(0, 0, 0, 0);
        uint64_t q = 0;
        if (valid) {
            ck = col[rb + k];
            if (h) hk = h[rb + k];
            if (label) lab = label[rb + k];
            vr = vrec[ck];
            q = h ? alias_q_of(hk, rh) : (uint64_t)1 << 32;
        }
        uint64_t Q = q;
#pragma unroll
        for (int d = G / 2; d > 0; d >>= 1) Q += (uint64_t)__shfl_xor((long long)Q, d, G);
        const uint64_t a = q * (uint64_t)rn;
        const bool heavy = valid && a >= Q;
        const uint64_t dinc = group_scan<G>(valid && !heavy ? Q - a : 0);
        const uint64_t E = group_scan<G>(heavy ? a - Q : 0);
        const uint64_t D = dinc - (valid && !heavy ? Q - a : 0);
        const uint64_t total = (uint64_t)__shfl((long long)E, G - 1, G);
        uint64_t hm = __ballot(heavy) >> (gi * G);
        if (G < kWave) hm &= ((uint64_t)1 << (G & 63)) - 1;
        const int ce = group_bound<G>(E, D, true), cd = group_bound<G>(D, E, false);
        const uint64_t dn = (uint64_t)__shfl((long long)D, cd & (G - 1), G);
        uint64_t keep = a;
        int al = D == 0 ? __ffsll((unsigned long long)hm) - 1 : ce;
        if (heavy) {
            keep = Q + E - (cd < G ? dn : total);
            const uint64_t later = (hm >> k) & ~(uint64_t)1;
            al = keep < Q && later != 0 ? k + __ffsll((unsigned long long)later) - 1 : k;
        } else if (al < 0 || al >= rn) {  // unreachable in exact arithmetic; a valid self-alias
            al = k;
            keep = Q;
        }
        al &= G - 1;
        const int32_t ca = __shfl(ck, al, G);
        const float ha = __shfl(hk, al, G);
        const uint32_t la = __shfl(lab, al, G);
        const uint4 va = make_uint4(__shfl(vr.x, al, G), __shfl(vr.y, al, G), __shfl(vr.z, al, G), __shfl(vr.w, al, G));
        write_records(buf, valid, rb + k, make_uint4((uint32_t)ck, __float_as_uint(hk), (uint32_t)ca, __float_as_uint(ha)),
                      make_uint4(valid ? alias_thr(keep, Q) : 0u, lab | (la << 8), (uint32_t)al, 0u), vr, va, prop);
    }
}

// Rows of 1 .. kAliasSmallRow entries: each wave takes 64 consecutive rows, by length in groups of
// 8, 16, 32 or 64 lanes per row.  Nothing goes through memory between the two passes, and the
// alias's part of a record comes from its lane (scale 20, the rows of up to 16 entries alone
// took 1.27 ms with a lane per row sweeping its entries one after another).
__global__ void __launch_bounds__(256) alias_small_kernel(const int64_t *row_ptr, const int32_t *col, const float *h,
                                                          const uint8_t *label, int64_t nv, const uint4 *vrec,
                                                          const float *rmax, uint4 *prop)
{
    __shared__ uint4 bufs[4][kWave * 4];
    uint4 *const buf = bufs[threadIdx.x / kWave];
    const int64_t nw = (int64_t)gridDim.x * 4;
    for (int64_t v0 = ((int64_t)blockIdx.x * 4 + threadIdx.x / kWave) * kWave; v0 < nv; v0 += nw * kWave) {
        const int64_t v = v0 + lane_id();
        int64_t b = 0, n = 0;
        float hmax = 0.0f;
        if (v < nv) {
            b = row_ptr[v];
            n = row_ptr[v + 1] - b;
            hmax = rmax ? rmax[v] : __uint_as_float(vrec[v].z);
        }
        alias_group_rows<8>(__ballot(n > 0 && n <= 8), col, h, label, vrec, b, (int32_t)n, hmax, buf, prop);
        alias_group_rows<16>(__ballot(n > 8 && n <= 16), col, h, label, vrec, b, (int32_t)n, hmax, buf, prop);
        alias_group_rows<32>(__ballot(n > 16 && n <= 32), col, h, label, vrec, b, (int32_t)n, hmax, buf, prop);
        alias_group_rows<64>(__ballot(n > 32 && n <= kAliasSmallRow), col, h, label, vrec, b, (int32_t)n, hmax, buf, prop);
    }
}

// The rows longer than kAliasHubRow, appended to `hubs` in any order (*nhub counts them).
__global__ void __launch_bounds__(256) alias_hub_list_kernel(const int64_t *row_ptr, int64_t nv, int32_t *hubs,
                                                             int *nhub)
{
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < nv; v += (int64_t)gridDim.x * 256)
        if (row_ptr[v + 1] - row_ptr[v] > kAliasHubRow) hubs[atomicAdd(nhub, 1)] = (int32_t)v;
}

// Pass 1 for the longest rows, a block of 1024 threads per row, two entries per thread at a time
// (scale 20, rows of up to 10^5: 1.77 ms with a wave per row, 0.28 so).
__global__ void __launch_bounds__(1024) alias_hub_scan_kernel(const int64_t *row_ptr, const float *h, const uint4 *vrec,
                                                              const float *rmax, uint4 *val, int32_t *idx,
                                                              ulonglong2 *rowinfo, const int32_t *hubs, const int *nhub)
{
    constexpr int kPer = 2, kWaves = 1024 / kWave;
    __shared__ uint64_t wq[kWaves];
    __shared__ u128 wd[kWaves], we[kWaves];
    __shared__ int wl[kWaves];
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    const int rows = *nhub;
    for (int hr = blockIdx.x; hr < rows; hr += gridDim.x) {
        const int64_t v = hubs[hr];
        const int64_t b = row_ptr[v];
        const int64_t n = row_ptr[v + 1] - b;
        if (n <= kAliasHubRow) continue;  // (the same for the whole block)
        const WideRow row(val, b, n);
        const float hmax = rmax ? rmax[v] : __uint_as_float(vrec[v].z);
        uint64_t qs = 0;
        for (int64_t k = threadIdx.x; k < n; k += 1024) qs += alias_q(h, b + k, hmax);
        qs = wave_sum_u64(qs);
        if (lane == 0) wq[wave] = qs;
        __syncthreads();
        uint64_t Q = 0;
        for (int w = 0; w < kWaves; ++w) Q += wq[w];
        u128 dcarry = 0, ecarry = 0;
        int64_t nl = 0;
        for (int64_t k0 = 0; k0 < n; k0 += 1024 * kPer) {
            const int64_t kt = k0 + (int64_t)threadIdx.x * kPer;
            uint64_t a[kPer];
            u128 td = 0, te = 0;
            int tl = 0;
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                a[i] = kt + i < n ? alias_q(h, b + kt + i, hmax) * (uint64_t)n : Q;  // (past the end: no deficit, no surplus)
                td += a[i] < Q ? Q - a[i] : 0;
                te += a[i] < Q ? 0 : a[i] - Q;
                tl += a[i] < Q ? 1 : 0;
            }
            const u128 dinc = wave_incl_scan_t(td), einc = wave_incl_scan_t(te);
            int linc = tl;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const int y = __shfl_up(linc, d, kWave);
                if (lane >= d) linc += y;
            }
            __syncthreads();  // the last tile's (or row's) sums have been read
            if (lane == kWave - 1) {
                wd[wave] = dinc;
                we[wave] = einc;
                wl[wave] = linc;
            }
            __syncthreads();
            u128 d = dcarry + dinc - td, e = ecarry + einc - te;
            int64_t l = nl + linc - tl;
#pragma unroll 1
            for (int w = 0; w < kWaves; ++w) {
                if (w < wave) {
                    d += wd[w];
                    e += we[w];
                    l += wl[w];
                }
                dcarry += wd[w];
                ecarry += we[w];
                nl += wl[w];
            }
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                if (kt + i >= n) break;
                int64_t pos;
                if (a[i] < Q) {
                    pos = l;
                    row.put(pos, d);  // deficits before this entry
                    d += Q - a[i];
                    ++l;
                } else {
                    pos = n - 1 - (kt + i - l);
                    e += a[i] - Q;
                    row.put(pos, e);  // surplus up to and including this entry
                }
                idx[b + pos] = (int32_t)(kt + i);
                row.place(kt + i) = (uint32_t)pos;
            }
        }
        if (threadIdx.x == 0) rowinfo[v] = make_ulonglong2((unsigned long long)Q, (unsigned long long)nl);
    }
}

// The alias of the entry at place t (-1: itself), and what a heavy one keeps.
template <typename Row>
__device__ __forceinline__ void alias_partner(const Row row, const int32_t *idx, int64_t b, int64_t n, int64_t nl,
                                              uint64_t Q, int64_t t, int32_t &al, uint64_t &keep)
{
    using T = typename Row::Sum;
    // A light entry looks for the first heavy j with E_j >= D (E_j at n - 1 - j), a heavy one for
    // the first light i with D_i > E (at i); sums ascend in i and j.  One loop for both, since a
    // wave has lanes of both: sum < key, key = D or E + 1.
    const bool light = t < nl;
    const T mine = row.sum(t), key = light ? mine : mine + 1;
    const int64_t at0 = light ? n - 1 : 0, dir = light ? -1 : 1;
    const int64_t m = light ? n - nl : nl;
    int64_t lo = 0, hi = m;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (row.sum(at0 + dir * mid) < key) lo = mid + 1;
        else hi = mid;
    }
    if (light) {
        al = lo < m ? idx[b + n - 1 - lo] : -1;  // (always there in exact arithmetic)
    } else {
        const T spent = row.sum(lo);  // (lo == nl: the last E, all the deficits)
        keep = (uint64_t)((T)Q + mine - spent);
        al = (keep < Q && t > nl) ? idx[b + t - 1] : -1;
    }
}

// Pass 2 for the rows longer than kAliasSmallRow, a lane per entry in the graph's order, so that
// reads and records are consecutive; each finds its partner by a binary search of the other
// sorted sequence, where neighbouring lanes search alike (scale 20: 1.60 ms; a wave per row
// merging 64 entries of both sequences at a time, entries and records in the order of the sums,
// 2.05 ms).
__global__ void __launch_bounds__(kBlock) alias_record_kernel(const int64_t *row_ptr, const int32_t *col,
                                                              const float *h, const uint8_t *label, int64_t nv,
                                                              int64_t ne, const uint4 *vrec, const float *rmax,
                                                              uint4 *val, const int32_t *idx,
                                                              const ulonglong2 *rowinfo, uint4 *prop)
{
    __shared__ uint4 bufs[kWavesPerBlock][kWave * 4];
    uint4 *const buf = bufs[threadIdx.x / kWave];
    const EntrySpan sp = entry_span(ne);
    int64_t r0 = -1;
    for (int64_t k0 = sp.k; k0 < sp.end; k0 += kWave) {
        const int64_t v = rows_of_entries(row_ptr, nv, k0, sp.end, r0);
        const int64_t e = k0 + lane_id(), b = row_ptr[v], n = row_ptr[v + 1] - b, k = e - b;
        const bool valid = e < sp.end && n > kAliasSmallRow;
        if (__ballot(valid) == 0) continue;
        uint4 r0v = make_uint4(0, 0, 0, 0), r1v = r0v, r2v = r0v, r3v = r0v;
        if (valid) {
            const ulonglong2 ri = rowinfo[v];
            const uint64_t Q = (uint64_t)ri.x;
            const int64_t nl = (int64_t)ri.y;
            const float hmax = rmax ? rmax[v] : __uint_as_float(vrec[v].z);
            const bool wide = n > kAliasHubRow;
            const int64_t t = wide ? WideRow(val, b, n).place(k) : NarrowRow(val, b, n).place(k);
            int32_t al;
            uint64_t keep = t < nl ? alias_q(h, e, hmax) * (uint64_t)n : Q;
            if (wide) alias_partner(WideRow(val, b, n), idx, b, n, nl, Q, t, al, keep);
            else alias_partner(NarrowRow(val, b, n), idx, b, n, nl, Q, t, al, keep);
            if (al < 0 && t < nl) keep = Q;  // unreachable in exact arithmetic; a valid self-alias
            const int64_t ea = al < 0 ? e : b + al;
            const int32_t ck = col[e], ca = col[ea];
            r0v = make_uint4((uint32_t)ck, __float_as_uint(h ? h[e] : 1.0f), (uint32_t)ca,
                             __float_as_uint(h ? h[ea] : 1.0f));
            r1v = make_uint4(alias_thr(keep, Q), label ? ((uint32_t)label[e] | ((uint32_t)label[ea] << 8)) : 0u,
                             (uint32_t)(ea - b), 0u);
            r2v = vrec[ck];
            r3v = vrec[ca];
        }
        write_records(buf, valid, e, r0v, r1v, r2v, r3v, prop);
    }
}

// Edge index build: each lane inserts its entry's key with a 64-bit compare-and-swap into the
// first free slot from the key's bucket on, then stores the entry's h in the slot's h part (rows
// are strictly ascending, so a key is inserted once).  The bucket is read first: slots seen taken
// stay taken, one seen free may have gone since, which the swap finds out (scale 20: 1.8 ms;
// swapping from the first slot on 4.7).  The table holds at
// least twice as many slots as keys, so every insert finds a slot within the scan.  tab: 8 uint64
// per bucket (5 keys, then 5 h).
__global__ void __launch_bounds__(kBlock) build_index_kernel(const int64_t *row_ptr, const int32_t *col,
                                                             const float *h, int64_t nv, int64_t ne,
                                                             unsigned long long *tab, uint64_t mask)
{
    const int lane = lane_id();
    const EntrySpan sp = entry_span(ne);
    int64_t r0 = -1;
    for (int64_t k0 = sp.k; k0 < sp.end; k0 += kWave) {
        const int64_t v = rows_of_entries(row_ptr, nv, k0, sp.end, r0);
        const int64_t k = k0 + lane;
        if (k >= sp.end) continue;
        const unsigned long long key = edge_key((int32_t)v, col[k]);
        uint64_t bk = mix64(key) & mask;
        bool done = false;
        for (uint64_t t = 0; t <= mask && !done; ++t) {
            unsigned long long *bucket = tab + bk * (2 * kIndexBucketU4);
            int s = 0;
            for (int i = 0; i < kIndexSlots; ++i) s += bucket[i] != kEmptyKey ? 1 : 0;
            for (; s < kIndexSlots && !done; ++s) {
                done = atomicCAS(&bucket[s], kEmptyKey, key) == kEmptyKey;
                if (done) reinterpret_cast<float *>(bucket + kIndexSlots)[s] = h ? h[k] : 1.0f;
            }
            bk = (bk + 1) & mask;
        }
    }
}

// Whether every entry (v, u) has its reverse (u, v) with the same h bits.  With the vertices
// ordered by degree, then id, only entries (v, u) with u before v look for their reverse, in u's
// row, the shorter one; their reverses are distinct entries of the other kind, so every entry of
// the other kind has its own reverse iff there are as many of both.  *balance: the difference.
// When it is not 0, or a reverse is missing or differs (bit 4 of *err), the graph is not
// symmetric.  Bound by the searches' dependent reads: scale 20, 31 M entries, 1.05 ms; bisecting
// instead of interpolating 2.1; bisecting the rows of both, a wave per row, 6.3.
__global__ void __launch_bounds__(kBlock) check_symmetry_kernel(const int64_t *row_ptr, const int32_t *col,
                                                                const float *h, int64_t nv, int64_t ne, int *err,
                                                                unsigned long long *balance)
{
    const int lane = lane_id();
    const EntrySpan sp = entry_span(ne);
    int64_t r0 = -1;
    int64_t more = 0;
    bool bad = false;
    for (int64_t k0 = sp.k; k0 < sp.end; k0 += kWave) {
        const int64_t v = rows_of_entries(row_ptr, nv, k0, sp.end, r0);
        const int64_t k = k0 + lane;
        if (k >= sp.end) continue;
        const int32_t u = col[k];
        const int64_t ub = row_ptr[u], du = row_ptr[u + 1] - ub, dv = row_ptr[v + 1] - row_ptr[v];
        if ((int64_t)u == v) continue;
        if (du > dv || (du == dv && (int64_t)u > v)) {
            --more;
            continue;
        }
        ++more;
        const int32_t pos = sorted_find_interp(col + ub, (int32_t)du, (int32_t)v, (int32_t)nv);
        if (pos < 0) bad = true;
        else if (h && __float_as_uint(h[ub + pos]) != __float_as_uint(h[k])) bad = true;
    }
    more = (int64_t)wave_sum_u64((uint64_t)more);
    if (__ballot(bad) != 0 && lane == 0) atomicOr(err, 16);
    if (lane == 0 && more != 0) atomicAdd(balance, (unsigned long long)more);
}

// Candidate nodes for the profiling kernels: candidate k is vertex k * stride (k < n), reported
// as {vertex, degree}.
__global__ void __launch_bounds__(kBlock) profile_pick_kernel(const int64_t *row_ptr, int64_t stride, int n,
                                                             int2 *out)
{
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k >= n) return;
    const int64_t v = (int64_t)k * stride;
    out[k] = make_int2((int32_t)v, (int32_t)(row_ptr[v + 1] - row_ptr[v]));
}

hipError_t launch_profile_pick(const int64_t *row_ptr, int64_t stride, int n, int2 *out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(profile_pick_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                       row_ptr, stride, n, out);
    return hipGetLastError();
}

// Profiling kernels (Section 5, "Flexi-Runtime Profiling Kernels"): evaluate workload
// weights of sampled nodes either as eRVS does (a wave scanning a row, coalesced) or
// as eRJS does (a lane proposing random neighbours).  Their time ratio per edge is the
// EdgeCost_RJS / EdgeCost_RVS constant of Eq. (runtime).
template <int KIND, bool W>
__global__ void __launch_bounds__(kBlock) profile_rvs_kernel(WalkArgs a, const int32_t *nodes, int nsample,
                                                             int per_node, float *sink)
{
    const int lane = lane_id();
    const int nw = gridDim.x * (kBlock / kWave);
    float acc = 0.0f;
    for (int s = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; s < nsample; s += nw) {
        const int32_t v = nodes[s];
        const uint4 rv = a.vrec[v];
        const int64_t b = row_start(a, rv, v), d = (int64_t)rv.y;
        const int64_t m = d < per_node ? d : per_node;
        const int32_t prev = a.col[b];
        const uint4 rp = a.vrec[prev];
        const int64_t pb = row_start(a, rp, prev), pd = (int64_t)rp.y;
        for (int64_t i = lane; i < m; i += kWave)
            acc += edge_weight<KIND, W>(a, a.q0, b + i, edge_rec(a, b + i), 1, prev, Mem{a.col + pb, pd, false, false},
                                        a.q0.schema[0], step_weights<KIND>(a.q0, (int32_t)d, (int32_t)pd));
    }
    acc = wave_max(acc);
    if (lane == 0 && acc < 0.0f) sink[0] = acc;  // never true; keeps the loads alive
}

template <int KIND, bool W>
__global__ void __launch_bounds__(kBlock) profile_rjs_kernel(WalkArgs a, const int32_t *nodes, int nsample,
                                                             int per_node, float *sink)
{
    const int s = blockIdx.x * kBlock + threadIdx.x;
    float acc = 0.0f;
    if (s < nsample) {
        const int32_t v = nodes[s];
        const uint4 rv = a.vrec[v];
        const int64_t b = row_start(a, rv, v), d = (int64_t)rv.y;
        const int32_t prev = a.col[b];
        const uint4 rp = a.vrec[prev];
        const int64_t pb = row_start(a, rp, prev), pd = (int64_t)rp.y;
        for (int t = 0; t < per_node; ++t) {
            const U4 x = philox((uint32_t)s, 0u, (uint32_t)t, 2u, a.q0.key0, a.q0.key1);
            const int64_t k = b + scaled_index(x.x0, x.x1, d);
            acc += edge_weight<KIND, W>(a, a.q0, k, edge_rec(a, k), 1, prev, Mem{a.col + pb, pd, false, true}, a.q0.schema[0],
                                        step_weights<KIND>(a.q0, (int32_t)d, (int32_t)pd));
        }
    }
    if (acc < 0.0f) sink[0] = acc;
}

// Random-read ceiling: each lane issues four independent 8-byte loads per round at
// addresses hashed from (lane, round), masked into a power-of-two array.  Its rate is the
// memory system's limit for the access pattern the walk kernel's proposals make.
__global__ void __launch_bounds__(kBlock) random_reads_kernel(const uint2 *a, uint64_t mask, int rounds,
                                                              unsigned *sink)
{
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned acc = 0;
    for (int it = 0; it < rounds; ++it) {
        uint2 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = a[mix64(t * 1315423911ull + (uint64_t)it * 64 + (uint64_t)k) & mask];
#pragma unroll
        for (int k = 0; k < 4; ++k) acc += v[k].x ^ v[k].y;
    }
    if (acc == 0x9E3779B9u) sink[0] = acc;  // keeps the loads; practically never true
}

// ---------------------------------------------------------------- launchers
hipError_t launch_random_reads(const uint2 *a, uint64_t mask, int blocks, int rounds, unsigned *sink, hipStream_t s)
{
    hipLaunchKernelGGL(random_reads_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, s, a, mask, rounds, sink);
    return hipGetLastError();
}

hipError_t launch_zero(unsigned long long *p, int n, hipStream_t s)
{
    hipLaunchKernelGGL(zero_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_moves(const MoveDev *moves, int n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(moves_kernel, dim3(32, (unsigned)std::min(n, 1024)), dim3(kBlock), 0, s, moves, n);
    return hipGetLastError();
}

hipError_t launch_preprocess(const int64_t *row_ptr, const float *h, int64_t nv, uint4 *vrec, hipStream_t s)
{
    int64_t blocks = (nv + kWavesPerBlock - 1) / kWavesPerBlock;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(preprocess_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, s, row_ptr, h, nv, vrec);
    return hipGetLastError();
}

hipError_t launch_layout(const int64_t *row_ptr, const int32_t *col, const float *h, int64_t nv, int64_t ne,
                         uint2 *edges, uint4 *vrec, uint32_t *start_hi, hipStream_t s)
{
    int64_t work = ne > nv ? ne : nv;
    int64_t blocks = (work + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(layout_kernel, dim3((unsigned)blocks), dim3(256), 0, s, row_ptr, col, h, nv, ne, edges, vrec,
                       start_hi);
    return hipGetLastError();
}

hipError_t launch_validate_rows(const int64_t *row_ptr, int64_t nv, int64_t ne, int *err, hipStream_t s)
{
    int64_t blocks = (nv + 1 + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(validate_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, s, row_ptr, nv, ne, err);
    return hipGetLastError();
}

hipError_t launch_validate_edges(const int64_t *row_ptr, const int32_t *col, const float *h, int64_t nv, int64_t ne,
                                 int *err, unsigned long long *max_deg, unsigned long long *cnt, hipStream_t s)
{
    hipLaunchKernelGGL(validate_edges_kernel, dim3(entry_blocks(std::max(nv, ne))), dim3(kBlock), 0, s, row_ptr, col, h,
                       nv, ne, err, max_deg, cnt);
    return hipGetLastError();
}

__global__ void export_alias_kernel(const uint4 *prop, int64_t ne, uint32_t *thr, int32_t *alias)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < ne; k += stride) {
        const uint4 r1 = prop[(int64_t)kPropU4 * k + 1];
        thr[k] = r1.x;
        alias[k] = (int32_t)r1.z;
    }
}

hipError_t launch_export_alias(const uint4 *prop, int64_t ne, uint32_t *thr, int32_t *alias, hipStream_t s)
{
    if (ne <= 0) return hipSuccess;
    int64_t blocks = (ne + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(export_alias_kernel, dim3((unsigned)blocks), dim3(256), 0, s, prop, ne, thr, alias);
    return hipGetLastError();
}

hipError_t launch_build_alias(const int64_t *row_ptr, const int32_t *col, const float *h, const uint8_t *label,
                              int64_t nv, int64_t ne, const uint4 *vrec, const float *rmax, uint4 *val, int32_t *idx,
                              ulonglong2 *rowinfo, int32_t *hubs, int *nhub, uint4 *prop, hipStream_t s)
{
    int64_t blocks = (nv + kWavesPerBlock - 1) / kWavesPerBlock;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    // the long rows, listed
    const unsigned lb = (unsigned)std::max<int64_t>(1, std::min<int64_t>(4096, (nv + 255) / 256));
    hipError_t e = hipMemsetAsync(nhub, 0, sizeof(int), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(alias_hub_list_kernel, dim3(lb), dim3(256), 0, s, row_ptr, nv, hubs, nhub);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // sums: a block per row for the longest, a wave for the others
    hipLaunchKernelGGL(alias_hub_scan_kernel, dim3(512), dim3(1024), 0, s, row_ptr, h, vrec, rmax, val, idx, rowinfo,
                       hubs, nhub);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(alias_scan_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, s, row_ptr, h, nv, vrec, rmax, val,
                       idx, rowinfo);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // records: a lane per entry, the short rows 64 per wave
    hipLaunchKernelGGL(alias_record_kernel, dim3(entry_blocks(ne)), dim3(kBlock), 0, s, row_ptr, col, h, label,
                       nv, ne, vrec, rmax, val, idx, rowinfo, prop);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int64_t sb = std::max<int64_t>(1, std::min<int64_t>(65536, (nv + 255) / 256));
    hipLaunchKernelGGL(alias_small_kernel, dim3((unsigned)sb), dim3(256), 0, s, row_ptr, col, h, label, nv, vrec, rmax,
                       prop);
    return hipGetLastError();
}

__global__ void __launch_bounds__(256) label_max_kernel(const uint8_t *label, int64_t ne, int *out)
{
    int m = 0;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < ne; k += (int64_t)gridDim.x * 256)
        m = max(m, (int)label[k]);
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, kWave));
    if (lane_id() == 0 && m > 0) atomicMax(out, m);
}

hipError_t launch_label_max(const uint8_t *label, int64_t ne, int *out, hipStream_t s)
{
    if (ne <= 0) return hipSuccess;
    int64_t blocks = (ne + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(label_max_kernel, dim3((unsigned)blocks), dim3(256), 0, s, label, ne, out);
    return hipGetLastError();
}

// Label groups, one wave per row: pass 1 counts each label's entries and takes its h maximum
// (a ballot and a wave maximum per label and 64-entry chunk), pass 2 scatters the entries in
// row order to their group's next positions (rank = earlier entries of the same label).
__global__ void __launch_bounds__(kBlock) label_group_kernel(const int64_t *row_ptr, const int32_t *col,
                                                             const float *h, const uint8_t *label, int64_t nv,
                                                             int nlab, int64_t *lrow, float *gmax, int32_t *vcol,
                                                             float *vh, uint8_t *vlab)
{
    const int lane = lane_id();
    const uint64_t below = lanes_below(lane);
    const int64_t nw = (int64_t)gridDim.x * (kBlock / kWave);
    for (int64_t v = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; v < nv; v += nw) {
        const int64_t b = row_ptr[v], n = row_ptr[v + 1] - b;
        int64_t pos[kMaxLabels];
        float mx[kMaxLabels];
#pragma unroll
        for (int l = 0; l < kMaxLabels; ++l) {
            pos[l] = 0;
            mx[l] = 0.0f;
        }
        for (int64_t k0 = 0; k0 < n; k0 += kWave) {
            const int64_t k = k0 + lane;
            const int lab = k < n ? (int)label[b + k] : -1;
            const float hv = k < n ? (h ? h[b + k] : 1.0f) : 0.0f;
#pragma unroll
            for (int l = 0; l < kMaxLabels; ++l) {
                if (l < nlab) {
                    const uint64_t m = __ballot(lab == l);
                    pos[l] += __popcll(m);
                    if (m != 0) mx[l] = fmaxf(mx[l], wave_max(lab == l ? hv : 0.0f));
                }
            }
        }
        int64_t start = b;
#pragma unroll
        for (int l = 0; l < kMaxLabels; ++l) {
            if (l < nlab) {
                if (lane == 0) {
                    lrow[v * nlab + l] = start;
                    gmax[v * nlab + l] = mx[l];
                }
                const int64_t c = pos[l];
                pos[l] = start;
                start += c;
            }
        }
        for (int64_t k0 = 0; k0 < n; k0 += kWave) {
            const int64_t k = k0 + lane;
            const int lab = k < n ? (int)label[b + k] : -1;
#pragma unroll
            for (int l = 0; l < kMaxLabels; ++l) {
                if (l < nlab) {
                    const uint64_t m = __ballot(lab == l);
                    if (lab == l) {
                        const int64_t p = pos[l] + __popcll(m & below);
                        vcol[p] = col[b + k];
                        if (vh) vh[p] = h[b + k];
                        vlab[p] = (uint8_t)l;
                    }
                    pos[l] += __popcll(m);
                }
            }
        }
    }
}

hipError_t launch_label_groups(const int64_t *row_ptr, const int32_t *col, const float *h, const uint8_t *label,
                               int64_t nv, int nlab, int64_t *lrow, float *gmax, int32_t *vcol, float *vh,
                               uint8_t *vlab, hipStream_t s)
{
    if (nv <= 0) return hipSuccess;
    int64_t blocks = (nv + kWavesPerBlock - 1) / kWavesPerBlock;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(label_group_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, s, row_ptr, col, h, label, nv,
                       nlab, lrow, gmax, vcol, vh, vlab);
    return hipGetLastError();
}

hipError_t launch_dequantize(const uint8_t *code, float h_scale, int64_t ne, float *h, hipStream_t s)
{
    if (ne <= 0) return hipSuccess;
    int64_t blocks = (ne + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(dequantize_kernel, dim3((unsigned)blocks), dim3(256), 0, s, code, h_scale, ne, h);
    return hipGetLastError();
}

hipError_t launch_pack8(const int32_t *col, const uint8_t *code, int64_t ne, uint32_t *erec8, hipStream_t s)
{
    if (ne <= 0) return hipSuccess;
    int64_t blocks = (ne + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(pack8_kernel, dim3((unsigned)blocks), dim3(256), 0, s, col, code, ne, erec8);
    return hipGetLastError();
}

hipError_t launch_build_index(const int64_t *row_ptr, const int32_t *col, const float *h, int64_t nv, int64_t ne,
                              unsigned long long *tab, uint64_t mask, hipStream_t s)
{
    hipLaunchKernelGGL(build_index_kernel, dim3(entry_blocks(ne)), dim3(kBlock), 0, s, row_ptr, col, h, nv, ne, tab,
                       mask);
    return hipGetLastError();
}

hipError_t launch_check_symmetry(const int64_t *row_ptr, const int32_t *col, const float *h, int64_t nv, int64_t ne,
                                 int *err, unsigned long long *balance, hipStream_t s)
{
    hipLaunchKernelGGL(check_symmetry_kernel, dim3(entry_blocks(ne)), dim3(kBlock), 0, s, row_ptr, col, h, nv, ne, err,
                       balance);
    return hipGetLastError();
}

template <int KIND, bool W>
static hipError_t launch_profile_t(const WalkArgs &a, bool rjs_style, const int32_t *nodes, int nsample,
                                   int per_node, float *sink, hipStream_t s)
{
    if (rjs_style) {
        hipLaunchKernelGGL((profile_rjs_kernel<KIND, W>), dim3((nsample + kBlock - 1) / kBlock), dim3(kBlock), 0,
                           s, a, nodes, nsample, per_node, sink);
    } else {
        int blocks = (nsample + kWavesPerBlock - 1) / kWavesPerBlock;
        hipLaunchKernelGGL((profile_rvs_kernel<KIND, W>), dim3(blocks), dim3(kBlock), 0, s, a, nodes, nsample,
                           per_node, sink);
    }
    return hipGetLastError();
}

hipError_t launch_profile(const WalkArgs &a, int kind, bool weighted, bool rjs_style, const int32_t *nodes,
                          int nsample, int per_node, float *sink, hipStream_t s)
{
    if (kind == kNode2Vec)
        return weighted ? launch_profile_t<kNode2Vec, true>(a, rjs_style, nodes, nsample, per_node, sink, s)
                        : launch_profile_t<kNode2Vec, false>(a, rjs_style, nodes, nsample, per_node, sink, s);
    if (kind == kSecondPR)
        return weighted ? launch_profile_t<kSecondPR, true>(a, rjs_style, nodes, nsample, per_node, sink, s)
                        : launch_profile_t<kSecondPR, false>(a, rjs_style, nodes, nsample, per_node, sink, s);
    return weighted ? launch_profile_t<kMetaPath, true>(a, rjs_style, nodes, nsample, per_node, sink, s)
                    : launch_profile_t<kMetaPath, false>(a, rjs_style, nodes, nsample, per_node, sink, s);
}

}  // namespace fw
