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

__global__ void fill_i32_kernel(int32_t *p, int64_t n, int32_t v)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
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
// that start a row: the rows are strictly ascending iff both are equal.  Reads col and h once, in
// order (scale 20: 0.36 ms; with a wave per row 3.6).
__global__ void __launch_bounds__(kBlock) validate_edges_kernel(const int64_t *row_ptr, const int32_t *col,
                                                                const float *h, int64_t nv, int64_t ne, int *err,
                                                                unsigned long long *max_deg, unsigned long long *cnt)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock, t0 = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    unsigned long long falls = 0, row_falls = 0, dmax = 0;
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
    }
    falls = wave_sum_u64(falls);
    row_falls = wave_sum_u64(row_falls);
    for (int d = kWave / 2; d > 0; d >>= 1) dmax = max(dmax, (unsigned long long)__shfl_xor((long long)dmax, d, kWave));
    if (__ballot(bad) != 0 && lane_id() == 0) atomicOr(err, 2);
    if (lane_id() == 0) {
        if (falls != 0) atomicAdd(cnt, falls);
        if (row_falls != 0) atomicAdd(cnt + 1, row_falls);
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
// Pass 1 (one wave per row): Q, then each light entry's D and each heavy entry's E, the
// light entries compacted at the row's front in index order and the heavy ones at its
// back in reverse order (val: the 128-bit sum, idx: the entry's offset), and {Q, light
// count} per row.  Pass 2 (one wave per row): both merges of the two sorted sequences,
// 64 entries of each at a time, and the 64-byte record of every entry:
//   {col_k, bits(h_k), col_a, bits(h_a)}, {threshold, label_k | label_a << 8, a, 0},
//   vrec[col_k], vrec[col_a]   (a: the alias's offset in the row).
using u128 = unsigned __int128;

// The sums of a row of n entries stay below n * Q <= n^2 * 2^32 (every q_k <= 2^32): 64 bits
// hold them for rows of at most 2^15 entries, which take the 64-bit path (half the lane
// exchanges of the 128-bit one).
constexpr int64_t kAlias64Max = (int64_t)1 << 15;
// Rows longer than this are merged by alias_hub_kernel, many waves per row.
constexpr int64_t kAliasHubRow = 8192;
// Rows of at most this many entries are built by alias_small_kernel, one lane per row.
constexpr int64_t kAliasSmallRow = 16;

template <typename T>
__device__ __forceinline__ T shfl_t(T x, int src)
{
    if constexpr (sizeof(T) == 8) {
        return (T)__shfl((long long)x, src, kWave);
    } else {
        const uint64_t lo = (uint64_t)__shfl((long long)(uint64_t)x, src, kWave);
        const uint64_t hi = (uint64_t)__shfl((long long)(uint64_t)(x >> 64), src, kWave);
        return ((u128)hi << 64) | lo;
    }
}

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

// A sum as stored in `val` (16 bytes, zero-extended from 64 bits).
template <typename T>
__device__ __forceinline__ T load_t(const uint4 *p)
{
    const uint4 x = *p;
    if constexpr (sizeof(T) == 8) return ((uint64_t)x.y << 32) | (uint64_t)x.x;
    else return ((u128)x.w << 96) | ((u128)x.z << 64) | ((u128)x.y << 32) | (u128)x.x;
}

template <typename T>
__device__ __forceinline__ uint4 pack_t(T x)
{
    return make_uint4((uint32_t)x, (uint32_t)((uint64_t)x >> 32), (uint32_t)((u128)x >> 64), (uint32_t)((u128)x >> 96));
}

// q_k of the construction: h_k relative to the row maximum in 32 fractional bits.
__device__ __forceinline__ uint64_t alias_q(const float *h, int64_t k, float hmax)
{
    if (h == nullptr || !(hmax > 0.0f)) return (uint64_t)1 << 32;
    return (uint64_t)floor(((double)h[k] / (double)hmax) * 4294967296.0);
}

__device__ __forceinline__ uint32_t alias_thr(u128 keep, uint64_t Q)
{
    const u128 t = (keep << 32) / (u128)Q;
    return t >= (u128)0xFFFFFFFFu ? 0xFFFFFFFFu : (uint32_t)t;
}

// Pass 1 on row [b, b + n) with maximum hmax, sums of type T.
template <typename T>
__device__ __forceinline__ void alias_scan_row(const float *h, int64_t b, int64_t n, float hmax, uint4 *val,
                                               int32_t *idx, ulonglong2 *rowinfo_v)
{
    const int lane = lane_id();
    const uint64_t below = lanes_below(lane);
    uint64_t qs = 0;
    for (int64_t k = lane; k < n; k += kWave) qs += alias_q(h, b + k, hmax);
    const uint64_t Q = wave_sum_u64(qs);
    T dcarry = 0, ecarry = 0;
    int64_t nl = 0, nh = 0;
    for (int64_t k0 = 0; k0 < n; k0 += kWave) {
        const int64_t k = k0 + lane;
        const bool valid = k < n;
        const uint64_t a = valid ? alias_q(h, b + k, hmax) * (uint64_t)n : 0;
        const bool light = valid && a < Q, heavy = valid && a >= Q;
        const uint64_t lm = __ballot(light), hm = __ballot(heavy);
        const T d = light ? (T)(Q - a) : (T)0, e = heavy ? (T)(a - Q) : (T)0;
        const T dinc = wave_incl_scan_t(d), einc = wave_incl_scan_t(e);
        if (light) {
            const int64_t pos = b + nl + __popcll(lm & below);
            val[pos] = pack_t<T>(dcarry + dinc - d);  // deficits before this entry
            idx[pos] = (int32_t)k;
        }
        if (heavy) {
            const int64_t pos = b + n - 1 - (nh + __popcll(hm & below));
            val[pos] = pack_t<T>(ecarry + einc);  // surplus up to and including this entry
            idx[pos] = (int32_t)k;
        }
        dcarry += shfl_t(dinc, kWave - 1);
        ecarry += shfl_t(einc, kWave - 1);
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
        if (n <= kAliasSmallRow) continue;  // alias_small_kernel
        const float hmax = rmax ? rmax[v] : __uint_as_float(vrec[v].z);
        if (n <= kAlias64Max) alias_scan_row<uint64_t>(h, b, n, hmax, val, idx, rowinfo + v);
        else alias_scan_row<u128>(h, b, n, hmax, val, idx, rowinfo + v);
    }
}

// Index of the first of the 64 wave lanes whose x (ascending over the lanes) is >= key
// (ge) or > key (!ge); 64 when there is none.
template <typename T>
__device__ __forceinline__ int wave_bound_t(T x, T key, bool ge)
{
    int c = 0;
#pragma unroll
    for (int s = kWave / 2; s > 0; s >>= 1) {
        const T y = shfl_t(x, c + s - 1);
        if (ge ? (y < key) : (y <= key)) c += s;
    }
    // c in [0, 63]: one more test decides between c and 64
    const T y = shfl_t(x, c);
    return (ge ? (y < key) : (y <= key)) ? c + 1 : c;
}

__device__ __forceinline__ void write_record(const int32_t *col, const float *h, const uint8_t *label,
                                             const uint4 *vrec, int64_t b, int32_t k, int32_t al, uint32_t thr,
                                             uint4 *prop)
{
    const uint32_t hk = h ? __float_as_uint(h[b + k]) : __float_as_uint(1.0f);
    const uint32_t ha = h ? __float_as_uint(h[b + al]) : __float_as_uint(1.0f);
    const uint32_t lab = label ? ((uint32_t)label[b + k] | ((uint32_t)label[b + al] << 8)) : 0u;
    const int32_t ck = col[b + k], ca = col[b + al];
    uint4 *r = prop + (int64_t)kPropU4 * (b + k);
    r[0] = make_uint4((uint32_t)ck, hk, (uint32_t)ca, ha);
    r[1] = make_uint4(thr, lab, (uint32_t)al, 0u);
    r[2] = vrec[ck];
    r[3] = vrec[ca];
}

// Pass 2 on row [b, b + n) with Q and nl from pass 1, sums of type T.
template <typename T>
__device__ __forceinline__ void alias_merge_row(const int32_t *col, const float *h, const uint8_t *label,
                                                const uint4 *vrec, const uint4 *val, const int32_t *idx, int64_t b,
                                                int64_t n, uint64_t Q, int64_t nl, float hmax, uint4 *prop)
{
    const int lane = lane_id();
    constexpr T kMax = ~(T)0;
    const int64_t nh = n - nl;  // >= 1 (the caller checked)
    // heavy entry j (in index order) sits at b + n - 1 - j
    const T e_last = load_t<T>(val + b + n - nh);
    // light entries: alias = the first heavy entry whose E reaches the entry's D
    for (int64_t li = 0, hj = 0; li < nl;) {
        if (hj >= nh) {
            // unreachable in exact arithmetic (the last E equals the total deficit, so
            // every light entry finds its heavy one); kept so that the loop always ends
            // and every record stays a valid self-alias
            for (int64_t i = li + lane; i < nl; i += kWave) {
                const int32_t k = idx[b + i];
                write_record(col, h, label, vrec, b, k, k, 0xFFFFFFFFu, prop);
            }
            break;
        }
        const int64_t i = li + lane, j = hj + lane;
        const T D = i < nl ? load_t<T>(val + b + i) : kMax;
        const T E = j < nh ? load_t<T>(val + b + n - 1 - j) : kMax;
        const int32_t hix = j < nh ? idx[b + n - 1 - j] : -1;
        const int c = wave_bound_t(E, D, true);
        const bool found = i < nl && c < kWave && hj + c < nh;
        const int32_t al = __shfl(hix, c & (kWave - 1), kWave);
        const int cnt = __popcll(__ballot(found));  // a prefix of the lanes (D ascends)
        if (cnt == 0) {
            hj += kWave;
            continue;
        }
        if (found) {
            const int32_t k = idx[b + i];
            const uint64_t a = alias_q(h, b + k, hmax) * (uint64_t)n;
            write_record(col, h, label, vrec, b, k, al, alias_thr((u128)a, Q), prop);
        }
        li += cnt;
    }
    // heavy entries: keep Q + E_j - D(n_j), alias the next heavy entry unless full
    for (int64_t hj = 0, li = 0; hj < nh;) {
        const int64_t i = li + lane, j = hj + lane;
        const T D = i < nl ? load_t<T>(val + b + i) : kMax;
        const T E = j < nh ? load_t<T>(val + b + n - 1 - j) : kMax;
        const int c = wave_bound_t(D, E, false);  // light entries with D <= E_j in this block
        const bool found = j < nh && c < kWave;
        const T dn = shfl_t(D, c & (kWave - 1));
        const int cnt = __popcll(__ballot(found));  // a prefix of the lanes (E ascends)
        if (cnt == 0) {
            li += kWave;
            continue;
        }
        if (found) {
            const T spent = li + c < nl ? dn : e_last;
            const T keep = (T)Q + E - spent;
            const int32_t k = idx[b + n - 1 - j];
            const int32_t al = (keep < (T)Q && j + 1 < nh) ? idx[b + n - 2 - j] : k;
            write_record(col, h, label, vrec, b, k, al, alias_thr((u128)keep, Q), prop);
        }
        hj += cnt;
    }
}

__global__ void __launch_bounds__(kBlock) alias_merge_kernel(const int64_t *row_ptr, const int32_t *col,
                                                             const float *h, const uint8_t *label, int64_t nv,
                                                             const uint4 *vrec, const float *rmax, const uint4 *val,
                                                             const int32_t *idx, const ulonglong2 *rowinfo,
                                                             uint4 *prop)
{
    const int lane = lane_id();
    const int64_t nw = (int64_t)gridDim.x * (kBlock / kWave);
    for (int64_t v = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; v < nv; v += nw) {
        const int64_t b = row_ptr[v];
        const int64_t n = row_ptr[v + 1] - b;
        if (n <= kAliasSmallRow) continue;  // alias_small_kernel
        const ulonglong2 ri = rowinfo[v];
        const uint64_t Q = (uint64_t)ri.x;
        const int64_t nl = (int64_t)ri.y;
        if (n - nl <= 0) {  // unreachable (the a_k sum to n * Q); every record stays a valid self-alias
            for (int64_t k = lane; k < n; k += kWave)
                write_record(col, h, label, vrec, b, (int32_t)k, (int32_t)k, 0xFFFFFFFFu, prop);
            continue;
        }
        if (n > kAliasHubRow) continue;  // alias_hub_kernel
        const float hmax = rmax ? rmax[v] : __uint_as_float(vrec[v].z);
        if (n <= kAlias64Max) alias_merge_row<uint64_t>(col, h, label, vrec, val, idx, b, n, Q, nl, hmax, prop);
        else alias_merge_row<u128>(col, h, label, vrec, val, idx, b, n, Q, nl, hmax, prop);
    }
}

// Rows of 1 .. kAliasSmallRow entries, one lane per row: the sweep itself, in entry order.
// A(k) = q_k * n.  With the current heavy entry j holding residual r: each light entry i
// (A < Q) first closes the heavy entries whose residual has fallen below Q (bucket j keeps
// r, aliased to the next heavy entry, which then holds A(j') - (Q - r)), then keeps A(i)
// with j as its alias, and r loses Q - A(i); the heavy entries left at the end are closed
// the same way, a full bucket being its own alias.  This is the table the two passes
// above build for longer rows (sums here stay below 16 * 16 * 2^32).
__global__ void __launch_bounds__(256) alias_small_kernel(const int64_t *row_ptr, const int32_t *col, const float *h,
                                                          const uint8_t *label, int64_t nv, const uint4 *vrec,
                                                          const float *rmax, uint4 *prop)
{
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < nv; v += (int64_t)gridDim.x * 256) {
        const int64_t b = row_ptr[v];
        const int32_t n = (int32_t)(row_ptr[v + 1] - b);
        if (n == 0 || n > kAliasSmallRow) continue;
        const float hmax = rmax ? rmax[v] : __uint_as_float(vrec[v].z);
        uint64_t Q = 0;
        for (int32_t k = 0; k < n; ++k) Q += alias_q(h, b + k, hmax);
        auto A = [&](int32_t k) { return alias_q(h, b + k, hmax) * (uint64_t)n; };
        int32_t j = 0;
        while (A(j) < Q) ++j;  // the first heavy entry (the A sum to n * Q)
        uint64_t r = A(j);
        for (int32_t i = 0; i < n; ++i) {
            const uint64_t ai = A(i);
            if (ai >= Q) continue;
            while (r < Q) {  // a later heavy entry exists while a light entry is left
                int32_t jn = j + 1;
                while (jn < n - 1 && A(jn) < Q) ++jn;
                write_record(col, h, label, vrec, b, j, jn, alias_thr((u128)r, Q), prop);
                r = A(jn) - (Q - r);
                j = jn;
            }
            write_record(col, h, label, vrec, b, i, j, alias_thr((u128)ai, Q), prop);
            r -= Q - ai;
        }
        for (;;) {
            int32_t jn = j + 1;
            while (jn < n && A(jn) < Q) ++jn;
            write_record(col, h, label, vrec, b, j, (r < Q && jn < n) ? jn : j, alias_thr((u128)r, Q), prop);
            if (jn >= n) break;
            r = A(jn) - (Q - r);
            j = jn;
        }
    }
}

// The rows longer than kAliasHubRow, appended to `hubs` in any order (*nhub counts them).
__global__ void __launch_bounds__(256) alias_hub_list_kernel(const int64_t *row_ptr, int64_t nv, int32_t *hubs,
                                                             int *nhub)
{
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < nv; v += (int64_t)gridDim.x * 256)
        if (row_ptr[v + 1] - row_ptr[v] > kAliasHubRow) hubs[atomicAdd(nhub, 1)] = (int32_t)v;
}

// Pass 2 for the long rows, one thread per entry (blockIdx.y picks the row, the blocks of a
// row stride over its entries): the same two merges, each entry finding its partner by a
// binary search of the other sorted sequence instead of a wave walking the row, so that a
// hub row is spread over many waves.  Light entry i: alias = the first heavy entry with
// E >= D_i.  Heavy entry j: keep Q + E_j - D(first light entry with D > E_j, or the last
// E), alias the next heavy entry unless it keeps a full bucket.
__global__ void __launch_bounds__(256) alias_hub_kernel(const int64_t *row_ptr, const int32_t *col, const float *h,
                                                        const uint8_t *label, const uint4 *vrec, const float *rmax,
                                                        const uint4 *val, const int32_t *idx,
                                                        const ulonglong2 *rowinfo, const int32_t *hubs,
                                                        const int *nhub, uint4 *prop)
{
    const int nh_rows = *nhub;
    for (int hr = blockIdx.y; hr < nh_rows; hr += gridDim.y) {
        const int64_t v = hubs[hr];
        const int64_t b = row_ptr[v];
        const int64_t n = row_ptr[v + 1] - b;
        const ulonglong2 ri = rowinfo[v];
        const uint64_t Q = (uint64_t)ri.x;
        const int64_t nl = (int64_t)ri.y, nh = n - nl;
        const float hmax = rmax ? rmax[v] : __uint_as_float(vrec[v].z);
        for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < n; t += (int64_t)gridDim.x * 256) {
            if (nh <= 0) {  // unreachable (the a_k sum to n * Q); a valid self-alias
                write_record(col, h, label, vrec, b, (int32_t)t, (int32_t)t, 0xFFFFFFFFu, prop);
                continue;
            }
            if (t < nl) {
                const u128 D = load_t<u128>(val + b + t);
                int64_t lo = 0, hi = nh;  // first heavy j with E_j >= D (E_j at b + n - 1 - j, ascending in j)
                while (lo < hi) {
                    const int64_t mid = (lo + hi) >> 1;
                    if (load_t<u128>(val + b + n - 1 - mid) < D) lo = mid + 1;
                    else hi = mid;
                }
                const int32_t k = idx[b + t];
                if (lo >= nh) {  // unreachable in exact arithmetic; a valid self-alias
                    write_record(col, h, label, vrec, b, k, k, 0xFFFFFFFFu, prop);
                    continue;
                }
                const uint64_t a = alias_q(h, b + k, hmax) * (uint64_t)n;
                write_record(col, h, label, vrec, b, k, idx[b + n - 1 - lo], alias_thr((u128)a, Q), prop);
            } else {
                const int64_t j = t - nl;
                const u128 E = load_t<u128>(val + b + n - 1 - j);
                int64_t lo = 0, hi = nl;  // first light i with D_i > E (D ascending in i)
                while (lo < hi) {
                    const int64_t mid = (lo + hi) >> 1;
                    if (load_t<u128>(val + b + mid) <= E) lo = mid + 1;
                    else hi = mid;
                }
                const u128 spent = lo < nl ? load_t<u128>(val + b + lo) : load_t<u128>(val + b + n - nh);
                const u128 keep = (u128)Q + E - spent;
                const int32_t k = idx[b + n - 1 - j];
                const int32_t al = (keep < (u128)Q && j + 1 < nh) ? idx[b + n - 2 - j] : k;
                write_record(col, h, label, vrec, b, k, al, alias_thr(keep, Q), prop);
            }
        }
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
// the other kind has its own reverse iff there are as many of both.  *balance: the difference
// (scale 20: 2.1 ms; searching the rows of both, a wave per row, 6.3).  Else, or when a
// reverse is missing or differs, the graph is not symmetric: bit 4 of *err for the latter.
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
        const int64_t pos = sorted_find(col + ub, du, (int32_t)v);
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

hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
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
                              int64_t nv, const uint4 *vrec, const float *rmax, uint4 *val, int32_t *idx,
                              ulonglong2 *rowinfo, int32_t *hubs, int *nhub, uint4 *prop, hipStream_t s)
{
    int64_t blocks = (nv + kWavesPerBlock - 1) / kWavesPerBlock;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(alias_scan_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, s, row_ptr, h, nv, vrec, rmax, val,
                       idx, rowinfo);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(alias_merge_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, s, row_ptr, col, h, label, nv,
                       vrec, rmax, val, idx, rowinfo, prop);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // the short rows, one lane each
    int64_t sb = (nv + 255) / 256;
    if (sb > 65536) sb = 65536;
    if (sb < 1) sb = 1;
    hipLaunchKernelGGL(alias_small_kernel, dim3((unsigned)sb), dim3(256), 0, s, row_ptr, col, h, label, nv, vrec, rmax,
                       prop);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // the long rows: listed, then one thread per entry
    if ((e = hipMemsetAsync(nhub, 0, sizeof(int), s)) != hipSuccess) return e;
    int64_t lb = (nv + 255) / 256;
    if (lb > 4096) lb = 4096;
    if (lb < 1) lb = 1;
    hipLaunchKernelGGL(alias_hub_list_kernel, dim3((unsigned)lb), dim3(256), 0, s, row_ptr, nv, hubs, nhub);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(alias_hub_kernel, dim3(64, 1024), dim3(256), 0, s, row_ptr, col, h, label, vrec, rmax, val, idx,
                       rowinfo, hubs, nhub, prop);
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
