// Device functions that the walk kernels share: weights, the membership test, one eRVS step
// by a whole wave (and by groups of lanes), path flushes and counters.
#pragma once

#include "fw_device.h"
#include "fw_internal.h"

namespace fw {

// An LDS address for the LDS-DMA load builtin (the pointer must lie in this block's LDS).
__device__ __forceinline__ __attribute__((address_space(3))) void *lds_ptr(uint4 *p)
{
    return (__attribute__((address_space(3))) void *)p;
}

// N(prev) for the membership test: a copy in this wave's LDS or the row of prev in col,
// read through one flat pointer either way.  `indexed`: lanes test different rows (eRJS
// style); an unstaged row then goes through the edge index when the graph has one, else
// an interpolation search (fewest probes per lane).  Otherwise the whole wave tests one
// row (an eRVS step): its probes hit the cache, and a branch-free bisection, whose trip
// count is the same in every lane, beats a search that is cheaper on average but waits
// for its slowest lane.
struct Mem {
    const int32_t *p;
    int64_t len;
    bool staged;
    bool indexed;
};

// u in N(prev): LDS copy, else the edge index if asked for, else a search of the row.
__device__ __forceinline__ bool in_prev_row(const WalkArgs &a, const Mem &m, int32_t prev, int32_t u)
{
    if (m.indexed) {
        if (!m.staged && a.mtab != nullptr) return index_contains(a.mtab, a.mtab_mask, prev, u);
        return sorted_contains_interp(m.p, (int32_t)m.len, u, (int32_t)a.nv);
    }
    return sorted_contains_bisect(m.p, (int32_t)m.len, u);
}

// The constants of query q: a device table for batched launches, the kernel argument
// block otherwise.
template <bool BATCH>
__device__ __forceinline__ const QueryDev &query(const WalkArgs &a, int32_t q)
{
    return BATCH ? a.queries[q] : a.q0;
}

// The workload weights of a step that depend on u only through u in N(prev): `mem` for
// u in N(prev), `oth` otherwise, `ret` for u = prev, and their smallest and largest
// (Node2Vec: 1, 1/q, 1/p from the query; second-order PageRank: the two branches of
// Eq. (2ndpr) at this step's d(v), d(v'), the return taking the second).
struct StepW {
    float mem, oth, ret, lo, hi;
};

template <int KIND>
__device__ __forceinline__ StepW step_weights(const QueryDev &Q, int32_t dv, int32_t dvp)
{
    if (KIND == kSecondPR) {
        // in float32 in the order of Eq. (2ndpr): ((1-g)/d(v) + g/d(v')) * max_d, ((1-g)/d(v)) * max_d
        const float t1 = Q.omg / (float)dv;
        const float t2 = Q.gamma / (float)(dvp > 0 ? dvp : 1);
        const float md = (float)(dv > dvp ? dv : dvp);
        const float in = (t1 + t2) * md, out = t1 * md;
        return StepW{in, out, out, fminf(in, out), fmaxf(in, out)};
    }
    return StepW{1.0f, Q.inv_q, Q.inv_p, Q.lo_w, Q.hi_w};
}

// Transition weight w~ = w * h of the edge at CSR position k (record e) at step j
// (Section 2.1, Eq. prob; Eq. node2vec; MetaPath rule; Eq. 2ndpr).  `m` holds N(prev)
// sorted; `sw` the step's weights, by value: through a reference the compiler makes of the three
// branches one load of a chosen address, with the weights in scratch memory, and every edge of
// a scan waits for it.
template <int KIND, bool W>
__device__ __forceinline__ float edge_weight(const WalkArgs &a, const QueryDev &Q, int64_t k, uint2 e, int j,
                                             int32_t prev, const Mem &m, uint8_t want, StepW sw)
{
    const float hv = W ? __uint_as_float(e.y) : 1.0f;
    if (KIND == kSecondPR) {
        if (j == 0) return hv;
        const int32_t u = (int32_t)e.x;
        if (u == prev) return sw.ret * hv;
        return in_prev_row(a, m, prev, u) ? sw.mem * hv : sw.oth * hv;
    }
    if (KIND == kNode2Vec) {
        if (j == 0) return hv;
        const int32_t u = (int32_t)e.x;
        if (u == prev) return Q.inv_p * hv;
        return in_prev_row(a, m, prev, u) ? hv : Q.inv_q * hv;
    } else {
        return a.label[k] == want ? hv : 0.0f;
    }
}

// The {col, bits(h)} record of CSR entry k: the 8-byte record, or the 4-byte record of an
// 8-bit-weight graph decoded (h = h_scale * code, one float32 product).
__device__ __forceinline__ uint2 edge_rec(const WalkArgs &a, int64_t k)
{
    if (a.erec8 != nullptr) {
        const uint32_t x = a.erec8[k];
        return make_uint2(x & 0xFFFFFFu, __float_as_uint((float)(x >> 24) * a.h_scale));
    }
    return a.edges[k];
}

// Store the n held path slots p0.. at dst (walk ended or suspended).
__device__ __forceinline__ void flush_path(int32_t *dst, int32_t n, int32_t p0, int32_t p1, int32_t p2)
{
    dst[0] = p0;
    if (n > 1) dst[1] = p1;
    if (n > 2) dst[2] = p2;
}

__device__ __forceinline__ int64_t row_start(const WalkArgs &a, uint4 r, int32_t v)
{
    return a.start_hi ? (int64_t)(((uint64_t)a.start_hi[v] << 32) | r.x) : (int64_t)r.x;
}

// u in N(prev) for the 64 items of one eRVS round, all lanes together: the round's items
// are consecutive entries of cur's sorted row, so the wave merges them with N(prev)
// (sorted, m.p[0, m.len)): it loads the next 64 entries of N(prev) from the wave's cursor
// `lo` (one coalesced load), each lane finds its item among them by a bisection over the
// lanes (ds_bpermute), and the block advances while some item lies beyond it.  The cursor
// then moves past everything below the round's largest item.  Over a whole scan this
// reads N(prev) once, in order, where a search per item costs log d(prev) dependent loads.
// A round whose largest item lies below the entry at the cursor holds no member and
// leaves the cursor where it is: it needs no bisection (the usual round of a hub row
// scanned from a short N(prev)).
// `valid`: the lane holds an item; every lane must call this.
__device__ __forceinline__ bool merge_member(const Mem &m, int32_t u, bool valid, int64_t &lo)
{
    const int lane = lane_id();
    const uint64_t vm = __ballot(valid);
    if (vm == 0) return false;
    // items are consecutive entries of a sorted row: the largest sits in the last valid lane
    const int32_t umax = __builtin_amdgcn_readlane(u, 63 - __builtin_clzll((unsigned long long)vm));
    bool found = false, done = !valid;
    int32_t c = 0;
    for (bool first = true;; first = false) {
        const int64_t vi = lo + lane;
        const int32_t v = vi < m.len ? m.p[vi] : INT32_MAX;
        if (first && umax < __builtin_amdgcn_readfirstlane(v)) return false;
        c = 0;
#pragma unroll
        for (int s = kWave / 2; s > 0; s >>= 1) {
            const int32_t pv = __shfl(v, c + s - 1, kWave);
            if (pv < u) c += s;
        }
        const int32_t vc = __shfl(v, c & (kWave - 1), kWave);
        const int32_t vlast = __shfl(v, kWave - 1, kWave);
        if (!done) {
            found = c < kWave && vc == u;
            done = u <= vlast;
        }
        if (__ballot(!done) == 0) break;
        lo += kWave;  // every open item lies beyond this whole block
    }
    lo += __shfl(c, kWave - 1, kWave);  // entries below the round's largest item
    return found;
}

// merge_member for rows scanned by 64 lanes and for the eRVS-only kernel, same results.  The block of N(prev) at
// the cursor is loaded before the items are first used (it does not depend on them), so
// that its load overlaps the load of the round's edges instead of following it.  Of the
// block, only entries within [smallest item, largest item] can equal an item; when there
// are few (a hub row scanned against a shorter N(prev): a handful per round), each is
// broadcast from its lane and compared with every item at once, with no LDS round trip;
// otherwise each lane bisects the block as merge_member does.  The cursor then moves past
// every entry up to the largest item (later rounds hold only larger items).  walk_kernel's hub
// rows keep merge_member: there the longer-lived block spills.
constexpr int kMergeBcast = 8;  // most in-range entries compared by broadcast (8: 2.98 s, 16: 3.01 s, 32: 3.20 s on eRVS-only scale 22)
__device__ __forceinline__ bool merge_member_early(const Mem &m, int32_t u, bool valid, int64_t &lo)
{
    const int lane = lane_id();
    int32_t v = lo + lane < m.len ? m.p[lo + lane] : INT32_MAX;
    const uint64_t vm = __ballot(valid);
    if (vm == 0) return false;
    // items are consecutive entries of a sorted row held by a prefix of the lanes
    const int32_t umin = __builtin_amdgcn_readlane(u, __builtin_ctzll((unsigned long long)vm));
    const int32_t umax = __builtin_amdgcn_readlane(u, 63 - __builtin_clzll((unsigned long long)vm));
    if (umax < __builtin_amdgcn_readfirstlane(v)) return false;
    bool found = false;
    for (;;) {
        const uint64_t inr = __ballot(v >= umin && v <= umax);
        if (__popcll(inr) <= kMergeBcast) {
            for (uint64_t mm = inr; mm != 0; mm &= mm - 1) {
                const int32_t e = __builtin_amdgcn_readlane(v, __builtin_ctzll((unsigned long long)mm));
                found = found || u == e;
            }
        } else {
            int32_t c = 0;
#pragma unroll
            for (int s = kWave / 2; s > 0; s >>= 1) {
                const int32_t pv = __shfl(v, c + s - 1, kWave);
                if (pv < u) c += s;
            }
            const int32_t vc = __shfl(v, c & (kWave - 1), kWave);
            found = found || (c < kWave && vc == u);
        }
        const uint64_t le = __ballot(v <= umax);  // a prefix of the block: entries up to the largest item
        if (~le != 0ull) {
            lo += __popcll(le);
            break;
        }
        lo += kWave;
        v = lo + lane < m.len ? m.p[lo + lane] : INT32_MAX;
    }
    return found && valid;
}

template <bool EARLY>
__device__ __forceinline__ bool merge_member_t(const Mem &m, int32_t u, bool valid, int64_t &lo)
{
    return EARLY ? merge_member_early(m, u, valid, lo) : merge_member(m, u, valid, lo);
}

// Transition weight from the membership of u in N(prev) (the same expression as
// edge_weight, for Node2Vec and second-order PageRank).
template <int KIND, bool W>
__device__ __forceinline__ float weight_of_member(uint2 e, int j, int32_t prev, bool member, StepW sw)
{
    const float hv = W ? __uint_as_float(e.y) : 1.0f;
    if (j == 0) return hv;
    if ((int32_t)e.x == prev) return sw.ret * hv;
    return member ? sw.mem * hv : sw.oth * hv;
}

// Shared eRVS threshold (plan rvs_share): after a scan round in which some lane drew a
// key, a lane whose threshold lies below the largest one, g, takes g.  Its remaining skip
// T - S is exponential with rate -thr (no item since its last draw has passed it), so
// scaled by thr / g it is the skip towards the first item whose key beats g; keys below g
// cannot win the argmax.  A lane with no threshold yet (-inf) keeps T = 0.
__device__ __forceinline__ void take_shared_threshold(float &thr, float &T, float &S, float g)
{
    if (thr > -INFINITY && thr < g) {
        T = g >= 0.0f ? INFINITY : ((T - S) * thr) / g;
        S = 0.0f;
        thr = g;
    }
}

// eRVS for one step, all 64 lanes cooperating.  Returns the next vertex or -1 when no
// neighbour has positive weight, with the h of the chosen edge in `hsel`.  `trig`
// receives the number of jump events.  `merge`: find u in N(prev) by merging the rows
// (merge_member) instead of searching `mem` per item.
template <int KIND, bool W, bool EARLY>
__device__ __forceinline__ int32_t rvs_step(const WalkArgs &a, const QueryDev &Q, const Mem &mem, uint32_t wid,
                                            int j, int32_t prev, int64_t base, int64_t deg, uint8_t want,
                                            const StepW &sw, uint32_t &trig, float &hsel, bool merge)
{
    const int lane = lane_id();
    const uint32_t k0 = Q.key0, k1 = Q.key1;
    float key = -INFINITY;
    int32_t bi = -1;
    float ru = 0.5f;
    int64_t mlo = 0;  // merge cursor in N(prev)
    // round 0: lane l keys neighbour l, k = u^(1/w~) kept as log(u) / w~
    const uint2 e0 = lane < deg ? edge_rec(a, base + lane) : make_uint2(0u, 0u);
    const bool mem0 = merge && merge_member_t<EARLY>(mem, (int32_t)e0.x, lane < deg, mlo);
    if (lane < deg) {
        const int64_t k = base + lane;
        const float wt = merge ? weight_of_member<KIND, W>(e0, j, prev, mem0, sw)
                               : edge_weight<KIND, W>(a, Q, k, e0, j, prev, mem, want, sw);
        const U4 x = philox(wid, (uint32_t)j, (uint32_t)lane, 1u, k0, k1);
        key = wt > 0.0f ? ln_f(unit_uniform(x.x0)) / wt : -INFINITY;
        ru = unit_uniform(x.x1);
        bi = lane;
    }
    const float lkg = wave_max(key);
    float thr = lkg;
    float T = (thr == -INFINITY) ? 0.0f : (thr >= 0.0f ? INFINITY : ln_f(ru) / thr);
    float S = 0.0f;
    uint32_t nt = 0;
    // scan: lane l owns neighbours l + 64, l + 128, ...; a key is drawn only where the
    // running weight passes the skip threshold T = log(r) / log(k_thr)
    for (int64_t i0 = kWave; i0 < deg; i0 += kWave) {
        const int64_t i = i0 + lane;
        const uint2 ei = i < deg ? edge_rec(a, base + i) : make_uint2(0u, 0u);
        const bool memi = merge && merge_member_t<EARLY>(mem, (int32_t)ei.x, i < deg, mlo);
        bool drew = false;
        if (i < deg) {
            const int64_t k = base + i;
            const float wt = merge ? weight_of_member<KIND, W>(ei, j, prev, memi, sw)
                                   : edge_weight<KIND, W>(a, Q, k, ei, j, prev, mem, want, sw);
            S = S + wt;
            if (S > T) {
                // key conditioned to beat thr: log u' = log1p(expm1(w~ * thr) * V)
                const U4 x = philox(wid, (uint32_t)j, (uint32_t)i, 1u, k0, k1);
                const float av = wt * thr;
                const float m1 = expm1_f(av);
                const float z = m1 * unit_uniform(x.x0);
                const float lg = log1p_f(z);
                key = lg / wt;
                bi = (int32_t)i;
                thr = key;
                S = 0.0f;
                T = thr >= 0.0f ? INFINITY : ln_f(unit_uniform(x.x1)) / thr;
                ++nt;
                drew = true;
            }
        }
        if (a.rvs_share && __ballot(drew) != 0) take_shared_threshold(thr, T, S, wave_max(thr));
    }
    wave_argmax(key, bi);
    trig = (uint32_t)wave_sum_u64(nt);
    if (!(key > -INFINITY)) return -1;
    const uint2 e = edge_rec(a, base + bi);
    hsel = W ? __uint_as_float(e.y) : 1.0f;
    return (int32_t)e.x;
}

// rvs_step with P = 64 * V reservoir lanes (V > 1, hub rows): lane l of the wave runs the
// virtual lanes l, l + 64, ..., l + 64 (V - 1), and virtual lane vl owns items vl, vl + P,
// vl + 2P, ... (Section 3.2, parallel form).  A round reads V blocks of 64 edges at once,
// so a long row is scanned with V times the reads in flight.  Results, `trig` and `hsel`
// as for rvs_step; the lane's best virtual lane (larger index wins ties) then enters the
// wave's argmax.
template <int KIND, bool W, int V, bool EARLY>
__device__ __forceinline__ int32_t rvs_step_hub(const WalkArgs &a, const QueryDev &Q, const Mem &mem, uint32_t wid,
                                            int j, int32_t prev, int64_t base, int64_t deg, uint8_t want,
                                            const StepW &sw, uint32_t &trig, float &hsel, bool merge)
{
    constexpr int P = kWave * V;
    const int lane = lane_id();
    const uint32_t k0 = Q.key0, k1 = Q.key1;
    float key[V], thr[V], T[V], S[V];
    int32_t bi[V];
    int64_t mlo = 0;  // merge cursor in N(prev)
    // round 0: virtual lane vl keys neighbour vl, k = u^(1/w~) kept as log(u) / w~
    uint2 e0[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int64_t l = lane + kWave * v;
        e0[v] = l < deg ? edge_rec(a, base + l) : make_uint2(0u, 0u);
    }
    float kmax = -INFINITY;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int64_t l = lane + kWave * v;
        const bool memv = merge && merge_member_t<EARLY>(mem, (int32_t)e0[v].x, l < deg, mlo);
        key[v] = -INFINITY;
        bi[v] = -1;
        T[v] = 0.5f;  // holds the threshold draw until lkg is known
        if (l < deg) {
            const float wt = merge ? weight_of_member<KIND, W>(e0[v], j, prev, memv, sw)
                                   : edge_weight<KIND, W>(a, Q, base + l, e0[v], j, prev, mem, want, sw);
            const U4 x = philox(wid, (uint32_t)j, (uint32_t)l, 1u, k0, k1);
            key[v] = wt > 0.0f ? ln_f(unit_uniform(x.x0)) / wt : -INFINITY;
            T[v] = unit_uniform(x.x1);
            bi[v] = (int32_t)l;
        }
        kmax = fmaxf(kmax, key[v]);
    }
    const float lkg = wave_max(kmax);
#pragma unroll
    for (int v = 0; v < V; ++v) {
        thr[v] = lkg;
        T[v] = (lkg == -INFINITY) ? 0.0f : (lkg >= 0.0f ? INFINITY : ln_f(T[v]) / lkg);
        S[v] = 0.0f;
    }
    uint32_t nt = 0;
    // scan: a key is drawn only where a virtual lane's running weight passes its skip
    // threshold T = log(r) / log(k_thr)
    for (int64_t i0 = P; i0 < deg; i0 += P) {
        bool drew = false;
        uint2 ei[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int64_t i = i0 + lane + kWave * v;
            ei[v] = i < deg ? edge_rec(a, base + i) : make_uint2(0u, 0u);
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int64_t i = i0 + lane + kWave * v;
            const bool memi = merge && merge_member_t<EARLY>(mem, (int32_t)ei[v].x, i < deg, mlo);
            if (i < deg) {
                const float wt = merge ? weight_of_member<KIND, W>(ei[v], j, prev, memi, sw)
                                       : edge_weight<KIND, W>(a, Q, base + i, ei[v], j, prev, mem, want, sw);
                S[v] = S[v] + wt;
                if (S[v] > T[v]) {
                    // key conditioned to beat thr: log u' = log1p(expm1(w~ * thr) * V)
                    const U4 x = philox(wid, (uint32_t)j, (uint32_t)i, 1u, k0, k1);
                    const float av = wt * thr[v];
                    const float m1 = expm1_f(av);
                    const float z = m1 * unit_uniform(x.x0);
                    const float lg = log1p_f(z);
                    key[v] = lg / wt;
                    bi[v] = (int32_t)i;
                    thr[v] = key[v];
                    S[v] = 0.0f;
                    T[v] = thr[v] >= 0.0f ? INFINITY : ln_f(unit_uniform(x.x1)) / thr[v];
                    ++nt;
                    drew = true;
                }
            }
        }
        if (a.rvs_share && __ballot(drew) != 0) {
            float tm = thr[0];
#pragma unroll
            for (int v = 1; v < V; ++v) tm = fmaxf(tm, thr[v]);
            const float g = wave_max(tm);
#pragma unroll
            for (int v = 0; v < V; ++v) take_shared_threshold(thr[v], T[v], S[v], g);
        }
    }
    float key0 = key[0];
    int32_t bi0 = bi[0];
#pragma unroll
    for (int v = 1; v < V; ++v)
        if (key[v] > key0 || (key[v] == key0 && bi[v] > bi0)) {
            key0 = key[v];
            bi0 = bi[v];
        }
    float &keyb = key0;
    int32_t &bib = bi0;
    wave_argmax(keyb, bib);
    trig = (uint32_t)wave_sum_u64(nt);
    if (!(keyb > -INFINITY)) return -1;
    const uint2 e = edge_rec(a, base + bib);
    hsel = W ? __uint_as_float(e.y) : 1.0f;
    return (int32_t)e.x;
}

// eRVS for up to 64/G steps at once, one G-lane group per step, for rows of at most G
// neighbours.  Such a step is decided by round 0 alone (every neighbour gets its key,
// there is nothing to scan), so the result equals the one-wave eRVS bit for bit.
// Takes its steps from `pool` (lanes in trial order of the ballot) and returns true
// for the lanes that were served, with the next vertex (or -1) in `res` and the h of
// the chosen edge in `hres`.
template <int KIND, bool W, bool BATCH>
__device__ __forceinline__ bool rvs_group_pass(const WalkArgs &a, int G, uint64_t &pool, int32_t q, int32_t wid,
                                               int32_t j, int32_t prev, int64_t base, int32_t deg, int64_t pbase,
                                               int32_t pdeg, uint8_t want, int32_t &res, float &hres)
{
    const int lane = lane_id();
    const int g = lane / G, r = lane % G;
    int src_of_group = -1, my_slot = -1;
    for (int s = 0; s < kWave / G; ++s) {
        int src = -1;
        if (pool != 0) {
            src = __ffsll((unsigned long long)pool) - 1;
            pool &= pool - 1;
        }
        if (g == s) src_of_group = src;
        if (lane == src) my_slot = s;
    }
    // every lane takes part in every shuffle: a step's owner may sit in a group that
    // serves nothing this pass, and a lane reading from an inactive lane gets garbage
    const int sl = src_of_group < 0 ? lane : src_of_group;
    const int32_t s_q = BATCH ? __shfl(q, sl, kWave) : 0;
    const uint32_t s_wid = (uint32_t)__shfl(wid, sl, kWave);
    const int32_t s_j = __shfl(j, sl, kWave);
    const int32_t s_prev = __shfl(prev, sl, kWave);
    const int64_t s_base = __shfl((long long)base, sl, kWave);
    const int32_t deg_of_src = __shfl(deg, sl, kWave);
    const int64_t s_pbase = __shfl((long long)pbase, sl, kWave);
    const int32_t s_pdeg = __shfl(pdeg, sl, kWave);
    const uint8_t s_want = KIND == kMetaPath ? (uint8_t)__shfl((int)want, sl, kWave) : (uint8_t)0;
    const int32_t s_deg = src_of_group < 0 ? 0 : deg_of_src;
    float key = -INFINITY;
    int32_t bi = -1;
    uint2 e = make_uint2(0u, 0u);
    if (r < s_deg) {
        const QueryDev &Q = query<BATCH>(a, s_q);
        const int64_t k = s_base + r;
        const Mem m = {a.col + s_pbase, s_pdeg, false, false};
        const StepW sw = step_weights<KIND>(Q, s_deg, s_pdeg);
        e = edge_rec(a, k);
        const float wt = edge_weight<KIND, W>(a, Q, k, e, s_j, s_prev, m, s_want, sw);
        const U4 x = philox(s_wid, (uint32_t)s_j, (uint32_t)r, 1u, Q.key0, Q.key1);
        key = wt > 0.0f ? ln_f(unit_uniform(x.x0)) / wt : -INFINITY;
        bi = r;
    }
    for (int o = G / 2; o > 0; o >>= 1) {
        const float k2 = __shfl_xor(key, o, kWave);
        const int32_t i2 = __shfl_xor(bi, o, kWave);
        if (k2 > key || (k2 == key && i2 > bi)) {
            key = k2;
            bi = i2;
        }
    }
    // the winner's edge from its lane of the group
    const int win = g * G + (key > -INFINITY ? bi : 0);
    const int32_t wx = __shfl((int32_t)e.x, win, kWave), wh = __shfl((int32_t)e.y, win, kWave);
    const int from = my_slot >= 0 ? my_slot * G : lane;
    const int32_t got = __shfl(key > -INFINITY ? wx : -1, from, kWave);
    const uint32_t got_h = (uint32_t)__shfl(wh, from, kWave);
    if (my_slot >= 0) {
        res = got;
        hres = W ? __uint_as_float(got_h) : 1.0f;
    }
    return my_slot >= 0;
}

// A wave's counters summed over its lanes and cleared: lane c gets counter c (lanes from kNumStats
// on 0).
__device__ __forceinline__ uint64_t take_stats(uint32_t (&cnt)[kStBytes], uint64_t &bytes)
{
    int lane = lane_id();
    asm volatile("" : "+v"(lane));  // the masks of the comparisons below are not kept across the walk
    uint64_t mine = 0;
#pragma unroll
    for (int c = 0; c < kStBytes; ++c) {
        const uint64_t v = wave_sum_u64(cnt[c]);
        mine = lane == c ? v : mine;
        cnt[c] = 0;
    }
    const uint64_t b = wave_sum_u64(bytes);
    mine = lane == kStBytes ? b : mine;
    bytes = 0;
    return mine;
}

// Adds counters (lane c holds counter c) to the device totals, which share one line: one request.
__device__ __forceinline__ void add_stats(const WalkArgs &a, uint64_t mine)
{
    const int lane = lane_id();
    if (lane < kNumStats && mine != 0) atomicAdd(&a.stats[lane], (unsigned long long)mine);
}

// Adds a wave's counters to the device totals, one after the other, and clears them.
__device__ __forceinline__ void flush_stats(const WalkArgs &a, uint32_t (&cnt)[kStBytes], uint64_t &bytes)
{
    const int lane = lane_id();
#pragma unroll
    for (int c = 0; c < kStBytes; ++c) {
        const uint64_t v = wave_sum_u64(cnt[c]);
        if (lane == 0 && v != 0) atomicAdd(&a.stats[c], (unsigned long long)v);
        cnt[c] = 0;
    }
    const uint64_t b = wave_sum_u64(bytes);
    if (lane == 0 && b != 0) atomicAdd(&a.stats[kStBytes], (unsigned long long)b);
    bytes = 0;
}

// The same once per block, at the kernel's end: sums is LDS for the block, kNumStats words per wave
// at `stride` words.  Every thread of the block calls.  The totals take about 120 M requests a
// second and a short launch spreads over thousands of waves: with an add per wave and counter
// 60000 MetaPath walkers x 1 step took 322 us with counters (42 without), now 49.
__device__ __forceinline__ void flush_stats_block(const WalkArgs &a, uint32_t (&cnt)[kStBytes], uint64_t &bytes,
                                                  uint64_t *sums, int stride)
{
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    const uint64_t mine = take_stats(cnt, bytes);
    if (lane < kNumStats) sums[wave * stride + lane] = mine;
    __syncthreads();
    if (wave == 0) {
        uint64_t total = 0;
        for (int w = 0; w < kWavesPerBlock; ++w) total += lane < kNumStats ? sums[w * stride + lane] : 0;
        add_stats(a, total);
    }
}

}  // namespace fw
