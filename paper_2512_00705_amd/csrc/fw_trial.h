// walk_kernel: the runtime kernel of FlexiWalker (arXiv 2512.00705, Section 5, "Concurrent
// Rejection and Reservoir Sampling" and "Dynamic Query Scheduling") for wave64.
//
// Every lane owns one walker and is a small state machine: in each pass of the loop a lane
// consumes the random read it issued in the pass before (a proposal, a start, label bounds),
// decides what follows from it, and issues its next one.  Lanes of a wave need not be at the
// same step or trial, so a lane whose trial was rejected delays nobody.  Open membership tests
// and vertex records that no proposal brought along are read within the pass.  A pass takes
// about 400 vector instructions for a trial of each lane; deciding a whole step per pass (three
// proposals loaded ahead and decided in turn, the slowest of 64 lanes setting the pass) took
// 1300 and up to six dependent round trips.
// Large launches are bound by random reads beyond L2, which cost a 128-byte line each: 49.7 G/s
// on this device, 42 beside the walk's writes (scale-22 Node2Vec job: 2.2 reads a step, 15.3 ->
// 10.7 ms, 39 G reads/s).  Small launches and graphs that stay in L2 are bound by the
// instructions of their passes.
//
// Steps that need eRVS (Section 3.2) wait in their lanes; the whole wave serves them, short
// rows in groups of 8/16/32 lanes and longer rows one at a time.
#pragma once

#include <algorithm>

#include "fw_lds.h"
#include "fw_walk.h"

namespace fw {

// What a lane waits for: an identifier and, in the low three bits, the 16-byte parts of its read.
enum Op : int {
    kNone = 0,          // no walker
    kStart = 1 << 3,    // the walker's start vertex (4 bytes, on its own)
    kTrial = 2 << 3,    // (within a pass) a proposal to draw
    kRvs = 3 << 3,      // eRVS by the whole wave
    kDead = 4 << 3,     // no neighbour of positive weight: the walk ends
    kMany = 13 << 3,    // many rejected trials: the next ones by the whole wave
    kRet = 5 << 3,      // accepted return edge (nothing to read: prev's record is kept)
    kVrec = 6 << 3 | 1, // cur's vertex record
    kCol = 7 << 3 | 1,  // member trial: a neighbour of prev
    kColR = 7 << 3 | 4, // the same through prev's proposal record, which also has its vertex record
    kGroup = 8 << 3,    // label groups: the wanted group's bounds (1 or 2 parts)
    kEdge = 9 << 3 | 1, // uniform proposal: an edge record
    kRec = 10 << 3 | 4  // proposal record
};

// What a pass decides for a lane.
enum Res : int {
    kNothing = 0,
    kRej,    // the trial is rejected
    kLook,   // its test needs a lookup
    kFin,    // the walk is over after j steps
    kPad,    // the same, early: the rest of its path is -1
    kSetup,  // cur's vertex record has arrived
    kAcc,    // the step takes cu, whose vertex record is not read yet,
    kAccR,   // ... is at rp
    kAccP    // ... is prev's
};

// Starts the reads of a pass: lane l wants np 16-byte parts (0..4) from p (aligned to 16).  In
// round i the four lanes of each quad fetch the parts of the quad's lane i by LDS DMA, so that
// the wave asks for each line once: four 16-byte loads by the lane itself are four requests
// with an address translation each, and translations beyond the CU's small first-level TLB
// are slow: random 64-byte records come at 21 G/s with four loads per lane and at 49.7 G/s this
// way, the rate of random 8-byte reads (8 GiB of records; already with one wave per SIMD).
// Every lane calls.
__device__ __forceinline__ void issue_reads(const uint4 *p, uint32_t np, uint4 *buf)
{
    const uint64_t ad = reinterpret_cast<uint64_t>(p);
    // (np rides in the low bits of the address; that of a start vertex, read elsewhere with np =
    // 0, is aligned to 4 bytes only)
    const uint32_t lo = ((uint32_t)ad & ~15u) | np, hi = (uint32_t)(ad >> 32);
    const uint32_t part = threadIdx.x & 3u;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the last pass's slots have been read
#define FW_ROUND(i)                                                                                            \
    {                                                                                                          \
        const uint32_t l = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, 0x55 * (i), 0xf, 0xf, false);     \
        const uint32_t h = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, 0x55 * (i), 0xf, 0xf, false);     \
        if (part < (l & 15u))                                                                                  \
            __builtin_amdgcn_global_load_lds(                                                                  \
                reinterpret_cast<const uint4 *>(((uint64_t)h << 32) | (uint64_t)(l & ~15u)) + part,            \
                lds_ptr(buf + (i) * kBufStride), 16, 0, 0);                                                    \
    }
    FW_ROUND(0)
    FW_ROUND(1)
    FW_ROUND(2)
    FW_ROUND(3)
#undef FW_ROUND
}

__device__ __forceinline__ uint32_t part_pos(const int32_t *ad) { return ((uint32_t)(uintptr_t)ad >> 2) & (kPart - 1); }

// A value loaded off the pipelined path (rare branches): waited for on the spot, so that no
// wait for it, which would also wait for the path stores, is left behind the branch.
template <typename T>
__device__ __forceinline__ T now(T x)
{
    static_assert(sizeof(T) == 4, "one register");
    asm volatile("" : "+v"(x));
    return x;
}

// The argument block read anew through its address (WalkArgs is the kernels' only argument):
// what only rare branches need holds no scalar registers across the loop.
using ArgBlock = const __attribute__((address_space(4))) WalkArgs;
__device__ __forceinline__ ArgBlock *rare_args()
{
    ArgBlock *p = (ArgBlock *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

__device__ __forceinline__ int64_t row_start_now(const WalkArgs &a, uint32_t lo, int32_t v)
{
    uint32_t hi = 0;
    if (a.start_hi) hi = now(a.start_hi[v]);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// eRVS for every lane with `mine`: short rows in groups of 8/16/32 lanes, several steps per
// pass; longer rows one at a time with the whole wave (every lane calls).
struct RvsServed {
    int32_t next;  // the next vertex, or -1 when no neighbour has positive weight
    float h;       // h of the chosen edge
    uint32_t trig; // jump events
};

template <int KIND, bool W, bool BATCH, int EV>
__device__ __forceinline__ RvsServed rvs_serve(const WalkArgs &a, int32_t *lds, bool mine, int32_t q, int32_t wid,
                                               int32_t j, int32_t prev, int64_t base, int32_t deg, int64_t pbase,
                                               int32_t pdeg, uint32_t want)
{
    constexpr bool kMem = uses_membership(KIND);
    const int lane = lane_id();
    uint64_t s8 = __ballot(mine && deg <= 8);
    uint64_t s16 = __ballot(mine && deg > 8 && deg <= 16);
    uint64_t s32 = __ballot(mine && deg > 16 && deg <= 32);
    uint64_t big = __ballot(mine && deg > 32);
    if (__popcll(s8) <= 4) {
        s16 |= s8;
        s8 = 0;
    }
    if (__popcll(s16) <= 2) {
        s32 |= s16;
        s16 = 0;
    }
    RvsServed out = {-1, 1.0f, 0u};
    int32_t res = -1;
    float hres = 1.0f;
    for (int G = 8; G <= 32; G <<= 1) {
        uint64_t pool = G == 8 ? s8 : (G == 16 ? s16 : s32);
        while (pool != 0)
            if (rvs_group_pass<KIND, W, BATCH>(a, G, pool, q, wid, j, prev, base, deg, pbase, pdeg, (uint8_t)want, res,
                                               hres)) {
                out.next = res;
                out.h = hres;
            }
    }
    while (big != 0) {
        const int src = __ffsll((unsigned long long)big) - 1;
        big &= big - 1;
        const int32_t s_q = BATCH ? bcast_i32(q, src) : 0;
        const uint32_t s_wid = bcast_u32((uint32_t)wid, src);
        const int32_t s_j = bcast_i32(j, src);
        const int32_t s_prev = bcast_i32(prev, src);
        const int64_t s_base = bcast_i64(base, src);
        const int32_t s_deg = bcast_i32(deg, src);
        const int64_t s_pbase = bcast_i64(pbase, src);
        const int32_t s_pdeg = bcast_i32(pdeg, src);
        const uint8_t s_want = KIND == kMetaPath ? (uint8_t)bcast_u32(want, src) : (uint8_t)0;
        const QueryDev &Q = query<BATCH>(a, s_q);
        const bool member_test = kMem && s_j > 0;
        Mem m = {a.col + s_pbase, s_pdeg, false, false};
        // merge the rows when N(prev) is not much longer than the row scanned
        const bool merge = member_test && (int64_t)s_pdeg <= (int64_t)kMergeRatio * s_deg;
        // stage N(prev) in LDS for the merge (its reads become LDS reads), or for the
        // per-item searches when they would read more than the staging
        if (member_test && s_pdeg <= a.lds_cap && (merge || (int64_t)s_pdeg <= (int64_t)s_deg * probes(s_pdeg))) {
            wave_lds_sync();
            for (int32_t i = lane; i < s_pdeg; i += kWave) lds[i] = a.col[s_pbase + i];
            wave_lds_sync();
            m.p = lds;
            m.staged = true;
        }
        uint32_t trig = 0;
        const StepW sw = step_weights<KIND>(Q, s_deg, s_pdeg);
        // P = 64 lanes, or 128 or 256 on a row of degree >= hub_deg
        if (EV == kEvHub && s_deg >= a.hub_deg)
            res = a.hub_v == 4 ? rvs_step_hub<KIND, W, 4, false>(a, Q, m, s_wid, s_j, s_prev, s_base, s_deg, s_want,
                                                                 sw, trig, hres, merge)
                               : rvs_step_hub<KIND, W, 2, false>(a, Q, m, s_wid, s_j, s_prev, s_base, s_deg, s_want,
                                                                 sw, trig, hres, merge);
        else
            res = rvs_step<KIND, W, true>(a, Q, m, s_wid, s_j, s_prev, s_base, s_deg, s_want, sw, trig, hres, merge);
        if (lane == src) out = {res, hres, trig};
    }
    return out;
}

// Also used to keep a wave-uniform value in a vector register (scalar ones are short).
__device__ __forceinline__ int64_t now64(int64_t x)
{
    const uint32_t lo = now((uint32_t)(uint64_t)x), hi = now((uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Trials t, t + 1, ... of one step (up to 64, up to the trial cap), one per lane: the first
// accepted one is the sample, as when they run one by one.  A step whose bound is loose (the
// paper's for second-order PageRank reaches the trial cap of 1024 here and there) would else
// hold its walker, and at the end the launch, for a pass per trial (24 walkers of 6 steps on
// that bound: 1200 us with three trials at a time, 75 us so).  The wave turns to it after as
// many rejections as half its walkers, since they wait meanwhile.  Every lane calls with the
// same arguments.
struct ManyStep {
    uint32_t wid, k0, k1;
    int32_t j, cur, prev;
    int64_t base, pbase;
    int32_t deg, pdeg;
    uint32_t want;
    float B, area, bE, bZ, hm, wp, wlo, whi, wm, wo;
    bool counted;  // regular trials count the bytes of a membership search
};
struct ManyDone {
    int kind;   // 0: none accepted, 1: u with weight h, 2: the return edge's column
    int32_t u;
    float h;
    int32_t n;  // trials taken
    uint64_t bytes;
};

// edge_rec through the argument block.
__device__ __forceinline__ void edge_of(ArgBlock &a, int64_t k, int32_t &u, float &h)
{
    if (a.erec8 != nullptr) {
        const uint32_t e = a.erec8[k];
        u = (int32_t)(e & 0xFFFFFFu);
        h = (float)(e >> 24) * a.h_scale;
    } else {
        const uint2 e = a.edges[k];
        u = (int32_t)e.x;
        h = __uint_as_float(e.y);
    }
}

template <int KIND, bool W, bool HPROP, bool STATS>
__device__ __forceinline__ ManyDone many_trials(ArgBlock &a, const ManyStep &m, int32_t t0)
{
    constexpr bool kMem = uses_membership(KIND);
    const int lane = lane_id();
    const int cnt = min(kWave, a.rjs_cap - t0);
    const bool mine = lane < cnt;
    const U4 x = philox(m.wid, (uint32_t)m.j, (uint32_t)(t0 + lane), 0u, m.k0, m.k1);
    const float z = unit_uniform(x.x3) * m.area;
    const bool ol = KIND == kNode2Vec && m.bE > 0.0f && z < m.bE;
    const bool mr = kMem && !ol && z < m.bZ;
    const int32_t n = mr ? m.pdeg : m.deg;
    const uint64_t tt = (uint64_t)x.x1 * (uint32_t)n + (((uint64_t)x.x0 * (uint32_t)n) >> 32);
    const int64_t k = (mr ? m.pbase : m.base) + (int64_t)(tt >> 32);
    int32_t u = m.prev;
    float h = 1.0f;
    bool acc = ol, open = false;
    if (mine && !ol) {
        uint32_t lb = 0;
        if (kMem && mr) {
            u = a.col[k];
            open = u != m.prev;
        } else {
            if (HPROP) {
                const uint4 r0 = a.prop[kPropU4 * k], r1 = a.prop[kPropU4 * k + 1];
                const bool keep = (uint32_t)tt < r1.x;
                u = (int32_t)(keep ? r0.x : r0.z);
                h = W ? __uint_as_float(keep ? r0.y : r0.w) : 1.0f;
                lb = (keep ? r1.y : r1.y >> 8) & 0xFFu;
            } else {
                edge_of(a, k, u, h);
                if (!W) h = 1.0f;
                if (KIND == kMetaPath) lb = a.label[k];
            }
            const float hw = HPROP ? 1.0f : h;
            const float y = unit_uniform(x.x2) * m.B;
            if (kMem) {
                const bool is_prev = u == m.prev;
                acc = y < (is_prev ? m.wp : m.wlo) * hw;
                open = !acc && !is_prev && y < m.whi * hw;
            } else {
                acc = y < (lb == m.want ? hw : 0.0f);
            }
        }
    }
    // look up the open tests before the first sure acceptance
    const uint64_t sure = __ballot(mine && acc);
    if (kMem) {
        open = open && (sure == 0 || lane < __ffsll((unsigned long long)sure) - 1);
        if (open) {
            float hx = 1.0f;
            bool found;
            const int32_t lv = mr ? m.cur : m.prev;
            if (a.mtab != nullptr) {
                found = index_find(a.mtab, a.mtab_mask, lv, u, hx);
            } else {
                const int64_t rb = mr ? m.base : m.pbase;
                const int32_t pos = sorted_find_interp(a.col + rb, mr ? m.deg : m.pdeg, u, (int32_t)a.nv);
                found = pos >= 0;
                int32_t same;
                if (mr && W && found) edge_of(a, rb + pos, same, hx);
            }
            if (mr) {
                h = W ? hx : 1.0f;
                acc = found && unit_uniform(x.x2) * m.hm < h;
            } else {
                const float hw = HPROP ? 1.0f : h;
                acc = unit_uniform(x.x2) * m.B < (found ? m.wm * hw : m.wo * hw);
            }
        }
    }
    const uint64_t accepted = __ballot(mine && acc);
    const int first = accepted != 0 ? __ffsll((unsigned long long)accepted) - 1 : cnt - 1;
    ManyDone d = {0, 0, 1.0f, first + 1, 0};
    if (accepted != 0) {
        d.kind = bcast_i32(ol ? 2 : 1, first);
        d.u = bcast_i32(u, first);
        d.h = bcast_f32(h, first);
    }
    if (STATS) {
        uint64_t by = 0;
        if (lane <= first && !ol)
            by = mr ? 4 + 4 * (uint64_t)probes(m.deg) + (W ? 4 : 0)
                    : (uint64_t)a.item_bytes + (HPROP ? 12 : 0) + (m.counted ? 4 * (uint64_t)probes(m.pdeg) : 0);
        d.bytes = wave_sum_u64(by);
    }
    return d;
}

constexpr int kAgainMost = 3, kAgainShare = 2;  // see walk_kernel's redraws

template <int KIND, bool W, int PROP, bool BATCH, bool STATS, int EV>
__global__ void __launch_bounds__(kBlock, trial_waves(EV)) walk_kernel(WalkArgs a)
{
    constexpr bool kMem = uses_membership(KIND);
    constexpr bool kLab = KIND == kMetaPath && PROP == 2;   // label-conditioned proposals
    constexpr bool kHprop = (W && PROP != 0) || kLab;       // proposals from records
    constexpr bool kStash = trial_stash(KIND, PROP);
    if (EV == kEvHot && a.resume && *a.parked == 0) return;  // nothing was parked
    extern __shared__ __attribute__((aligned(16))) int32_t lds_all[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    uint4 *buf = reinterpret_cast<uint4 *>(lds_all) + wave * kBufU4;
    const uint4 *slot = buf + (threadIdx.x & 3u) * kBufStride + ((threadIdx.x & (kWave - 1)) >> 2) * 4;
    uint4 *stash = reinterpret_cast<uint4 *>(lds_all) + kWavesPerBlock * kBufU4 + (kStash ? wave * kWave : 0);
    int32_t *parts = lds_all + kWavesPerBlock * (kBufU4 + (kStash ? kWave : 0)) * 4 + wave * kWave * kPart;
    int32_t *lds_aux = lds_all + kWavesPerBlock * ((kBufU4 + (kStash ? kWave : 0)) * 4 + kWave * kPart);
    int32_t *lds = lds_aux + (BATCH ? kQueryTop * 2 : (KIND == kMetaPath ? 16 : 0)) + wave * (kMem ? a.lds_cap : 0);
    const int lane = lane_id();
    const uint64_t below = lanes_below(lane);

    // the schema (one query) or every stride-th query's first walker (a batch) in LDS
    const uint8_t *schema = reinterpret_cast<const uint8_t *>(lds_aux);
    int64_t *qtop = reinterpret_cast<int64_t *>(lds_aux);
    const int32_t qstride = BATCH ? (a.nq + kQueryTop - 1) / kQueryTop : 1;
    if (BATCH) {
        for (int32_t t = threadIdx.x; t < kQueryTop; t += kBlock) {
            const int64_t e = (int64_t)t * qstride;
            qtop[t] = e < a.nq ? a.queries[e].first : INT64_MAX;
        }
        __syncthreads();
    } else if (KIND == kMetaPath) {
        if (threadIdx.x < 64) reinterpret_cast<uint8_t *>(lds_aux)[threadIdx.x] = a.q0.schema[threadIdx.x];
        __syncthreads();
    }

    int op = kNone;
    const uint4 *p = nullptr;  // address of the lane's read in flight
    int32_t sv = 0;            // kStart: the start vertex
    uint32_t elab = 0;  // uniform MetaPath proposal: the edge's label
    int32_t q = 0;      // query of the lane's walker
    int32_t wid = 0;    // walker index within its query (n < 2^31)
    int32_t *row = nullptr;  // its path
    int32_t cur = 0, prev = -1, j = 0;
    int64_t base = 0, pbase = 0;  // row starts of cur and prev (label groups: pbase, pdeg hold the group)
    int32_t deg = 0, pdeg = 0;
    float hm = 1.0f, hs = 0.0f, phm = 1.0f, phs = 0.0f;  // h_MAX and h_SUM of cur and prev
    int32_t trials = 0;
    int32_t stop_j = 0;  // resumable walks: suspend when j reaches this step
    bool fell_back = false;
    bool force = false;  // a parked walk's first step: eRVS
    bool mb = false;     // the step uses the member board (counted bytes only)
    // eRJS board of the step: the test's height B, the return column [0, bE) and member region
    // [bE, bZ) of U * area; the weight of a proposal of prev, the smallest and largest weight of
    // any other (equal when the test needs no membership)
    float B = 0.0f, area = 0.0f, bE = 0.0f, bZ = 0.0f, wp = 1.0f, wlo = 1.0f, whi = 1.0f;
    float wmem = 1.0f, woth = 1.0f;  // second-order PageRank: the step's two weights
    uint32_t ux = 0, aux = 0;        // the trial's test draw; its coin, or which part of the 16 bytes it proposed
    int32_t cu = 0;                  // the trial's candidate and its h
    float ch = 1.0f;
    float hlast = 1.0f;              // h of the edge prev -> cur; on a symmetric graph also h(cur, prev)
    int32_t jm = 0;                  // MetaPath: j mod schema length, the wanted label, the next one
    uint32_t want = 0, want_next = 0;
    // constants of a batched walker's query
    uint32_t bk0 = 0, bk1 = 0;
    float bw0 = 0.0f, bw1 = 0.0f, bavg = 0.0f;
    int32_t bL = 0, blen = 1;
    uint32_t st[kStBytes];
#pragma unroll
    for (int c = 0; c < kStBytes; ++c) st[c] = 0;
    uint64_t st_bytes = 0;

    // The walkers that the wave hands to its lanes: [wnext, wend).  It starts with a share of its
    // own of the first static_n walkers (all of them when the lanes hold the launch, so that few
    // walkers spread over all waves) and then fetches chunks of the others from the counter.
    // All waves add to one address, which takes about 120 M adds a second: with an atomic for
    // each pass in which some lane had finished, the scale-22 job took 32 ms instead of 12.
    // Chunks shrink with what is left, so that no wave holds walkers that another could start.
    // Only waves that are resident from the start (static_waves) have a share.
    const int64_t wv = (int64_t)blockIdx.x * kWavesPerBlock + wave;
    int64_t wnext = 0, wend = 0;
    if (wv < a.static_waves) {
        wnext = wv * a.static_each + min(wv, a.static_more);
        wend = wnext + a.static_each + (wv < a.static_more ? 1 : 0);
    }
    int64_t left = a.n - a.static_n;  // not yet handed to any wave, when last seen
    bool exhausted = left <= 0;
    unsigned long long qfirst = 0;  // lane 0: the counter's value when a chunk of qcnt was asked for
    int qcnt = 0;
    const int gshift = 65 - __builtin_clzll((unsigned long long)gridDim.x * kWavesPerBlock);  // left / 2-4 x the waves
    int64_t w0 = -1;  // walker handed to the lane in this pass

    auto Lq = [&]() -> int32_t { return BATCH ? bL : a.q0.L; };
    auto key0 = [&]() -> uint32_t { return BATCH ? bk0 : a.q0.key0; };
    auto key1 = [&]() -> uint32_t { return BATCH ? bk1 : a.q0.key1; };
    auto invp = [&]() -> float { return BATCH ? bw0 : a.q0.inv_p; };
    auto invq = [&]() -> float { return BATCH ? bw1 : a.q0.inv_q; };
    for (;;) {
        if (STATS && __ballot((st[kStTrials] | st[kStTriggers] | st[kStSteps]) > 0x40000000u) != 0)
            flush_stats(a, st, st_bytes);

        // 1. consume the read that arrived
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        int was = op;
        int res = kNothing;
        bool flush = false;  // the part of the path that ends with slot j goes out in this pass
        // The cases below are tests of their own, not one chain: a chain becomes a tree of
        // branches whose merges copy every value that some case sets (a quarter of the loop's
        // vector instructions).  This keeps the compiler from joining them.
        auto apart = [&]() { asm volatile("" : "+v"(was), "+v"(res)); };
        const uint4 *rp = slot;  // the vertex record of cur (kSetup) or of the accepted candidate (kAccR)
        const float wm = KIND == kSecondPR ? wmem : 1.0f;
        const float wo = KIND == kSecondPR ? woth : invq();
        if (was == (kHprop ? (int)kRec : (int)kEdge)) {
            uint32_t lb = 0;
            if (kHprop) {
                const uint4 x0 = slot[0], x1 = slot[1];
                const bool keep = aux < x1.x;
                cu = (int32_t)(keep ? x0.x : x0.z);
                ch = W ? __uint_as_float(keep ? x0.y : x0.w) : 1.0f;
                rp = slot + (keep ? 2 : 3);
                if (KIND == kMetaPath) lb = (keep ? x1.y : x1.y >> 8) & 0xFFu;
            } else {
                if (a.erec8 != nullptr) {
                    const uint32_t e = reinterpret_cast<const uint32_t *>(slot)[aux];
                    cu = (int32_t)(e & 0xFFFFFFu);
                    ch = W ? (float)(e >> 24) * a.h_scale : 1.0f;
                } else {
                    const uint2 e = reinterpret_cast<const uint2 *>(slot)[aux];
                    cu = (int32_t)e.x;
                    ch = W ? __uint_as_float(e.y) : 1.0f;
                }
                lb = elab;
            }
            if (STATS)
                st_bytes += (uint64_t)a.item_bytes + (kHprop ? 12 : 0) +
                            ((kMem && j > 0 && !mb) ? 4 * (uint64_t)probes(pdeg) : 0);
            const float hw = kHprop ? 1.0f : ch;  // the test is on w~ (uniform) or w (h-proportional)
            const float y = unit_uniform(ux) * B;
            if (kMem) {
                const bool is_prev = cu == prev;
                res = y < (is_prev ? wp : wlo) * hw ? (kHprop ? kAccR : kAcc) : !is_prev && y < whi * hw ? kLook : kRej;
                if (kStash && res == kLook) stash[lane] = *rp;
            } else if (kLab) {
                // a proposal of weight 0 from a label group: the group's weights are all 0
                res = ch > 0.0f ? kAccR : kPad;
                if (STATS && res == kPad) st[kStEarly] += 1;
            } else {
                res = y < (lb == want ? hw : 0.0f) ? (kHprop ? kAccR : kAcc) : kRej;
            }
            if (res != kLook) {
                st[kStTrials] += 1;
                st[kStRjs] += res >= kAcc ? 1 : 0;
            }
        }
        apart();
        if (kMem) {
            if (was == (kHprop ? (int)kColR : (int)kCol)) {
                // member region: keep a neighbour u of prev when it is one of cur (not prev)
                if (kHprop) {
                    cu = (int32_t)slot[0].x;
                    stash[lane] = slot[2];
                } else {
                    cu = reinterpret_cast<const int32_t *>(slot)[aux];
                }
                if (STATS) st_bytes += 4 + 4 * (uint64_t)probes(deg) + (W ? 4 : 0);
                res = cu != prev ? kLook : kRej;
                if (res == kRej) st[kStTrials] += 1;
            }
            apart();
        }
        if (was == kVrec) res = kSetup;
        if (KIND == kNode2Vec) {
            if (was == kRet) {
                // the board's extra column belongs to the return edge
                cu = prev;
                ch = hlast;
                res = kAccP;
                st[kStTrials] += 1;
                st[kStRjs] += 1;
            }
            apart();
        }
        if (kLab) {
            if (was >= kGroup && was < kEdge) {
                const int64_t g0 = reinterpret_cast<const int64_t *>(slot)[aux];
                const int64_t g1 = reinterpret_cast<const int64_t *>(slot)[aux + 1];
                st_bytes += 8;
                if (g1 == g0) {
                    res = kPad;  // an empty group ends the walk
                    st[kStEarly] += 1;
                } else {
                    pbase = g0;
                    pdeg = (int32_t)(g1 - g0);
                    bool rjs;
                    if (a.strategy == kRjsOnly) {
                        rjs = true;
                    } else if (a.strategy == kRandomSelect) {
                        const U4 x = philox((uint32_t)wid, (uint32_t)j, 0u, 4u, key0(), key1());
                        rjs = unit_uniform(x.x0) < 0.5f;
                    } else if (a.strategy == kDegreeSelect) {
                        rjs = deg >= a.d_lo;
                    } else if (a.strategy == kRvsOnly) {
                        rjs = false;
                    } else {
                        rjs = deg >= a.d_lo && a.rho < (float)deg;  // a tie goes to eRVS
                    }
                    B = area = 1.0f;
                    op = rjs ? kTrial : kRvs;
                }
            }
            apart();
        }
        if (__ballot(was == kStart || was == kDead) != 0) {
            if (was == kStart) {
                ArgBlock *const ra = rare_args();
                const int32_t L = Lq();
                st_bytes += 12 + 4 * (uint64_t)L;
                cur = sv;
                prev = -1;
                hlast = 1.0f;
                j = 0;
                stop_j = a.tick_steps;
                parts[lane * kPart + part_pos(row)] = sv;
                flush = part_pos(row) == kPart - 1;
                if (KIND == kMetaPath) {
                    jm = 0;
                    want = BATCH ? now((uint32_t)a.queries[q].schema[0]) : schema[0];
                }
                op = kVrec;
                p = a.vrec + cur;
                if (sv < 0 || (int64_t)sv >= ra->nv) {
                    atomicOr(ra->err, 1);
                    res = kPad;
                } else if (L == 0) {
                    res = kFin;
                }
            }
            apart();
            if (was == kDead) {
                res = kPad;
                st[kStEarly] += 1;
            }
        }
        // An open membership test, and a member trial (mt), looks (prev or cur, cu) up: one bucket of the
        // edge index, or a search of the row.  In the same pass: a pass of its own would run all
        // of the pass's other parts for the lanes that have nothing to do there.
        auto look_up = [&](const bool mt) {
            const uint64_t key = edge_key(mt ? cur : prev, cu);
            bool look = res == kLook, found = false;
            float hx = 1.0f;
            if (a.mtab != nullptr) {
                uint64_t b = mix64(key) & a.mtab_mask;
                for (;;) {
                    issue_reads(a.mtab + b * kIndexBucketU4, look ? 4u : 0u, buf);
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    if (look) {
                        bool empty;
                        found = index_match(slot[0], slot[1], slot[2], slot[3], key, hx, empty);
                        look = !found && !empty;  // a full bucket without the key: on to the next
                        b = (b + 1) & a.mtab_mask;
                    }
                    if (__ballot(look) == 0) break;  // (the table always has empty slots)
                }
            } else if (look) {
                ArgBlock *const ra = rare_args();
                const int64_t rb = mt ? base : pbase;
                const int32_t pos = now(sorted_find_interp(ra->col + rb, mt ? deg : pdeg, cu, (int32_t)ra->nv));
                found = pos >= 0;
                if (mt && W && found) hx = now(__uint_as_float(edge_rec(a, rb + pos).y));
            }
            if (res == kLook) {
                // member trial: kept with probability h(cur, u) / h_MAX
                if (!W) hx = 1.0f;
                const float hw = kHprop ? 1.0f : ch;
                const float thr = mt ? (found ? hx : 0.0f) : found ? wm * hw : wo * hw;
                if (mt) ch = hx;
                res = unit_uniform(ux) * (mt ? hm : B) < thr ? (kStash ? kAccR : kAcc) : kRej;
                if (kStash) rp = stash + lane;
                st[kStTrials] += 1;
                st[kStRjs] += res >= kAcc ? 1 : 0;
            }
        };
        if (kMem && __ballot(res == kLook) != 0) look_up(was == (kHprop ? (int)kColR : (int)kCol));
        apart();
        // Serving a step by the wave costs about a pass, in which each of the other lanes could
        // have had a trial: it starts once the step has taken as many as there are lanes at work
        // (Node2Vec, p = 1/4, q = 4, 109000 x 52 at scale 18: from a quarter of the lanes 1.38 ms,
        // half 1.15, all 1.09, twice 1.08; 2nd-PageRank at scale 20: half and all 7.2 ms, twice
        // 7.6), without lookups at half (MetaPath at scale 18: 0.77 ms, all 0.83).
        const int active = __popcll(__ballot(was != kNone));
        const int many_from = max(4, kMem ? active : active / 2);
        // Rejected uniform proposals are drawn again within the pass while half of the lanes at work
        // have one: a trial takes about 100 vector instructions here, 130 more where some lane looks
        // up, and 400 in a pass, whose other parts have nothing to do for these lanes.  The others
        // wait, so at most kAgainMost times (Node2Vec, p = 1/4, q = 4, 109000 x 52 at scale 18: 1200 us
        // without, 1044, 1025, 1012 us with one, two, three; while a quarter of the lanes have one:
        // 1020 us with two, 1045 with four).  MetaPath, 100000 x 40 at scale 16: 841 -> 732 us; 61
        // walkers x 40: 138 -> 116.  Unweighted, p = 1/4, q = 4 again: 770 -> 693 us; where nothing is
        // rejected the test costs 4 % (p = q = 1, 300000 x 40 at scale 12: 245 -> 255).
        if (PROP == 0) {
            const int again_below = min(many_from, a.rjs_cap) - 1;
#pragma unroll 1
            for (int again = 0; again < kAgainMost; ++again) {
                const bool more = res == kRej && trials < again_below;
                const int rejected = __popcll(__ballot(more));
                if (rejected == 0 || kAgainShare * rejected < active) break;
                const U4 x = philox((uint32_t)wid, (uint32_t)j, (uint32_t)trials + 1u, 0u, key0(), key1());
                const float z = unit_uniform(x.x3) * area;
                const bool ol = KIND == kNode2Vec && bE > 0.0f && z < bE;
                const bool mr = kMem && !ol && z < bZ;
                if (more) {
                    ++trials;
                    ux = x.x2;
                    res = kAccP;
                    cu = prev;
                    ch = hlast;
                    const int32_t n = mr ? pdeg : deg;
                    const uint64_t t = (uint64_t)x.x1 * (uint32_t)n + (((uint64_t)x.x0 * (uint32_t)n) >> 32);
                    const int64_t k = (mr ? pbase : base) + (int64_t)(t >> 32);
                    if (mr) {
                        cu = now(a.col[k]);
                        res = cu != prev ? kLook : kRej;
                        if (STATS) st_bytes += 4 + 4 * (uint64_t)probes(deg) + (W ? 4 : 0);
                    } else if (!ol) {
                        const uint32_t lb = KIND == kMetaPath ? now((uint32_t)a.label[k]) : 0u;
                        const uint2 e = edge_rec(a, k);
                        cu = (int32_t)now(e.x);
                        ch = W ? __uint_as_float(now(e.y)) : 1.0f;
                        if (STATS)
                            st_bytes += (uint64_t)a.item_bytes + ((kMem && j > 0 && !mb) ? 4 * (uint64_t)probes(pdeg) : 0);
                        const float y = unit_uniform(ux) * B;
                        if (kMem) {
                            const bool is_prev = cu == prev;
                            res = y < (is_prev ? wp : wlo) * ch ? kAcc : !is_prev && y < whi * ch ? kLook : kRej;
                        } else {
                            res = y < (lb == want ? ch : 0.0f) ? kAcc : kRej;
                        }
                    }
                    if (res != kLook) {
                        st[kStTrials] += 1;
                        st[kStRjs] += res >= kAcc ? 1 : 0;
                    }
                }
                if (kMem && __ballot(res == kLook) != 0) look_up(mr);
            }
            apart();
        }
        if (res == kRej) {
            ++trials;
            op = !kLab && trials >= many_from ? kMany : kTrial;
            if (trials >= a.rjs_cap) {
                op = kRvs;  // exact fall-back: eRVS draws are independent of eRJS draws
                fell_back = true;
            }
        }

        // a step that has rejected many trials takes the next ones 64 at a time
        if (!kLab && __ballot(op == kMany) != 0) {
            for (uint64_t todo = __ballot(op == kMany); todo != 0; todo &= todo - 1) {
                const int src = __ffsll((unsigned long long)todo) - 1;
                ManyStep m;
                m.wid = now(bcast_u32((uint32_t)wid, src));
                m.k0 = BATCH ? bcast_u32(bk0, src) : a.q0.key0;
                m.k1 = BATCH ? bcast_u32(bk1, src) : a.q0.key1;
                m.j = now(bcast_i32(j, src));
                m.cur = now(bcast_i32(cur, src));
                m.prev = now(bcast_i32(prev, src));
                m.base = now64(bcast_i64(base, src));
                m.pbase = now64(bcast_i64(pbase, src));
                m.deg = now(bcast_i32(deg, src));
                m.pdeg = now(bcast_i32(pdeg, src));
                m.want = KIND == kMetaPath ? bcast_u32(want, src) : 0u;
                m.B = now(bcast_f32(B, src));
                m.area = now(bcast_f32(area, src));
                m.bE = now(bcast_f32(bE, src));
                m.bZ = now(bcast_f32(bZ, src));
                m.hm = now(bcast_f32(hm, src));
                m.wp = now(bcast_f32(wp, src));
                m.wlo = now(bcast_f32(wlo, src));
                m.whi = now(bcast_f32(whi, src));
                m.wm = now(bcast_f32(wm, src));
                m.wo = now(bcast_f32(wo, src));
                m.counted = kMem && m.j > 0 && bcast_i32(mb, src) == 0;
                int32_t t = bcast_i32(trials, src);
                ManyDone d;
                uint64_t by = 0;
                do {
                    d = many_trials<KIND, W, kHprop, STATS>(*rare_args(), m, t);
                    t += d.n;
                    by += d.bytes;
                } while (d.kind == 0 && t < a.rjs_cap);
                if (lane == src) {
                    st[kStTrials] += (uint32_t)(t - trials);
                    st[kStRjs] += d.kind != 0 ? 1 : 0;
                    st_bytes += by;
                    trials = t;
                    cu = d.u;
                    ch = d.kind == 2 ? hlast : d.h;
                    res = d.kind == 2 ? kAccP : d.kind == 1 ? kAcc : kNothing;
                    if (d.kind == 0) {
                        op = kRvs;
                        fell_back = true;
                    }
                }
            }
        }

        // a walker for this lane
        if (qcnt > 0) {
            wnext = bcast_i64((int64_t)qfirst, 0) + a.static_n;
            wend = min(wnext + qcnt, a.n);
            left = a.n - wend;
            exhausted = left <= 0;
            qcnt = 0;
        }
        if (wnext < wend) {
            const uint64_t idle = __ballot(was == kNone);
            if (was == kNone) {
                w0 = wnext + __popcll(idle & below);
                w0 = w0 < wend ? w0 : -1;
            }
            wnext += __popcll(idle);
        }
        if (w0 >= 0) {
            ArgBlock *const ra = rare_args();
            op = kStart;
            if (BATCH) {
                int32_t t = 0;  // last first-level entry at or below the walker, then the queries up to the next one
#pragma unroll
                for (int s = kQueryTop / 2; s > 0; s >>= 1)
                    if (qtop[t + s] <= w0) t += s;
                int32_t lo = t * qstride, hi = min(lo + qstride, ra->nq) - 1;
                while (lo < hi) {
                    const int32_t mid = (lo + hi + 1) >> 1;
                    if (ra->queries[mid].first <= w0) lo = mid;
                    else hi = mid - 1;
                }
                q = lo;
                const QueryDev &Q = ra->queries[q];
                wid = (int32_t)(w0 - Q.first);
                bk0 = Q.key0;
                bk1 = Q.key1;
                bw0 = KIND == kSecondPR ? Q.gamma : Q.inv_p;
                bw1 = KIND == kSecondPR ? Q.omg : Q.inv_q;
                bavg = Q.wavg1;
                bL = Q.L;
                blen = KIND == kMetaPath ? Q.schema_len : 1;
                asm volatile("" : "+v"(bk0), "+v"(bk1), "+v"(bw0), "+v"(bw1), "+v"(bavg), "+v"(bL), "+v"(blen));
                row = Q.paths + (int64_t)wid * ((int64_t)bL + 1);
                p = reinterpret_cast<const uint4 *>(Q.starts + wid);
            } else {
                wid = (int32_t)w0;
                row = ra->q0.paths + w0 * ((int64_t)a.q0.L + 1);
                p = reinterpret_cast<const uint4 *>(ra->q0.starts + wid);
            }
            // a suspended walk resumes after pj steps, a parked one at its step pj
            int32_t pj = 0;
            if (BATCH && ra->queries[q].prog) pj = now(ra->queries[q].prog[wid]);
            if (EV == kEvHot && ra->resume) {
                const int32_t l = now((BATCH ? ra->queries[q].lengths : ra->q0.lengths)[wid]);
                force = l < 0;
                pj = force ? -1 - l : kDone;
            }
            if (pj < 0) {
                op = kNone;  // finished in an earlier launch
            } else if (pj > 0 || (EV == kEvHot && force)) {
                // cur and prev are the last two slots the walk wrote, and prev's row is N(prev)
                j = pj;
                cur = now(row[pj]);
                prev = -1;
                hlast = 1.0f;
                if (pj > 0) {
                    prev = now(row[pj - 1]);
                    const uint4 pr = ra->vrec[prev];
                    pbase = row_start_now(a, now(pr.x), prev);
                    pdeg = (int32_t)now(pr.y);
                    phm = W ? now(__uint_as_float(pr.z)) : 1.0f;
                    phs = W ? now(__uint_as_float(pr.w)) : (float)pdeg;
                    if (KIND == kNode2Vec && W && ra->bound != 0) {
                        const int64_t pos = sorted_find(ra->col + pbase, pdeg, cur);
                        if (pos >= 0) hlast = now(__uint_as_float(edge_rec(a, pbase + pos).y));
                    }
                }
                // the slots of the part that slot pj is in are held again
                const int32_t t = (int32_t)part_pos(row + pj);
                for (int32_t k = max(0, t - pj); k <= t; ++k) parts[lane * kPart + k] = now(row[pj - t + k]);
                stop_j = pj + a.tick_steps;
                st_bytes += 4 + 8 + 16;
                if (KIND == kMetaPath) {
                    jm = pj % (BATCH ? blen : a.q0.schema_len);
                    want = BATCH ? now((uint32_t)ra->queries[q].schema[jm]) : schema[jm];
                }
                op = kVrec;
                p = a.vrec + cur;
            }
            w0 = -1;
        }

        // 2. eRVS for every lane that needs it; without the scan the walk is parked before the
        //    step, for a second launch of the kEvHot form to resume
        if (EV == kEvNone) {
            if (op == kRvs) {
                ArgBlock *const ra = rare_args();
                flush = true;
                (BATCH ? ra->queries[q].lengths : ra->q0.lengths)[wid] = -1 - j;
                *ra->parked = 1;
                op = kNone;
            }
        } else if (__ballot(op == kRvs) != 0) {
            const bool mine = op == kRvs;
            const RvsServed v =
                rvs_serve<KIND, W, BATCH, EV>(a, lds, mine, q, wid, j, prev, base, deg, pbase, pdeg, want);
            if (mine) {
                cu = v.next;
                ch = v.h;
                res = v.next >= 0 ? kAcc : kPad;
                st[kStEarly] += v.next >= 0 ? 0 : 1;
                st[kStTriggers] += v.trig;
                uint64_t by = (uint64_t)deg * (uint64_t)a.item_bytes;
                if (kMem && j > 0) {
                    const uint64_t stage = 4 * (uint64_t)pdeg;
                    const uint64_t search = 4 * (uint64_t)deg * (uint64_t)probes(pdeg);
                    by += stage < search ? stage : search;
                }
                st_bytes += by;
                if (v.next >= 0) st[fell_back ? kStFallback : kStRvs] += 1;
                force = false;
            }
        }

        // 3. apply the step (update) and write the path
        apart();
        if (res >= kAcc) {
            ++j;
            const uint32_t t = part_pos(row + j);
            parts[lane * kPart + t] = cu;
            flush = t == kPart - 1;
            st[kStSteps] += 1;
            if (KIND == kMetaPath) {
                want = want_next;
                jm = jm + 1 == (BATCH ? blen : a.q0.schema_len) ? 0 : jm + 1;
            }
            if (j == Lq()) {
                res = kFin;
            } else if (BATCH && a.tick_steps > 0 && j == stop_j) {
                flush = true;
                a.queries[q].prog[wid] = j;  // suspend until the next launch
                op = kNone;
                res = kNothing;
            }
        }
        // the wave writes the held parts that are full or at their walk's end, one after the
        // other, and the -1 slots after a walk that ended early
        const bool over = res == kFin || res == kPad;
        for (uint64_t out = __ballot(flush || over); out != 0; out &= out - 1) {
            const int src = __ffsll((unsigned long long)out) - 1;
            int32_t *const r = reinterpret_cast<int32_t *>(bcast_i64(reinterpret_cast<int64_t>(row), src));
            const int32_t jj = bcast_i32(j, src);
            const int32_t end = bcast_i32(res == kPad ? Lq() : j, src);
            const int32_t first = jj - (int32_t)part_pos(r + jj);
            for (int32_t k = lane; first + k <= end; k += kWave) {
                const int32_t v = first + k <= jj ? parts[src * kPart + (k & (kPart - 1))] : -1;
                if (first + k >= 0) r[first + k] = v;
            }
        }
        if (over) {
            ArgBlock *const ra = rare_args();
            (BATCH ? ra->queries[q].lengths : ra->q0.lengths)[wid] = j;
            if (BATCH && ra->queries[q].prog) {
                ra->queries[q].prog[wid] = kDone;
                atomicAdd(ra->queries[q].done, 1);
            }
            op = kNone;
        }

        // an accepted vertex whose record no proposal brought along is read in the same pass, too
        if (__ballot(res == kAcc) != 0) {
            issue_reads(a.vrec + cu, res == kAcc ? 1u : 0u, buf);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (res == kAcc) {
                res = kAccR;
                rp = slot;
            }
        }

        // 4. step set-up: row of cur, board, strategy (Section 4.1)
        apart();
        if (res >= kSetup) {
            // the new vertex's row start, degree, h_MAX, h_SUM
            int64_t nb = base;
            int32_t nd = deg;
            float nm = hm, ns = hs;
            if (res == kAccP) {
                nb = pbase;
                nd = pdeg;
                nm = phm;
                ns = phs;
            } else {
                const uint4 r = *rp;
                nb = row_start_now(a, r.x, res == kSetup ? cur : cu);
                nd = (int32_t)r.y;
                nm = W ? __uint_as_float(r.z) : 1.0f;
                ns = W ? __uint_as_float(r.w) : (float)nd;
            }
            if (res > kSetup) {
                prev = cur;
                cur = cu;
                hlast = ch;
                pbase = base;
                pdeg = deg;
                phm = hm;
                phs = hs;
            }
            base = nb;
            deg = nd;
            hm = nm;
            hs = ns;
            st_bytes += 16;
            trials = 0;
            fell_back = false;
            mb = false;
            if (KIND == kMetaPath) {  // the next step's label, asked for a step ahead
                const int32_t jn = jm + 1 == (BATCH ? blen : a.q0.schema_len) ? 0 : jm + 1;
                want_next = BATCH ? a.queries[q].schema[jn] : schema[jn];
            }
            op = kTrial;
            if (kLab) {
                // the wanted label's group of the row: its one proposal is the sample
                if ((int32_t)want < a.nlab) {
                    const int64_t gi = (int64_t)cur * a.nlab + want;
                    aux = (uint32_t)gi & 1u;
                    op = kGroup + 1 + (int)aux;
                    p = reinterpret_cast<const uint4 *>(a.lrow) + (gi >> 1);
                } else {
                    if (deg != 0) st_bytes += 8;
                    op = kDead;
                }
            } else if (a.strategy == kRvsOnly) {
                op = kRvs;
            } else {
                bool rjs;
                if (KIND == kSecondPR && j > 0) {
                    // in float32 in the order of Eq. (2ndpr), as step_weights
                    const float t1 = (BATCH ? bw1 : a.q0.omg) / (float)deg;
                    const float t2 = (BATCH ? bw0 : a.q0.gamma) / (float)(pdeg > 0 ? pdeg : 1);
                    const float md = (float)(deg > pdeg ? deg : pdeg);
                    wmem = (t1 + t2) * md;
                    woth = t1 * md;
                }
                const float wr = KIND == kSecondPR ? woth : invp();
                const float sm = KIND == kSecondPR ? wmem : 1.0f, so = KIND == kSecondPR ? woth : invq();
                const float smax = KIND == kSecondPR ? fmaxf(sm, so) : BATCH ? fmaxf(1.0f, so) : a.q0.hi_w;
                float wmax = 1.0f, wavg = 1.0f;  // max and mean of the workload weight
                if (KIND == kMetaPath) {
                    wavg = 0.5f;
                } else if (j > 0) {
                    wmax = KIND == kSecondPR ? smax : BATCH ? fmaxf(fmaxf(wr, 1.0f), so) : a.q0.wmax1;
                    wavg = KIND == kSecondPR ? (sm + so) / 2.0f : BATCH ? bavg : a.q0.wavg1;
                }
                // get_weight_max: max(w) * h_MAX; the split bound's column height leaves the
                // return weight 1/p out; h-proportional proposals bound w alone
                const bool split = KIND == kNode2Vec && a.bound != 0 && j > 0;
                const float hB = kHprop ? 1.0f : hm;
                B = split ? smax * hB : wmax * hB;
                const float E = split ? fmaxf(0.0f, wr * hlast - (kHprop ? B * hlast : B)) : 0.0f;
                area = kHprop ? B * hs + E : (float)deg * B + E;
                bE = E;
                bZ = E;
                wlo = whi = 1.0f;
                if (kMem && j > 0) {
                    wp = wr;
                    wlo = KIND == kSecondPR ? fminf(sm, so) : BATCH ? fminf(1.0f, so) : a.q0.lo_w;
                    whi = smax;
                }
                bool member = false;
                // member board: regular columns at the lower weight w_oth take every proposal,
                // a region of area (w_mem - w_oth) * h_MAX * d(v') adds the members' excess,
                // the return edge keeps a column for its own; used when its area is the smaller
                if (kMem && a.bound == 2 && j > 0 && pdeg > 0 && sm > so) {
                    const float areg = kHprop ? so * hs : ((float)deg * so) * hm;
                    const float Rm = ((sm - so) * hm) * (float)pdeg;
                    const float Em = KIND == kNode2Vec ? fmaxf(0.0f, wr * hlast - so * (W ? hlast : 1.0f)) : 0.0f;
                    const float am = (areg + Rm) + Em;
                    if (am < area) {
                        member = true;
                        area = am;
                        bE = Em;
                        bZ = Em + Rm;
                        B = kHprop ? so : so * hm;
                        wp = fminf(wr, so);
                        wlo = whi = so;
                    }
                }
                mb = member;
                if (a.strategy == kAuto) {
                    st_bytes += W && deg != 0 ? 8 : 0;
                    // Eq. (runtime) with get_weight_sum = mean(w) * h_SUM; with the split board
                    // or h-proportional proposals the eRJS cost is area / S per step against
                    // deg for eRVS
                    const bool boards = split || kHprop || member;
                    const float lhs = a.rho * (boards ? area : B), S = wavg * hs;
                    rjs = deg >= a.d_lo && lhs < (boards ? (float)deg * S : S);
                } else {
                    st_bytes += W && deg != 0 ? 4 : 0;
                    rjs = true;
                    if (a.strategy == kRandomSelect) {
                        // comparison policy: a fair coin from the walker's own stream
                        const U4 x = philox((uint32_t)wid, (uint32_t)j, 0u, 4u, key0(), key1());
                        rjs = unit_uniform(x.x0) < 0.5f;
                    } else if (a.strategy == kDegreeSelect) {
                        rjs = deg >= a.d_lo;  // comparison policy: eRJS at high degree
                    }
                }
                // h-proportional proposals need some positive h: else eRVS
                if (rjs && kHprop && !(hs > 0.0f)) {
                    rjs = false;
                    fell_back = true;
                }
                op = rjs ? kTrial : kRvs;
            }
            if (EV == kEvHot && force) op = kRvs;
            if (deg == 0) op = kDead;
        }

        // 5. draw a trial (Section 3.3): a return-column trial reads nothing, a member trial a
        //    neighbour of prev, any other an edge or a proposal record
        if (op == kTrial) {
            const U4 x = philox((uint32_t)wid, (uint32_t)j, (uint32_t)trials, 0u, key0(), key1());
            ux = x.x2;
            const float z = unit_uniform(x.x3) * area;
            const bool ol = KIND == kNode2Vec && bE > 0.0f && z < bE;
            const bool mr = kMem && !ol && z < bZ;
            // floor(R n / 2^64) and the high half of its fraction, R = x1 : x0
            const int32_t n = (mr || kLab) ? pdeg : deg;
            const uint64_t t = (uint64_t)x.x1 * (uint32_t)n + (((uint64_t)x.x0 * (uint32_t)n) >> 32);
            const int64_t k = ((mr || kLab) ? pbase : base) + (int64_t)(t >> 32);
            if (kHprop) {
                aux = (uint32_t)t;  // the coin
                p = (kLab ? a.lprop : a.prop) + kPropU4 * k;
                op = mr ? kColR : kRec;
            } else if (mr) {
                op = kCol;
                aux = (uint32_t)k & 3u;
                p = reinterpret_cast<const uint4 *>(a.col) + (k >> 2);
            } else {
                op = kEdge;
                if (a.erec8 != nullptr) {
                    aux = (uint32_t)k & 3u;
                    p = reinterpret_cast<const uint4 *>(a.erec8) + (k >> 2);
                } else {
                    aux = (uint32_t)k & 1u;
                    p = reinterpret_cast<const uint4 *>(a.edges) + (k >> 1);
                }
                if (KIND == kMetaPath) elab = a.label[k];
            }
            if (ol) op = kRet;
        }

        // 6. issue the lanes' reads
        if (op == kStart) sv = *reinterpret_cast<const int32_t *>(p);
        issue_reads(p, (uint32_t)op & 7u, buf);

        // 7. ask for the counter's next chunk; it is handed out in the next pass
        const uint64_t idle = __ballot(op == kNone);
        if (idle != 0) {
            if (wnext >= wend && !exhausted) {
                qcnt = (int)min((int64_t)kWave, (left >> gshift) + 8);
                if (lane == 0) qfirst = atomicAdd(a.queue, (unsigned long long)qcnt);
            } else if (idle == ~0ull && wnext >= wend) {
                break;
            }
        }
    }

    // (the waves' read slots are free: no lane waits for a read)
    if (STATS) {
        // (Served ticks of one step keep an add per wave and counter: per block, such a tick of 700 walkers
        // takes 33 us instead of 50, and a request of 300 of them ends within the 10 ms for which the
        // server's queue is expected to hold the next one back.  With these adds 30 requests in ticks of
        // 64 steps at scale 20 take 2.42 ms, per block 2.29.)
        if (BATCH && a.tick_steps == 1) flush_stats(a, st, st_bytes);
        else flush_stats_block(a, st, st_bytes, reinterpret_cast<uint64_t *>(lds_all), kBufU4 * 2);
    }
}

// Launches the instance for one logic kind; see launch_walk.  Launches with counters have no
// kEvNone form, batches no kEvHub form (the callers choose none).
template <int KIND, bool W, int PROP, bool BATCH, bool STATS>
static void launch_trial_ev(const WalkArgs &args, int ev, int grid, hipStream_t s)
{
    WalkArgs a = args;
    a.lds_cap = trial_lds_cap(KIND, PROP, BATCH, ev, a.lds_cap);
    const size_t lds = trial_lds_bytes(KIND, PROP, BATCH, ev, a.lds_cap);
    if (!BATCH && ev == kEvHub)
        hipLaunchKernelGGL((walk_kernel<KIND, W, PROP, BATCH, STATS, BATCH ? kEvHot : kEvHub>), dim3(grid),
                           dim3(kBlock), lds, s, a);
    else if (!STATS && ev == kEvNone)
        hipLaunchKernelGGL((walk_kernel<KIND, W, PROP, BATCH, STATS, STATS ? kEvHot : kEvNone>), dim3(grid),
                           dim3(kBlock), lds, s, a);
    else
        hipLaunchKernelGGL((walk_kernel<KIND, W, PROP, BATCH, STATS, kEvHot>), dim3(grid), dim3(kBlock), lds, s, a);
}

template <int KIND, bool W, int PROP>
static void launch_trial_p(const WalkArgs &a, bool batch, int ev, int grid, hipStream_t s)
{
    if (batch) {
        if (a.stats) launch_trial_ev<KIND, W, PROP, true, true>(a, ev, grid, s);
        else launch_trial_ev<KIND, W, PROP, true, false>(a, ev, grid, s);
    } else {
        if (a.stats) launch_trial_ev<KIND, W, PROP, false, true>(a, ev, grid, s);
        else launch_trial_ev<KIND, W, PROP, false, false>(a, ev, grid, s);
    }
}

// Resident blocks per CU of the counter-free variant (the runtime's figure leaves out the scalar
// registers, which the compiled wave count holds).
template <int KIND, bool W, int PROP>
static int trial_blocks_p(bool batch, int ev, int lds_cap)
{
    const void *f = batch ? (ev == kEvNone ? (const void *)walk_kernel<KIND, W, PROP, true, false, kEvNone>
                                           : (const void *)walk_kernel<KIND, W, PROP, true, false, kEvHot>)
                          : (ev == kEvHub    ? (const void *)walk_kernel<KIND, W, PROP, false, false, kEvHub>
                             : ev == kEvNone ? (const void *)walk_kernel<KIND, W, PROP, false, false, kEvNone>
                                             : (const void *)walk_kernel<KIND, W, PROP, false, false, kEvHot>);
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &nb, f, kBlock, trial_lds_bytes(KIND, PROP, batch, ev, trial_lds_cap(KIND, PROP, batch, ev, lds_cap))) !=
        hipSuccess)
        nb = 1;
    return std::max(1, std::min(nb, trial_waves(ev)));
}

}  // namespace fw
