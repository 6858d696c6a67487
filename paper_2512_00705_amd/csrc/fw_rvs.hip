// rvs_kernel: walks whose every step is sampled by eRVS (strategy FW_RVS_ONLY, one query;
// FlexiWalker, arXiv 2512.00705, Section 3.2), and the launch of either walk kernel.
//
// Every lane owns a walker; the wave serves its lanes' steps, short rows in groups of
// 8/16/32 lanes, longer rows one at a time with the whole wave (round 0 keys the first 64
// neighbours, then each lane scans its strided neighbours with the jump of Eq. (jump), and a
// wave argmax picks the next vertex).  The block of N(prev) is loaded ahead of the round's
// items (merge_member_early).
#include <algorithm>
#include <atomic>

#include "fw_lds.h"
#include "fw_walk.h"

namespace fw {

// Dynamic LDS of a block: each wave's N(prev) staging area.
static size_t rvs_lds_bytes(int lds_cap) { return (size_t)kWavesPerBlock * (size_t)lds_cap * sizeof(int32_t); }

// HV: virtual lanes per lane on rows of degree >= hub_deg (P = 64 * HV there); a variant of
// its own so that the extra lane state costs the other plans no registers.
template <int KIND, bool W, bool STATS, int HV>
__global__ void __launch_bounds__(kBlock, HV > 1 ? kMinWavesHub : STATS ? kMinWavesCounted : kMinWavesRvsOnly) rvs_kernel(WalkArgs a)
{
    extern __shared__ int32_t lds_all[];
    int32_t *lds = lds_all + (threadIdx.x / kWave) * a.lds_cap;
    const int lane = lane_id();
    const uint64_t below = lanes_below(lane);
    const uint64_t mine = ~0ull >> (kWave - a.wave_lanes);  // lanes that take walkers (1 <= wave_lanes <= 64)
    const QueryDev &Q = a.q0;

    enum { kIdle, kSetup, kServe, kAdv };
    int mode = kIdle;
    int32_t wid = -1, cur = 0, prev = -1, j = 0, nxt = -1;
    int64_t base = 0, pbase = 0;
    int32_t deg = 0, pdeg = 0;
    // path slots held back so that they go out together: from a 16-byte-aligned slot up to
    // four (one 16-byte store), from an 8-byte-aligned one two; npend slots ending at slot j
    // are held in p0, p1, p2
    int32_t p0 = 0, p1 = 0, p2 = 0, npend = 0;
    uint32_t st[kStBytes];
#pragma unroll
    for (int c = 0; c < kStBytes; ++c) st[c] = 0;
    uint64_t st_bytes = 0;
    bool exhausted = false;

    for (;;) {
        if (STATS && __ballot((st[kStTriggers] | st[kStSteps]) > 0x40000000u) != 0) flush_stats(a, st, st_bytes);

        // 1. hand walkers to idle lanes: one atomic per wave.  Only the wave's first wave_lanes
        //    lanes take walkers (see launch_walk), since a wave serves its lanes' steps one after
        //    another, and so half of them may as well wait for the others: the counter takes about
        //    120 M adds a second (MetaPath, 180000 x 5 at scale 15: 920 us with an add as soon as a
        //    lane is idle, 680 so; Node2Vec, 100000 x 2 at scale 17: 862 and 744).
        const uint64_t idle = __ballot(mode == kIdle) & mine;
        if (!exhausted && 2 * __popcll(idle) >= a.wave_lanes) {
            const int leader = __ffsll((unsigned long long)idle) - 1;
            const int cnt = __popcll(idle);
            unsigned long long first = 0;
            if (lane == leader) first = atomicAdd(a.queue, (unsigned long long)cnt);
            first = (unsigned long long)bcast_i64((int64_t)first, leader);
            if ((int64_t)first + cnt >= a.n) exhausted = true;
            if ((idle >> lane) & 1) {
                const int64_t w = (int64_t)first + __popcll(idle & below);
                if (w < a.n) {
                    int32_t *row = Q.paths + w * ((int64_t)Q.L + 1);
                    const int32_t s = Q.starts[w];
                    row[0] = s;
                    st_bytes += 12 + 4 * (uint64_t)Q.L;
                    if (s < 0 || (int64_t)s >= a.nv) {
                        atomicOr(a.err, 1);
                        for (int r = 1; r <= Q.L; ++r) row[r] = -1;
                        Q.lengths[w] = 0;
                    } else {
                        wid = (int32_t)w;
                        cur = s;
                        prev = -1;
                        j = 0;
                        mode = kSetup;
                    }
                }
            }
        }
        if (__ballot(mode != kIdle) == 0) {
            if (exhausted) break;
            continue;
        }

        // 2. step set-up: row of cur
        if (mode == kSetup) {
            if (j == Q.L) {
                Q.lengths[wid] = j;
                mode = kIdle;
            } else {
                const uint4 r = a.vrec[cur];
                base = row_start(a, r, cur);
                deg = (int32_t)r.y;
                st_bytes += 16;
                nxt = -1;
                mode = deg == 0 ? kAdv : kServe;
                if (KIND == kMetaPath && a.proposal == 2 && deg != 0) {
                    // the plan reads the wanted label's group bounds: an empty group ends the walk
                    const int32_t wl = (int32_t)Q.schema[j % Q.schema_len];
                    int64_t g0 = 0, g1 = 0;
                    if (wl < a.nlab) {
                        g0 = a.lrow[(int64_t)cur * a.nlab + wl];
                        g1 = a.lrow[(int64_t)cur * a.nlab + wl + 1];
                    }
                    st_bytes += 8;
                    if (g1 == g0) mode = kAdv;
                }
            }
        }

        // 3. eRVS for every lane that needs it (Section 5)
        {
            const bool want_rvs = mode == kServe;
            const uint8_t want = KIND == kMetaPath && want_rvs ? Q.schema[j % Q.schema_len] : (uint8_t)0;
            uint64_t s8 = __ballot(want_rvs && deg <= 8);
            uint64_t s16 = __ballot(want_rvs && deg > 8 && deg <= 16);
            uint64_t s32 = __ballot(want_rvs && deg > 16 && deg <= 32);
            uint64_t big = __ballot(want_rvs && deg > 32);
            if (__popcll(s8) <= 4) {
                s16 |= s8;
                s8 = 0;
            }
            if (__popcll(s16) <= 2) {
                s32 |= s16;
                s16 = 0;
            }
            // the per-step accounting is the same whichever lanes served the step
            auto served = [&](int32_t res, uint32_t trig) {
                nxt = res;
                mode = kAdv;
                st[kStTriggers] += trig;
                uint64_t by = (uint64_t)deg * (uint64_t)a.item_bytes;
                if (uses_membership(KIND) && j > 0) {
                    const uint64_t stage = 4 * (uint64_t)pdeg;
                    const uint64_t search = 4 * (uint64_t)deg * (uint64_t)probes(pdeg);
                    by += stage < search ? stage : search;
                }
                st_bytes += by;
                if (res >= 0) st[kStRvs] += 1;
            };
            int32_t res = -1;
            float hres = 1.0f;
            for (int G = 8; G <= 32; G <<= 1) {
                uint64_t pool = G == 8 ? s8 : (G == 16 ? s16 : s32);
                while (pool != 0)
                    if (rvs_group_pass<KIND, W, false>(a, G, pool, 0, wid, j, prev, base, deg, pbase, pdeg, want, res,
                                                       hres))
                        served(res, 0);
            }
            while (big != 0) {
                const int src = __ffsll((unsigned long long)big) - 1;
                big &= big - 1;
                const uint32_t s_wid = bcast_u32((uint32_t)wid, src);
                const int32_t s_j = bcast_i32(j, src);
                const int32_t s_prev = bcast_i32(prev, src);
                const int64_t s_base = bcast_i64(base, src);
                const int32_t s_deg = bcast_i32(deg, src);
                const int64_t s_pbase = bcast_i64(pbase, src);
                const int32_t s_pdeg = bcast_i32(pdeg, src);
                const uint8_t s_want = KIND == kMetaPath ? (uint8_t)bcast_u32(want, src) : (uint8_t)0;
                const bool member_test = uses_membership(KIND) && s_j > 0;
                Mem m = {a.col + s_pbase, s_pdeg, false, false};
                // merge the rows when N(prev) is not much longer than the row scanned
                const bool merge = member_test && (int64_t)s_pdeg <= (int64_t)kMergeRatio * s_deg;
                // stage N(prev) in LDS for the merge (its reads become LDS reads), or for the
                // per-item searches when they would read more than the staging
                if (member_test && s_pdeg <= a.lds_cap &&
                    (merge || (int64_t)s_pdeg <= (int64_t)s_deg * probes(s_pdeg))) {
                    wave_lds_sync();
                    for (int32_t i = lane; i < s_pdeg; i += kWave) lds[i] = a.col[s_pbase + i];
                    wave_lds_sync();
                    m.p = lds;
                    m.staged = true;
                }
                uint32_t trig = 0;
                const StepW sw = step_weights<KIND>(Q, s_deg, s_pdeg);
                // P = 64 lanes, or 64 * HV on a row of degree >= hub_deg
                if (HV > 1 && s_deg >= a.hub_deg)
                    res = rvs_step_hub<KIND, W, HV, true>(a, Q, m, s_wid, s_j, s_prev, s_base, s_deg, s_want, sw, trig,
                                                          hres, merge);
                else
                    res = rvs_step<KIND, W, true>(a, Q, m, s_wid, s_j, s_prev, s_base, s_deg, s_want, sw, trig, hres,
                                                  merge);
                if (lane == src) served(res, trig);
            }
        }

        // 4. apply the step (update) and write the path
        if (mode == kAdv) {
            int32_t *row = Q.paths + (int64_t)wid * ((int64_t)Q.L + 1);
            if (nxt < 0) {
                if (npend > 0) {
                    flush_path(row + (j + 1 - npend), npend, p0, p1, p2);
                    npend = 0;
                }
                // pad with -1: single slots up to a 16-byte boundary, then 16-byte stores
                int r = j + 1;
                for (; r <= Q.L && (reinterpret_cast<uintptr_t>(row + r) & 15) != 0; ++r) row[r] = -1;
                for (; r + 3 <= Q.L; r += 4) *reinterpret_cast<int4 *>(row + r) = make_int4(-1, -1, -1, -1);
                for (; r <= Q.L; ++r) row[r] = -1;
                Q.lengths[wid] = j;
                st[kStEarly] += 1;
                mode = kIdle;
            } else {
                const int32_t s = j + 1;
                if (npend == 0) {
                    const uintptr_t ad = reinterpret_cast<uintptr_t>(row + s);
                    if (((ad & 15) == 0 && s + 3 <= Q.L) || ((ad & 7) == 0 && s + 1 <= Q.L)) {
                        p0 = nxt;
                        npend = 1;
                    } else {
                        row[s] = nxt;
                    }
                } else {
                    int32_t *first = row + (s - npend);
                    // the group's size follows from its first slot as when it was started
                    if ((reinterpret_cast<uintptr_t>(first) & 15) != 0 || s - npend + 3 > Q.L) {
                        *reinterpret_cast<int2 *>(first) = make_int2(p0, nxt);
                        npend = 0;
                    } else if (npend == 3) {
                        *reinterpret_cast<int4 *>(first) = make_int4(p0, p1, p2, nxt);
                        npend = 0;
                    } else {
                        if (npend == 1) p1 = nxt;
                        else p2 = nxt;
                        ++npend;
                    }
                }
                st[kStSteps] += 1;
                prev = cur;
                cur = nxt;
                pbase = base;
                pdeg = deg;
                ++j;
                mode = kSetup;
            }
        }
    }

    if (STATS) {
        __shared__ uint64_t sums[kWavesPerBlock * kNumStats];
        flush_stats_block(a, st, st_bytes, sums, kNumStats);
    }
}

// ---------------------------------------------------------------- launches
template <int KIND, bool W, bool STATS>
static void launch_rvs_s(const WalkArgs &args, int grid, hipStream_t s)
{
    WalkArgs a = args;
    a.lds_cap = rvs_lds_cap(a.lds_cap);
    const size_t lds = rvs_lds_bytes(a.lds_cap);
    const int hv = a.hub_deg > 0 ? a.hub_v : 1;
    if (hv == 4) hipLaunchKernelGGL((rvs_kernel<KIND, W, STATS, 4>), dim3(grid), dim3(kBlock), lds, s, a);
    else if (hv == 2) hipLaunchKernelGGL((rvs_kernel<KIND, W, STATS, 2>), dim3(grid), dim3(kBlock), lds, s, a);
    else hipLaunchKernelGGL((rvs_kernel<KIND, W, STATS, 1>), dim3(grid), dim3(kBlock), lds, s, a);
}

template <int KIND, bool W>
static hipError_t launch_rvs(const WalkArgs &a, int grid, hipStream_t s)
{
    if (a.stats != nullptr) launch_rvs_s<KIND, W, true>(a, grid, s);
    else launch_rvs_s<KIND, W, false>(a, grid, s);
    return hipGetLastError();
}

template <int KIND, bool W>
static int rvs_blocks(int lds_cap)
{
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, rvs_kernel<KIND, W, false, 1>, kBlock,
                                                     rvs_lds_bytes(rvs_lds_cap(lds_cap))) != hipSuccess)
        nb = 1;
    return nb > 0 ? nb : 1;
}

static hipError_t launch_trial(const WalkArgs &a, const WalkShape &w, int ev, hipStream_t s)
{
    if (w.kind == kNode2Vec) return launch_trial_node2vec(a, w.weighted, w.batch, ev, w.grid, s);
    if (w.kind == kSecondPR) return launch_trial_secondpr(a, w.weighted, w.batch, ev, w.grid, s);
    return launch_trial_metapath(a, w.weighted, w.batch, ev, w.grid, s);
}

// Blocks per CU that are resident at once, of the kernel the launch takes.  Asked of the
// runtime once per kernel and lds_cap: it depends on nothing else.
static int resident_blocks(const WalkArgs &a, const WalkShape &w)
{
    static std::atomic<uint32_t> known[kNumKinds][2][2][3][4];  // (lds_cap + 1) << 8 | blocks
    const bool rvs_only = !w.batch && a.strategy == kRvsOnly;
    std::atomic<uint32_t> &k = known[w.kind - 1][w.weighted][w.batch][a.proposal][rvs_only ? 3 : w.ev];
    const uint32_t have = k.load(std::memory_order_relaxed);
    if ((have >> 8) == (uint32_t)a.lds_cap + 1) return (int)(have & 255u);
    int nb;
    if (rvs_only)
        nb = w.kind == kNode2Vec   ? (w.weighted ? rvs_blocks<kNode2Vec, true>(a.lds_cap) : rvs_blocks<kNode2Vec, false>(a.lds_cap))
             : w.kind == kSecondPR ? (w.weighted ? rvs_blocks<kSecondPR, true>(a.lds_cap) : rvs_blocks<kSecondPR, false>(a.lds_cap))
                                   : (w.weighted ? rvs_blocks<kMetaPath, true>(a.lds_cap) : rvs_blocks<kMetaPath, false>(a.lds_cap));
    else
        nb = w.kind == kNode2Vec   ? trial_blocks_node2vec(w.weighted, w.batch, a.proposal, w.ev, a.lds_cap)
             : w.kind == kSecondPR ? trial_blocks_secondpr(w.weighted, w.batch, a.proposal, w.ev, a.lds_cap)
                                   : trial_blocks_metapath(w.weighted, w.batch, a.proposal, w.ev, a.lds_cap);
    k.store(((uint32_t)a.lds_cap + 1) << 8 | (uint32_t)nb, std::memory_order_relaxed);
    return nb;
}

// 15000 walkers x 52 steps (two more blocks' worth than CUs): 110 us at 1 or 2, 119 at 3;
// 84000 x 2: 34.4, 28.6, 25.9 us; 110000 x 52 with loose bounds: 1.26, 1.23, 1.34 ms.
// Uniform proposals of the other walks reject most (2nd-PageRank at scale 20, 100000 x 40: 7.2 ms
// at 2, 6.2 at 3, 5.7 at 4; MetaPath at scale 18, 60000 x 40: 774, 653, 617 us), and the wave
// takes its lanes' long runs of rejections one after another, as eRVS.
constexpr int kSpread = 2;

WalkShape walk_shape(const WalkArgs &a, int kind, bool weighted, bool batch, int ev, int64_t n, int plan_grid)
{
    int dev = 0, cus = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (cus <= 0) cus = 1;
    // Counted and resumable launches have no kEvNone form, and one that the kEvHot form's lanes
    // hold whole gains nothing from it and would only pay for the second launch.
    const bool trials_only = ev == kEvNone;
    if (ev == kEvNone && (a.stats != nullptr || a.tick_steps > 0 || n <= (int64_t)cus * 4 * trial_waves(kEvHot) * kWave)) ev = kEvHot;
    WalkShape w{kind, weighted, batch, ev, 1, 1};
    const int64_t full = (int64_t)resident_blocks(a, w) * cus;
    // Never more waves than walkers: few walkers get one lane or a few per wave, since a wave
    // serves its lanes' eRVS steps one after another.  Where every step is eRJS there is nothing
    // to serve, and beyond kSpread waves per SIMD half-empty waves only compete for issue slots.
    // So do eRVS walks of one step: see launch_walk.  Second-order PageRank with gamma = 0 weighs all
    // neighbours alike, so its uniform proposals reject few (25000 x 40 at scale 12: 240 us on twice
    // the waves, 200 so).
    int64_t need = std::max<int64_t>(1, (n + kWavesPerBlock - 1) / kWavesPerBlock);
    const bool one = !batch && a.strategy == kRvsOnly && a.q0.L <= 1;
    const bool first_order = kind == kSecondPR && a.q0.gamma == 0.0f;
    if (one || (trials_only && (kind == kNode2Vec || a.proposal != 0 || first_order)))
        need = std::max(std::min(need, (int64_t)cus * (one ? 1 : kSpread)), (n + kBlock - 1) / kBlock);
    w.grid = plan_grid > 0 ? plan_grid : (int)std::min(full, need);
    w.resident = (int)std::min<int64_t>(full, w.grid);
    return w;
}

hipError_t launch_walk(const WalkArgs &args, const WalkShape &w, hipStream_t s)
{
    WalkArgs a = args;
    const bool rvs_only = !w.batch && a.strategy == kRvsOnly;
    int ev = w.ev;
    if (ev == kEvNone && a.stats != nullptr) ev = kEvHot;
    const int64_t waves = (int64_t)(rvs_only ? w.grid : w.resident) * kWavesPerBlock;
    // rvs_kernel: walkers spread over all waves, and a wave holds only a quarter of its share at
    // a time: a walk's cost varies with the rows it meets, and walkers that have not started go to
    // the waves that are done first.  Rows short enough to be served several at a time (mean below
    // 12) want more lanes that wait: half.  Full waves, spread whole, by halves, by quarters, in ms:
    // 30001 x 40 at scale 19: 76.0, 12.8, 10.3, 9.0; MetaPath, 100000 x 20 at scale 18: -, 5.1,
    // 4.6, 3.9; mean row of 8, 400000 x 5 at scale 14: -, 0.99, 0.94, 1.14.
    // Walks of one step scan the rows of their starts, which differ little (later steps meet rows in
    // proportion to their length), and take less than their turn at the counter, which serves about
    // 120 M a second: up to 64 at a time on a wave per SIMD, then more waves (scale 17, 6000 x 1 and
    // 300000 x 1: 230 and 734 us by quarters over all waves, now 112 and 268).
    const int64_t share = a.q0.L <= 1 ? waves : waves * (a.ne < 12 * a.nv ? 2 : 4);
    a.wave_lanes = (int32_t)std::min<int64_t>(kWave, (a.n + share - 1) / share);
    // walk_kernel: a launch of up to a quarter more walkers than lanes is shared out over the waves;
    // of a larger one seven eighths, the rest goes by the counter to the waves that are done first.
    // The counter's round trips take longer than a short walk: at 300000 walkers on 262144 lanes
    // MetaPath by label groups, 40 steps at scale 14, takes 171 us whole and 271 by the counter,
    // Node2Vec on the default plan, 20 steps at scale 18, 1.33 and 1.40 ms; at twice the lanes whole
    // is slower (default plan, 500000: 2.08 and 1.90 ms).
    const bool whole = a.n <= waves * kWave * 5 / 4;
    a.static_n = whole ? a.n : a.n - a.n / 8;
    a.static_waves = waves;
    a.static_each = a.static_n / waves;
    a.static_more = a.static_n % waves;
    if (rvs_only || ev == kEvNone || !whole) {
        const hipError_t e = launch_zero(a.queue, ev == kEvNone ? kQueueWords : 1, s);
        if (e != hipSuccess) return e;
    }
    if (rvs_only) {
        if (w.kind == kNode2Vec)
            return w.weighted ? launch_rvs<kNode2Vec, true>(a, w.grid, s) : launch_rvs<kNode2Vec, false>(a, w.grid, s);
        if (w.kind == kSecondPR)
            return w.weighted ? launch_rvs<kSecondPR, true>(a, w.grid, s) : launch_rvs<kSecondPR, false>(a, w.grid, s);
        return w.weighted ? launch_rvs<kMetaPath, true>(a, w.grid, s) : launch_rvs<kMetaPath, false>(a, w.grid, s);
    }
    a.parked = (int *)(a.queue + 1);
    const hipError_t e = launch_trial(a, w, ev, s);
    if (e != hipSuccess || ev != kEvNone) return e;
    // the walks that met an eRVS step (usually none) run on in the form that has the scan; all
    // walkers shared out whole, since most have only their length read (4 M walkers of 5 steps, one
    // of them parked: 0.94 ms, by the counter 1.86, none parked 0.92)
    a.resume = 1;
    a.static_n = a.n;
    a.static_each = a.n / waves;
    a.static_more = a.n % waves;
    return launch_trial(a, w, kEvHot, s);
}

}  // namespace fw
