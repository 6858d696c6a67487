// LDS of the walk kernels: what a block holds, and how much of a plan's lds_cap finds room beside it.
#pragma once

#include "fw_device.h"
#include "fw_internal.h"

namespace fw {

// LDS that each of `blocks` resident blocks of a CU can have (it is given out in parts of 1280 bytes).
constexpr int lds_per_block(int blocks) { return 160 * 1024 / 1280 / blocks * 1280; }

constexpr int kQueryTop = 256;  // entries of the query table's first level in LDS

// Resident waves per SIMD that the kernel is compiled for.  Without the scan its registers
// spill nothing and LDS holds four blocks per CU; one wave per SIMD already saturates random
// reads, more only hide the arithmetic between them.
constexpr int trial_waves(int ev) { return ev == kEvHub ? 3 : 4; }

// Where a wave's reads arrive: 64 slots of 64 bytes, lane l's at (l % 4) * kBufStride + (l / 4) * 4
// uint4; each quad of lanes fetches its four lanes' slots one after another, its lanes 16 bytes
// each (see issue_reads).  The stride's extra 16 bytes spread the slots of a quad over the banks.
constexpr int kBufStride = 65;
constexpr int kBufU4 = 4 * kBufStride;

constexpr bool trial_stash(int kind, int prop) { return uses_membership(kind) && prop == 1; }

// Path slots are held back in LDS until they fill an aligned part of 64 bytes and go out
// together: a random write of 16 or 32 bytes costs the memory 2.4 times one of 64 (22.8 against
// 54 G/s alone; random reads beside one write in eight: 33.9 G/s with 16-byte writes, 42.0 with
// 64-byte writes in proportion).  part_pos(row + s): the place of slot s in its part.
constexpr int kPart = 16;

// Dynamic LDS of a block: each wave's read slots, its stash of 64 vertex records (the record of
// a proposal whose membership test is open) and its held path slots, the schema or the query
// table's first level, each wave's N(prev) staging area (where the kernel has the scan).
constexpr size_t trial_lds_bytes(int kind, int prop, bool batch, int ev, int lds_cap)
{
    return (size_t)kWavesPerBlock * (kBufU4 * 16 + kWave * kPart * 4) +
           (trial_stash(kind, prop) ? (size_t)kWavesPerBlock * kWave * 16 : 0) +
           (batch ? (size_t)kQueryTop * 8 : (kind == kMetaPath ? 64 : 0)) +
           (uses_membership(kind) && ev != kEvNone ? (size_t)kWavesPerBlock * (size_t)lds_cap * sizeof(int32_t) : 0);
}

// The part of a plan's lds_cap that walk_kernel uses (a longer N(prev) is searched in place): at most
// what leaves room for the blocks that its registers allow.  Fewer blocks cost more than staging
// gains (300000 x 20 at scale 18, default plan: 1.42 ms with four blocks per CU, 1.99 with two,
// 3.26 with one; with half the steps by eRVS 25.6, 37.0, 63.1 ms).
constexpr int trial_lds_cap(int kind, int prop, bool batch, int ev, int lds_cap)
{
    const int other = (int)trial_lds_bytes(kind, prop, batch, kEvNone, 0), entry = (int)sizeof(int32_t) * kWavesPerBlock;
    const int most = (lds_per_block(trial_waves(ev)) - other) / entry / kWave * kWave;
    return lds_cap < most ? lds_cap : most;
}

// The same for rvs_kernel (30001 x 40 at scale 19: 9.1 ms with seven blocks per CU, 11.6 with
// five, 19.9 with two; 300000 x 10 at scale 16: 9.0, 11.4, 19.1).
constexpr int rvs_lds_cap(int lds_cap)
{
    const int most = lds_per_block(kMinWavesRvsOnly) / ((int)sizeof(int32_t) * kWavesPerBlock) / kWave * kWave;
    return lds_cap < most ? lds_cap : most;
}

}  // namespace fw
