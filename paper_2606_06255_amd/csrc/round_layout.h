// Layout and capacity rules of the multi-pick sampler, shared by its kernels,
// the launchers and the host tests.
#pragma once

#include <cstdint>

#include "prune_bound.h"

namespace rfps {

// Threads and wavefronts of a sampler workgroup.
constexpr int kRBlock = 512;
constexpr int kRLanes = 64;
constexpr int kRWaves = kRBlock / kRLanes;
// Lookahead steps of a wavefront, and so candidates of a workgroup, at most.
constexpr int kMaxSteps = 8;
constexpr int kMaxRec = kRWaves * kMaxSteps;
constexpr int kMinSteps = 2;
// Candidates one merge lists, and so the selections one round may settle
// (the merge stops there; a shorter round is always valid).
constexpr int kList = 256;
constexpr int kListWords = kList / kRLanes;
// Side of the 16 x 16 blocks the matrix cores filter.
constexpr int kBlk = 16;
// Static LDS of a sampler workgroup, at most; the rest of the compute unit's
// is its tiles and points.
constexpr uint32_t kRoundsStatic = 27712;

// A published slot: K + 1 units of four 64-bit words, one unit per candidate
// and one for the bound.  A word is tag << 48 | 48 payload bits.
constexpr int kUnit = 4;
RFPS_HOST_DEVICE inline uint32_t slot_units(uint32_t K) { return K + 1u; }

// Tile slots of a workgroup: its tiles are dealt to the wavefronts in turn,
// and every wavefront's share is padded to whole filter blocks.
RFPS_HOST_DEVICE inline uint32_t wave_slots(uint32_t tiles)
{
    return ((tiles + kRWaves - 1) / kRWaves + kBlk - 1) / kBlk * kBlk;
}

RFPS_HOST_DEVICE inline uint32_t rounds_lds_need(uint32_t tiles, uint32_t pts)
{
    return wave_slots(tiles) * kRWaves * 36u + pts * 20u;
}

// The share a workgroup may take: R candidates with whole coordinates per
// slot, a private copy of the distances and the sort buffers of one list, as
// counted here, against the budget the caller passes.  This is the sampler's
// documented capacity (RFPS_ERR_CAPACITY beyond it); the layout above needs
// less for every share it admits (4 bytes less per point, and more than the
// padding of the tile slots costs).
RFPS_HOST_DEVICE inline uint32_t share_bytes(uint32_t tiles, uint32_t pts, uint32_t G, uint32_t R)
{
    uint32_t sort = 2 * kRLanes;
    while (sort < G * R)
        sort <<= 1;
    const uint32_t keys = 2u * sort, picks = 6u * kRLanes;
    const uint32_t padded = tiles ? (tiles + 31u) / 32u * 32u : 32u;
    return tiles * 40u + padded * 16u + pts * 24u + G * (6u * R + 2u) * 4u + (2u * kRLanes + 2u) * 4u + sort * 4u +
           (keys > picks ? keys : picks) * 4u + 128u;
}
RFPS_HOST_DEVICE inline bool share_granted(uint32_t tiles, uint32_t pts, uint32_t G, uint32_t R,
                                                       uint32_t budget)
{
    return pts <= 65535u && share_bytes(tiles, pts, G, R) <= budget;
}

// Shape of a team: its workgroups, the candidates each publishes per round
// and the lookahead steps of each wavefront.  A cloud most of whose tiles
// hold many of its picks (few, full tiles: a spinning sweep sampled to a
// quarter) needs depth, one with several tiles per pick breadth.  Measured
// sampling times in ms for (workgroups, candidates, steps), by picks per tile:
//                                   (256, 3, 2)  (128, 3, 2)  (64, 3, 2)  (64, 6, 4)
//   sweep of 114,624 (2,154 tiles)  3: 2.70         2.30         2.14        2.47
//                                   6.5: 4.18       3.73         3.61        3.44
//                                   13: 6.38        5.98         6.24        5.24
//   room of 40,000 (3,643 tiles)    2: 1.56         1.36         1.51        1.69
//                                   6.5: 2.89       2.84         3.52        3.09
// The line of six is a sweep's: there depth pays from about five picks a tile.
// A room or a very large sweep is up to 16 % faster broad at 6.5 (room of
// 120,000: (256, 3, 2) 6.07, the rule's (64, 6, 4) 7.06; sweep of 1,000,000:
// 14.7, and 16.1 by the rule).
constexpr int kDeepPicks = 6;  // picks per tile from which depth pays
struct TeamShape {
    int G, K, steps;
};
RFPS_HOST_DEVICE inline TeamShape team_shape(uint32_t tiles, uint32_t m)
{
    TeamShape t;
    const bool deep = m > (uint32_t)kDeepPicks * tiles;
    // enough workgroups that the exchange, whose cost grows with the team,
    // still replaces more local work than it adds: up to six picks a tile the
    // rule is within 7 % of the best of ten shapes from 602 to 39,449 tiles
    // (12 % on a sweep of 602 at 5.5 picks)
    if (deep)
        t.G = tiles < 400 ? 16 : tiles < 1500 ? 32 : 64;
    else
        t.G = tiles < 500 ? 32 : tiles < 2500 ? 64 : tiles < 12000 ? 128 : 256;
    t.K = deep ? 6 : 3;
    t.steps = deep ? 4 : 2;
    return t;
}

// Batches: team sizes are per_xcd >> level.  A workgroup has two slots of the
// largest size side by side on the board; the control words of the levels
// follow.
constexpr int kBatchLevels = 6;
constexpr int kBatchSlotWords = 2 * 64;
// Candidates a workgroup of a batch publishes, by level and (a whole XCD) by
// the points a workgroup holds.  Few workgroups must publish many for a round
// to settle many picks; a large team lists enough of few.  Measured with the
// device full, ms for 4 | 6 | 8 | 15 candidates: 1,024 points on 32
// workgroups 0.43 | 0.46 | 0.50 | -, 16,384 on 32 1.50 | 1.45 | 1.51 | -,
// 50,000 on 32 3.23 | 2.83 | 2.80 | -, 65,536 on 32 - | - | 3.95 | 4.50, 8,192
// on 2 - | - | 2.40 | 2.05, 16,384 on 4 - | - | 2.30 | 2.03.
constexpr int kBatchK = 15;  // at most (a slot's words)
RFPS_HOST_DEVICE inline int batch_k(int level, unsigned long long points_per_group)
{
    if (level > 2)
        return kBatchK;
    return level > 0 || points_per_group >= 1500u ? 8 : points_per_group >= 400u ? 6 : 4;
}
// Lookahead steps of a wavefront in a batch: 4 (2 cost up to 20 % where a
// workgroup's share is full and gain 1 % where it is small; 8 gain nothing).
constexpr int kBatchSteps = 4;
// A workgroup publishes fewer candidates than it has (so its next one bounds
// the rest): K is at most kBatchK here, and at most 8 otherwise.
static_assert(kBatchK < kRWaves * kMinSteps && kMinSteps <= kBatchSteps, "candidates of a workgroup");

// One workgroup for a whole cloud (solo_cloud.h): a ring of keys and the
// coordinates in LDS, at most 16 points a thread in registers.
constexpr uint32_t kSoloRingBytes = 1024;
constexpr int kSoloPoints = 8192;
RFPS_HOST_DEVICE inline uint32_t solo_lds(uint32_t n) { return kSoloRingBytes + n * 16u; }
// Whether a single call gives a cloud to one workgroup.  Measured, sampling
// from call to completion in us, by one workgroup and by a team.  A quarter of
// the points: 512 points 43 | 155, 1,024 73 | 213, 2,048 167 | 263, 3,000
// 270 | 301, 3,500 352 | 374, 4,000 400 | 378.  A selection costs one workgroup
// the same throughout and a team less and less, so with eight points a lane
// (above 3,072) most of a cloud is a team's: 3,584 points of a room, half of
// them 701 | 709, three quarters 1,042 | 982, all 1,386 | 1,283; of a cube, all
// 1,385 | 985.
constexpr int kSoloSingle = 3584, kSoloSingleAll = 3072;
RFPS_HOST_DEVICE inline bool solo_single(int n, int m)
{
    return n <= kSoloSingleAll || (n <= kSoloSingle && m <= n / 2);
}
static_assert(kSoloRingBytes + kSoloSingle * 16u <= 65536u, "no opt-in for more LDS");

// Bytes a workgroup's share may take by that rule: what a compute unit has
// beside 6,496 bytes.
constexpr uint32_t kRoundsReserve = 6496;
RFPS_HOST_DEVICE inline uint32_t rounds_budget(uint32_t max_lds)
{
    return max_lds <= kRoundsReserve + 1024u ? 0u : (max_lds - kRoundsReserve - 256u) & ~255u;
}
// Dynamic LDS the sampler is launched with.
RFPS_HOST_DEVICE inline uint32_t rounds_dynamic(uint32_t max_lds)
{
    return max_lds > kRoundsStatic + 1024u ? (max_lds - kRoundsStatic) & ~63u : 0u;
}

}  // namespace rfps
