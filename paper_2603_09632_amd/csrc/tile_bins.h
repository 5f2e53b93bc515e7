// Binning by tile: the tile sort for grids whose per-tile counters fit LDS.
#pragma once
#include "common.h"

namespace xgs {

constexpr int kBinThreads = 1024;
constexpr int kBinWaves = kBinThreads / 64;
// Blocks that share the Gaussians (one per CU), and the fewest Gaussians that
// are worth a block of their own.
constexpr int kBinMaxBlocks = 256;
constexpr int kBinMinChunk = 256;
// Tiles whose counters fit 64 KB of LDS; also the limit of the order table.
constexpr int kBinMaxTiles = 16384;
// Pairs that one wavefront sorts in registers (4 per lane), and one workgroup
// in LDS.
// A wavefront needs no barrier, but a longer list on one wavefront is the last
// to end (1,286 instances: 27 us against 16 with the workgroup form).
constexpr int kBinWaveKeys = 256;
constexpr int kBinBlockKeys = 2048;
// Runs that the first pass of the merge makes one, and so the longest lists that
// need no other (a list has at most 8,193 x 16,384 pairs, 65 of them); pairs that a
// workgroup of the merge sorts in LDS, and those workgroups (one fills a CU).
constexpr int kBinFan = 1024;
constexpr int kBinFanKeys = kBinFan * kBinBlockKeys;
constexpr int kBinMergeKeys = 8192;
constexpr int kBinMergeBlocks = 256;
// Lists that are merged by ranks.
constexpr int kBinRankKeys = 8 * kBinBlockKeys;
// Workgroups that take the longer lists (six to a CU by their LDS).
constexpr int kBinLongBlocks = 1536;
// Above this many instances per tile (of the capacity) the radix form is used: it
// has caught up.  On 48 tiles, this form against the radix form: 2,000 instances
// on each 36 / 80 us, 4,000 59 / 84, 8,000 89 / 95.
constexpr int64_t kBinMaxMeanList = 8192;

struct BinPlan {
    int blocks;     // blocks of the counting and scattering passes
    int64_t chunk;  // Gaussians per block
};

inline BinPlan bin_plan(int64_t n) {
    int64_t nb = (n + kBinMinChunk - 1) / kBinMinChunk;
    nb = nb < 1 ? 1 : nb > kBinMaxBlocks ? kBinMaxBlocks : nb;
    BinPlan p;
    p.chunk = ((n + nb - 1) / nb + 63) / 64 * 64;
    if (p.chunk < 64) p.chunk = 64;
    p.blocks = (int)((n + p.chunk - 1) / p.chunk);
    if (p.blocks < 1) p.blocks = 1;
    return p;
}

// A list above kBinBlockKeys has at most twice its length over kBinBlockKeys runs.
inline int64_t bin_max_runs(int64_t cap) { return 2 * (cap / kBinBlockKeys) + 1; }

struct BinWs {
    uint64_t* pairs;    // [cap] (depth bits << 32 | Gaussian), grouped by tile
    uint32_t* hist;     // [blocks][tiles] counts, then offsets within the tile
    uint32_t* totals;   // [tiles]
    uint2* runs;        // (tile, first position in its list) of the runs of lists above kBinBlockKeys
    uint32_t* n_runs;
    uint64_t* merged;   // [cap] runs of kBinFanKeys pairs, where a list can be longer
};

// Carves the workspace; *bytes is what it takes.
BinWs carve_bins(void* base, int64_t n, int64_t cap, int64_t tiles, size_t* bytes);

// Whether the sizes are in the range of bin_tile_sort.
bool bins_apply(int64_t n, int64_t cap, int64_t tiles);

// Same results as the radix form of the tile sort, bit for bit.
xgs_status bin_tile_sort(const xgs_projected* p, int64_t n, int tiles_x, int64_t tiles, const BinWs& w,
                         xgs_binning* b, hipStream_t st);

}  // namespace xgs
