// chop_internal.h -- structures shared by the host runtime and the kernels of
// libdaqisland (not part of the public ABI; see include/daq.h for that).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "daq.h"

namespace daqk {

// Samples per thread: one 16-byte load per channel row.
constexpr int kVec = 8;
// Halo groups on one side for the largest window (post + 1 or pre + 1).
constexpr int kMaxHaloGroups = (DAQ_MAX_WINDOW + 1 + kVec - 1) / kVec;
// Channel count of one calorimeter (a 6 x 9 crystal grid, Section 3): the
// count for which the fused kernel can keep a whole tile in registers or LDS.
constexpr int kResidentChannels = 54;
// Kernel variants (daq_schedule.variant).
constexpr int kVariantReload = 0;    // rows read into registers, read again to write out
constexpr int kVariantResident = 1;  // rows kept in registers until written out
constexpr int kVariantStream = 2;    // rows DMA'd into LDS; two work-groups per CU
constexpr int kVariantReload18 = 3;  // as kVariantReload, 18 rows in flight per round (6 there)
constexpr int kVariantReload27 = 4;  // as kVariantReload, 27 rows in flight per round
constexpr int kVariantSplit = 5;     // scan pass (flag bits), edge and copy passes
constexpr int kVariantPipe = 6;      // one persistent kernel: scan tiles and copy chunks from shared counters
constexpr int kVariantLast = 6;
// Packed positions per chunk of a row: the copy pass writes one chunk of a
// channel group per wave (one 16-byte word per lane), and the persistent
// schedule records the island holding every multiple of it.
#ifndef DAQ_COPY_CHUNK
#define DAQ_COPY_CHUNK 512
#endif
constexpr int kCopyChunk = DAQ_COPY_CHUNK;
// Tile of the LDS variant: groups of 8 samples per row buffer, work-group size.
constexpr int kStreamGroups = 80;
constexpr int kStreamThreads = 256;
// Per-fill tile modes.
constexpr int kModeChop = 0;
constexpr int kModeStream = 1;

// Samples of a tile of the split variant's scan (one wave's 16-byte loads).
constexpr int kScanTile = 512;
// Its work-groups: the rows of a tile are shared by their waves, each with
// this many rows in flight (54 channels: 14 a wave, all at once).
constexpr int kScanThreads = 256;
constexpr int kScanRows = 14;
// The scan of launches without a fill of more than kNarrowChannels channels, and
// with at least kNarrowTiles tiles a CU: a wave per tile, kNarrowRows rows in
// flight. Whole calls over 24 fills of 560,000 samples, four waves per tile
// against this: 1 channel 116.8 / 38.3 us, 6 136.4 / 59.0, 12 154.1 / 92.4, 20
// 184.8 / 139.9, 28 207.8 / 189.6. Short launches are chains of loads, which
// four waves shorten: one fill of 8,191 samples, 12 channels 12.4 / 13.0, 20
// channels 12.9 / 14.3; of 560,000, 12 channels 21.8 / 19.0.
constexpr int kNarrowRows = 7;
constexpr int kNarrowChannels = 28;
constexpr int kNarrowTiles = 2;
// The scan computes its fill's pedestals itself up to this many pedestal
// samples (16 lanes hold them, 8 each); k_prepare does for more.
constexpr int kScanPed = 128;
// Split schedule: longer pedestals than this take a kernel with a work-group per
// channel after k_prepare.
#ifndef DAQ_LONG_PED
#define DAQ_LONG_PED 512
#endif
constexpr int kLongPed = DAQ_LONG_PED;
// Edge pass: a work-group takes a group of tiles, one 64-sample flag word per
// thread; every fill's summaries start at a whole group.
constexpr int kEdgeThreads = 256;
constexpr int kGroupTiles = kEdgeThreads * 64 / kScanTile;
// Tiles whose summaries one work-group adds up: a calorimeter fill of 560,000
// samples is one such segment; longer fills have segment summaries too.
constexpr int kSegGroups = 36;
constexpr int kSegTiles = kSegGroups * kGroupTiles;
// Emit pass: threads per work-group, and the launches that take it in place of the
// edge and copy passes: one fill, or up to kEmitFills of kEmitSamples samples
// together. Whole calls at the nominal pulse rate, emit against edge + copy, on
// one stream: 2 x 8,191 samples 14.1 / 18.5 us, 4 x 70,000 24.1 / 26.7, 4 x 140,000
// 32.3 / 34.8, 3 x 280,000 35.3 / 37.5, 2 x 560,000 39.0 / 37.7, 4 x 560,000 63.7 /
// 63.9. On three streams in turn its work-groups leave the other launches less
// room: 4 x 70,000 16.6 / 16.0, 2 x 560,000 29.1 / 27.8, 4 x 560,000 51.8 / 51.1.
constexpr int kEmitThreads = 512;
#ifndef DAQ_EMIT_FILLS
#define DAQ_EMIT_FILLS 4
#endif
constexpr int kEmitFills = DAQ_EMIT_FILLS;
constexpr int64_t kEmitSamples = 1 << 20;

// Flags of a stretch of samples, as a fill's islands see them (gap = pre + post
// + 1: windows of flags at most gap apart are one island). Stretches add up
// from left to right.
struct FlagSum {
    int32_t first, last;  // first and last flag, or -1
    int32_t begin;        // first flag of the island that holds `last`
    int32_t len;          // sum over neighbouring flags of min(their distance, gap)
    int32_t cnt;          // neighbouring flags more than gap apart
};

// Device-side view of one fill and where its results go.
struct FillDev {
    const int16_t *raw;
    int64_t n;          // samples
    int64_t stride;     // elements between channel rows
    int32_t C;
    int32_t np;         // pedestal samples
    int32_t thr;
    int32_t pre;
    uint64_t *flags;    // split variant: threshold flags, bit t % 64 of word t / 64; whole
                        // words, zero past the last sample
    int32_t *ped;       // may be null
    int64_t tile_base;  // global index of the fill's first tile in the launch
    int32_t post;
    int32_t gl;         // halo groups of 8 samples left of a tile: ceil((post + 1) / 8)
    int32_t gr;         // halo groups right of a tile: ceil((pre + 1) / 8)
    int32_t wide;       // 0: halo groups are ordinary thread groups of the tile;
                        // 1: extra groups loaded by a separate loop (wide windows)
    int32_t mode;       // kModeChop or kModeStream
    int32_t pad1;
    int64_t tout;       // samples a tile owns (decides and writes)
    int64_t n_tiles;
    int64_t sum_base;   // split variant: where the fill's groups of tiles begin, a multiple of kGroupTiles
    daq_island *isl;
    int64_t cap;
    daq_counts *counts;
    int16_t *out;       // may be null (find only)
    int64_t out_stride;
    int32_t *runs;      // split and pipe variants: (start, offset) of every island
                        // (room for the worst-case island count)
    union {
        int32_t *cmap;   // pipe variant: island holding packed position
                         // k * kCopyChunk, for every such position < total_len
        int64_t sum_at;  // split variant: index of the fill's first tile summary
    };
    int64_t *qsum;      // Q-method: decimated sums, or null
    int32_t *acc;       // Q-method: fill-by-fill accumulator rows, or null
    int64_t acc_stride;
};
static_assert(sizeof(FillDev) % 16 == 0, "descriptors are read as 16-byte words");

// Per-launch sizes kept in device memory so that a captured graph can be
// replayed for any batch that fits the scratch it was captured with.
struct BatchHdr {
    int32_t n_fills;
    int32_t stream_loads;  // 1: the scan reads raw rows non-temporally (batches larger than the caches)
    int64_t total_tiles;
    int64_t total_groups;  // split variant: groups of tiles of all fills
    int64_t pad2;
};
static_assert(sizeof(BatchHdr) % 16 == 0, "the descriptor table follows the header in one buffer");

struct KArgs {
    const FillDev *table;  // device table of n_fills entries, or null: use `one`
    const BatchHdr *hdr;   // device header, or null: use the three fields below
    int32_t n_fills;
    int32_t stream_loads;
    int64_t total_tiles;
    uint64_t *tile_state;  // one look-back word per tile (not the split variant)
    uint32_t *ticket;      // 16 words: tile dispenser; pipe variant: copy cursor, give-up flag
    int64_t *thr_eff;      // per fill: threshold + sum of pedestals
    uint64_t *tile_pref;   // pipe variant: finished tiles of each fill (one word per fill)
    const int64_t *tile_bases;  // split variant: each fill's tile_base and sum_base, with table
    const int64_t *sum_bases;
    int4 *sums;            // split variant: packed FlagSum of every tile
    FlagSum *seg_sums;     // split variant: the same of the segments of long fills
    int64_t total_groups;  // split variant, when hdr is null
    int32_t part, parts;   // split variant: this launch covers fill group `part`
                           // of `parts` equal groups of the batch
    int32_t split;         // 1: the split variant
    int32_t long_ped;      // split variant: most channels of a fill with more than kLongPed pedestal samples, or 0
    // which kernels are launched (split variant; read by the host alone)
    int16_t q_fused;       // the Q-method's pass takes the scan's place
    int16_t q_small;       // .. and loads accumulator rows together (launches the caches hold)
    int16_t ped_scan;      // the scan computes the pedestals
    int16_t narrow;        // the scan takes a wave per tile (fills of few channels)
    int16_t multi_seg;     // a fill has more than kSegTiles tiles
    int16_t fused;         // the emit pass takes the edge and copy passes' place
    int16_t copies;        // some fill has packed rows to write
    int16_t pad16;
    FillDev one;
};

struct GatherArgs {
    const int16_t *raw;
    int64_t n;  // samples
    int64_t stride;
    int32_t C;
    int32_t pad;
    const daq_island *isl;
    int64_t cap;
    daq_counts *counts;
    int16_t *out;
    int64_t out_stride;
};

// Tile geometry of one fill: halo groups, mode and the samples each tile
// owns. Halos up to a quarter of the tile's groups are ordinary groups of the
// tile; wider ones are loaded apart. The LDS variant takes 54-channel fills
// with such halos; every other fill uses the register path.
struct TileShape {
    int32_t gl, gr, wide, mode;
    int64_t tout;
};
inline TileShape tile_shape(int32_t pre, int32_t post, int32_t channels, int threads, int variant) {
    TileShape t;
    if (variant == kVariantSplit) {  // no halo: windows are the later passes' business
        t.gl = t.gr = t.wide = 0;
        t.mode = kModeChop;
        t.tout = kScanTile;
        return t;
    }
    t.gl = (post + 1 + kVec - 1) / kVec;
    t.gr = (pre + 1 + kVec - 1) / kVec;
    if (variant == kVariantStream && channels == kResidentChannels && (t.gl + t.gr) * 4 <= kStreamGroups) {
        t.mode = kModeStream;
        t.wide = 0;
        t.tout = (int64_t)(kStreamGroups - t.gl - t.gr) * kVec;
        return t;
    }
    t.mode = kModeChop;
    t.wide = (t.gl + t.gr) * 4 > threads ? 1 : 0;
    t.tout = (int64_t)(t.wide ? threads : threads - t.gl - t.gr) * kVec;
    return t;
}

hipError_t launch_prepare(const KArgs &a, int blocks, hipStream_t s);
hipError_t launch_chop(const KArgs &a, int threads, int variant, int grid, hipStream_t s);
// Split variant: the scan pass, then the edge and copy passes, over the fill
// group a.part of a.parts.
// Descriptors of up to kPutFills fills travel as kernel arguments into their
// table (no host staging buffer, no copy call).
constexpr int kPutFills = 16;
struct PutDescArgs {
    FillDev d[kPutFills];
    BatchHdr hdr;
    FillDev *dst;      // table entry of d[0]
    int64_t *tile_bases, *sum_bases;  // entries of d[0]
    BatchHdr *dst_hdr; // written when write_hdr
    int32_t count, write_hdr;
};
static_assert(sizeof(PutDescArgs) + sizeof(KArgs) <= 3840, "kernel arguments of the scan (explicit arguments well below 4 KB)");

// With `put` (split schedule, pedestals in the scan, one part): the scan takes
// the descriptors from its arguments and writes the table for the later passes.
hipError_t launch_scan(const KArgs &a, int grid, hipStream_t s, const PutDescArgs *put = nullptr);
hipError_t launch_emit(const KArgs &a, int edge_grid, int copy_grid, hipStream_t s);
// Both in one kernel, for launches of few fills of at most kSegTiles tiles.
hipError_t launch_emit_fused(const KArgs &a, int wgs_per_fill, hipStream_t s);
// Work-groups per CU of the copy pass's persistent grid.
#ifndef DAQ_COPY_WGS_PER_CU
#define DAQ_COPY_WGS_PER_CU 4
#endif
constexpr int kCopyWgsPerCu = DAQ_COPY_WGS_PER_CU;
hipError_t launch_pipe(const KArgs &a, int threads, int grid, hipStream_t s);
hipError_t launch_q(const KArgs &a, int threads, bool small, int grid, hipStream_t s);
hipError_t launch_unpack12(const uint8_t *in, int64_t in_stride, int32_t C, int64_t n, int16_t *out,
                           int64_t out_stride, int grid, hipStream_t s);
// Most fill groups a split launch is cut into (one HIP stream each).
#ifndef DAQ_MAX_PARTS
#define DAQ_MAX_PARTS 4
#endif
constexpr int kMaxParts = DAQ_MAX_PARTS;
hipError_t launch_gather(const GatherArgs &g, int n_cu, hipStream_t s);

// Island compression: one fill's packed rows and where its stream goes.
struct ZFillDev {
    const int16_t *packed;
    int64_t stride;            // elements between packed rows
    const daq_counts *counts;  // total_len: samples per row to compress
    int64_t max_len;           // rows hold at most this many samples
    uint32_t *hdr;             // C * ceil(L / 64) block headers
    int64_t *offsets;          // C * ceil(L / 64) payload word offsets, or null
    uint32_t *words;
    int64_t cap;               // words that fit
    int64_t *n_words;          // payload words of the whole stream
    int32_t C;
    int32_t pad;
};
// Fills per launch (the descriptors travel as kernel arguments, and 16 lanes
// share the work-groups out), waves per work-group, work-groups per launch
// (each wave of the pack pass sums the payload sizes of its fill's work-groups
// before its own).
constexpr int kZMaxFills = 16;
constexpr int kZWaves = 4;
#ifndef DAQ_Z_MAX_GRID
#define DAQ_Z_MAX_GRID 2048
#endif
constexpr int kZMaxGrid = DAQ_Z_MAX_GRID;
struct ZArgs {
    ZFillDev f[kZMaxFills];
    int64_t *gofs;  // scratch: payload words of each work-group of the grid, then of each wave
    int32_t n;
};
hipError_t launch_z(const ZArgs &a, int grid, hipStream_t s);

// Decompression: one stream back into packed rows.
struct ZStreamDev {
    const uint32_t *hdr;
    const int64_t *offsets;
    const uint32_t *words;
    int64_t n_words;
    int16_t *out;
    int64_t out_stride;
    int64_t L;
    int32_t C;
    int32_t pad;
};
struct ZDecArgs {
    ZStreamDev f[kZMaxFills];
    int32_t wg0[kZMaxFills + 1];  // first work-group of each stream, then the launch's number, then INT32_MAX
};
// one: a wave takes one group at most, and each of the n streams has `grid`
// work-groups; else `grid` is the launch's, shared out by wg0.
hipError_t launch_unz(const ZDecArgs &a, int n, bool one, int grid, hipStream_t s);

}  // namespace daqk
