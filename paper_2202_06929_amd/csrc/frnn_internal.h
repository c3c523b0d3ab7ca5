// Internal declarations shared by the host driver (frnn_api.cpp) and the HIP
// kernels (frnn_kernels.hip).  Not part of the public interface.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace frnn {

constexpr int kBlock = 256;          // threads per workgroup (4 wave64)
constexpr int kWaves = kBlock / 64;
constexpr int kBoundsBlocks = 256;   // most bounds partials per event
constexpr int kScanTile = 4096;      // elements per workgroup in the scans
constexpr int kListCap = 16;         // neighbours a query may collect in the main search
constexpr int kQTile = 32;           // queries of one cell handled together by a wave
constexpr int kRing = 128;           // first-stage survivors queued per wave (a power of two)
constexpr int kMaxReach = 3;         // largest cell_div
constexpr int kMaxAxes = 4;          // binned coordinates: 3, or 4 with cell_div 1
// Cells per binned axis.  The bound keeps the float32 rounding of a cell
// coordinate under the cell margin; with four axes it also lets the four
// coordinates of a cell pack into one 32-bit word (8 bits each; 10 bits each
// with three axes).
constexpr int kGridAxisMax3 = 1024;
constexpr int kGridAxisMax4 = 256;
constexpr int kMaxK = 4096;
// Most pieces of the search (wave_start has an entry per piece).
constexpr int kMaxPieceCount = 98304;
// A cell's fixed cost in the search (its runs' bounds, its candidates' first
// loads), in queries, when the queries are divided among the waves by work.
// Weights of 0, 1, 2 and 4, in us a call: a 120k-point event 60.8, 59.1, 59.2 and 59.2,
// its nearest 8 64.9, 65.9, 67.6 and 69.6, 300k 12-D points 127.7, 125.3, 125.2 and 127.1,
// 60k rows of 32 floats 82.3, 80.8, 81.6 and 83.3, six events served 196, 193, 192 and 194.
constexpr unsigned int kTileWeight = 1;
// Fewest rows per wave of the search.  Below it more waves only repeat the fixed costs
// (the cells they cut, partly filled list write-outs), above it too few run at once: a
// 20,000-point event of crowded cells took 121, 120, 119, 124 and 140 us with at least
// 1, 2, 4, 8 and 16 rows, and a 2,000-point event 55.5, 54.8, 55.0, 57.0 and 60.6 us.
constexpr long long kMinWaveRows = 4;
// Rows per piece from which the search takes more rounds of workgroups.  Pieces of this
// size keep the rows, cell starts and ids that an XCD's resident waves read (about a
// thousand pieces) near its 4 MB of L2: a batch of 5.6M 8-D points took 2,561, 2,286,
// 2,096, 1,975 and 1,955 us with 1, 2, 4, 8 and 16 rounds (683 to 43 rows per piece), six
// events of 610k points in all 251, 246 and 249 us with pieces of up to 128, 32 and 16
// rows, a 300k-point 12-D event 156.5 and 154.7 us with up to 128 and 32.
constexpr long long kRowsPerPiece = 32;
constexpr int kClaimStride = 32;  // words between the XCDs' counters: 128 bytes
constexpr int kKeysBlock = 1024;     // threads per workgroup of the key/histogram pass
constexpr int kKeysPer = 2;          // points per thread of the key/histogram pass
constexpr int kKeysSpan = kKeysBlock * kKeysPer;
// Binning through tiles (k_bin, k_tiles), for calls whose largest event has at most
// kBinMaxRows rows, which is what the tables hold (a share per thread of k_tiles, two rows
// per thread of k_bin), not where the other binning overtakes it: whole builds of 2^20 rows
// of 3, 8, 12 and 32 floats 200, 286, 416 and 1,652 us through tiles and 250, 338, 467 and
// 1,726 by atomics, of one row more 252, 338, 476 and 1,737 (by atomics).  Shares of
// kKeysBlock or twice as many rows, at most kBinMaxShares an event; tiles of up to
// 2^kTileShiftMax cells and, on average, at most kTilePointsMin points: fewer leave the
// shares' segments of a tile too short, more too few tiles for the CUs (120k points: whole
// build 64.9, 65.3, 66.5 and 70.7 us with 256, 512, 1024 and 2048; 300k points 138.8,
// 138.0, 141.8, 141.5).  Calls of more than kTilePointsFrom rows have tiles enough for
// kTilePointsLarge (a batch of 5.6M rows 1754, 1651, 1639, 1660).
constexpr int kTilesBlock = 512;
constexpr int kBinMaxShares = 512;
constexpr int kBinMaxRows = kBinMaxShares * kKeysBlock * 2;
constexpr int kBinMaxTiles = 4096;
constexpr int kTileShiftMax = 12;
constexpr int kTilePointsMin = 512;
constexpr int kTilePointsLarge = 1024;
constexpr long long kTilePointsFrom = 1 << 19;
// Rows per share of a call (0: binning by atomics).
constexpr int bin_span_for(long long max_n) {
    return max_n > kBinMaxRows ? 0 : (max_n > kBinMaxShares * kKeysBlock ? 2 * kKeysBlock : kKeysBlock);
}
// Most tiles an event of n rows can have: n_cells / 2^shift rounded up, where with the shift
// at its largest n_cells <= cells_max, and below it n_cells / 2^shift < 2n / tile_points.
constexpr int bin_tiles_bound(long long n, int tile_points) {
    const long long by_points = (2 * n + tile_points - 1) / tile_points;
    const long long by_cells = ((2 * n > 32768 ? 2 * n : 32768) + (1 << kTileShiftMax) - 1) >> kTileShiftMax;
    return static_cast<int>(by_points > by_cells ? by_points : by_cells);
}
static_assert(bin_tiles_bound(kBinMaxRows, kTilePointsMin) <= kBinMaxTiles, "the tiles of an event fit k_bin's LDS");
// Tiles of many points are shared among workgroups of k_tiles: cells are of one size, so
// that points that crowd into few of them (narrow axes beside an outlier) would leave a
// whole event to one workgroup.  A tile of crowd_least points, eight times what a tile is
// aimed at, or more gets, beside its own workgroup, one for every half of crowd_least, from
// the blocks that the event's tiles leave over (for every whole, two, ... of crowd_least
// where those are too few).  Its points are counted before by the shares that hold many of
// them (crowd_reported: three quarters of the tile's mean share, so that a count comes short
// by less than three quarters of crowd_points); ordinary tiles' shares stay below and add
// nothing.  120k points in one tile: 581 us for the rows' stage by one workgroup, 61 in
// parts; the whole build 782 and 262 us, of 400k points 2,490 and 1,353.
// (tile_points is a power of two: quotients are shifts.)
constexpr int crowd_least(int tile_points) { return 8 * tile_points; }
constexpr int crowd_points(int tile_points, int shares) {
    return 16 * shares > crowd_least(tile_points) ? 16 * shares : crowd_least(tile_points);
}
constexpr bool crowd_reported(unsigned int points, int tile_points, int shares) {
    // (A product of 24-bit factors: at most 2,048 points and 512 shares.)
    return (points & 0xffffu) * ((4u * shares) & 0xffffu) >=
           3u * static_cast<unsigned int>(crowd_points(tile_points, shares));
}
// Where the counts of an event's tiles begin: an event of crowd_least rows and more has
// fewer than 2n / tile_points + 1 tiles, fewer than lie before the next event's.
constexpr long long crowd_at(long long row0, int tile_points) { return row0 >> (__builtin_ctz(tile_points) - 2); }
// Blocks of k_tiles for an event: its tiles at most, and some more where a tile may be
// crowded, so that there are always blocks over.
constexpr int tile_blocks(int n, int tile_points) {
    const int more = n < crowd_least(tile_points) ? 0 : (n >> (__builtin_ctz(tile_points) + 5)) + 2;
    return bin_tiles_bound(n, tile_points) + more;
}
// Log2 of the points per workgroup beside the tiles' own, for the sum of an event's counts.
constexpr int crowd_shift(unsigned int crowded, int n, int n_tiles, int tile_points) {
    int shift = __builtin_ctz(tile_points) + 2;
    while (crowded >> shift > static_cast<unsigned int>(tile_blocks(n, tile_points) - n_tiles)) ++shift;
    return shift;
}
constexpr int kPlaceBlock = 256;     // threads per workgroup of the placement pass
constexpr int kPlaceTile = 256;      // queries per workgroup of the placement pass (and kept tile)
constexpr int kKeptGroup = 64;       // kept tiles per group (one workgroup of the kept-totals pass)
constexpr int kSumsBlock = 1024;     // threads per workgroup of the kept-totals pass
constexpr unsigned int kWaveKeys = 512;  // hits of the longest list that one wave of the placement pass collects
constexpr int kOwnerWindow = 3072;   // output positions formed in LDS at a time in placement
constexpr int kPlaceWords = 4096;    // LDS words of placement: an output window, four waves' or one workgroup's hits
// Placement workgroups at least (all of them collect long lists): six per CU, so that
// many small events with long lists keep as many lists in flight as the CUs hold (50,000
// lists of a 60k-point event: whole build 175, 139, 127 and 129 us with 512, 1024, 1536
// and 2048; 2,000 points without any 55.0, 55.2, 55.0 and 55.2).
constexpr int kPlaceMinBlocks = 1536;
constexpr int kMaxEvents = 65535;  // events per call (the second grid dimension)
// A kept count with this bit set belongs to a long list (more than kListCap
// neighbours, or more than K without the search's own selection), which the
// placement pass collects again; other lists sit at kListCap slots per original row.
constexpr unsigned int kKeptLong = 1u << 31;
// With this bit the list has kListCap + 1 to kExtCap entries: the low bits hold the count,
// the bits between the number of its block of kListCap entries in the extension, where the
// entries past its first kListCap lie.  The search keeps up to search_spill(DP) such
// entries of a batch of queries (fewer where LDS would cost 48-float rows a workgroup).
// A few percent of the queries of an ordinary event have such lists; collected again one
// per wave they took the placement of a batch of 64 events (148,000 of 5.6M queries) to
// 457 us, against 254 from the extension, of a 120k-point event to 14.8 against 12.4 and
// of a 60k-point 32-D event to 16.1 against 11.6.  Denser graphs, whose spilled hits
// overflow, lose 1 to 2%.
constexpr unsigned int kKeptExt = 1u << 30;
constexpr int kKeptExtBits = 6;
constexpr unsigned int kKeptExtCount = (1u << kKeptExtBits) - 1u;
constexpr int kExtCap = 32;
constexpr int search_spill(int dpad) { return dpad == 48 ? 32 : 64; }
constexpr long long kExtBlocksMax = 1 << (30 - kKeptExtBits);

// One event of a call: its rows in the concatenated points and its share of the
// cell-key space.  The first event starts at row 0 and cell 0.
struct EventDesc {
    const float *pts;  // the event's points (device, row-major [n, d])
    long long row0;    // first row of the event in the call's row numbering
    long long cell0;   // first cell key of the event
    int n;             // rows of the event
    int cells_max;     // cells reserved for the event
    int tile0;         // first scan tile of the event's cells (cell0 / kScanTile)
    int pad;
};

// Per-block min/max of the binned coordinates and a non-finite flag.
struct BoundsPartial {
    float mn[kMaxAxes];
    float mx[kMaxAxes];
    int nonfinite;
    int pad;
};

// The grid of one event, derived on the device from its bounds.
// Axis 0 varies fastest in a cell key.  Axes past the binned count have one cell.
struct Plan {
    float lo[kMaxAxes];     // smallest binned coordinate per axis
    float inv_c[kMaxAxes];  // 1 / cell edge per axis (float32)
    float c[kMaxAxes];      // cell edge per axis
    int G[kMaxAxes];        // cells per axis
    int n_cells;            // product of G
    int reach;              // neighbour cells searched on each side, per axis
    int abort;              // a coordinate was NaN or infinite
    int axes;               // binned coordinates (3 or 4)
    int tile_shift;         // log2 of the cells per tile (set, as the next, where points are binned through tiles)
    int n_tiles;            // tiles of the event
};

// Bits per axis in a packed cell coordinate word (axis p at bits [p b, p b + b)).
__host__ __device__ constexpr int cell_bits(int axes) { return axes == 4 ? 8 : 10; }

// Single-address atomics serialise across the chip (about 11 ns each), so these
// are touched only by rare events (bad input) or once.
struct Counters {
    unsigned int abort;            // some event had a non-finite coordinate
    unsigned int capped;           // queries with more than K neighbours (summed after the search)
    unsigned long long tested;     // pairs examined, summed over the search workgroups
    unsigned long long survived;   // pairs that reached the second stage, likewise
};

// Counts of one search workgroup.  They lie in the ranks' memory: a workgroup has at
// least 16 rows beyond the first eight (kMinWaveRows), so the ranks are the larger.
struct SearchCounts {
    unsigned long long tested;    // pairs examined
    unsigned long long survived;  // pairs that reached the second stage
    unsigned int capped;          // queries with more than K neighbours
    unsigned int pad;
};

// Result summary copied to the host at the end of a call (event 0's grid).
struct Report {
    long long n_edges;
    unsigned long long tested;
    unsigned long long survived;  // pairs that passed the first-stage partial test
    int abort;
    unsigned int capped;
    unsigned int heavy;
    int n_cells;
    int G[kMaxAxes];
    float c[kMaxAxes];
};

// Device buffers of one call, carved from the caller's workspace.
struct Workspace {
    EventDesc *ev;              // [n_events]
    Plan *plans;                // [n_events]
    BoundsPartial *part;        // [n_events * kBoundsBlocks]
    Counters *ctr;
    Report *report;
    long long *edge_off;        // [n_events + 2] first edge of each event, then E, then a status; before the
                                // search, the sums of the events' counts of crowded tiles
    unsigned int *pcell;        // [rows] packed cell coordinates of each point; with rank, the tile binning's entries
    unsigned int *rank;         // [rows] arrival rank inside its cell; from the search on, the SearchCounts
    unsigned int *cell_count;   // [cells] histogram or the tile binning's tables; in the search, the extension
    unsigned int *cell_start;   // [cells + 1] exclusive scan of the histogram
    unsigned long long *sums_cells;  // [tiles of cells + 1] per-tile histogram totals
    unsigned long long *sums_kept;   // [tiles of kPlaceTile rows] kept neighbours before the tile in its group
    unsigned long long *sums_kept2;  // [groups of kKeptGroup tiles] per-group kept totals
    float *sorted;              // [rows, dpad] points in cell order, zero-padded rows
    unsigned int *sorted_id;    // [2 rows] per sorted row: its original row, then its packed cell
    unsigned int *kept;         // [rows] kept word per original row: the neighbours kept (| kKeptLong for a long
                                // list), or kKeptExt, the list's block of the extension and the count; before
                                // the search, the counts of crowded tiles (crowd_at)
    unsigned int *long_slots;   // [rows] sorted rows of the queries with long lists, queued per XCD in the part
                                // of the XCD's rows
    unsigned int *temp;         // [rows * kListCap] neighbour lists of up to kListCap entries
    unsigned int *wave_start;   // [kMaxPieceCount + 1] first sorted row of each search piece
    unsigned int *claims;       // [8 kClaimStride] each XCD's counts of long lists and of extension blocks;
                                // cleared by the pass before the search that cuts the pieces
    long long rows;
    long long cells;
    int tiles_cells_n;
    int tiles_kept_n;
    int groups_kept_n;
    size_t total_bytes;
};

int64_t cells_max_for(int64_t n);
int dpad_for(int d);
// Fills descs[e] (if not null) for events given by row offsets; returns the total
// cell count (pts stays null; callers set it).
long long describe_events(const int64_t *event_offsets, int n_events, EventDesc *descs);
// Workspace layout for events of the given sizes (host arithmetic; base may be null).
Workspace layout(void *base, long long rows, long long cells, int n_events, int d);

// Pinned host memory that the kernels of a call write its result into; one per calling
// thread, so it serves whichever device is current in a call: it is portable, and its
// address is asked for again when another device is.
struct MappedResult {
    void *host = nullptr;
    void *dev = nullptr;  // the current device's address, or null (the result is copied back)
    int device = -1;      // the device that dev belongs to
    bool mapped = false;
    // For the current device; false if there is no pinned memory.
    bool ready(size_t bytes) {
        if (!host) {
            mapped = hipHostMalloc(&host, bytes, hipHostMallocMapped | hipHostMallocCoherent | hipHostMallocPortable) ==
                     hipSuccess;
            if (!mapped) {
                (void)hipGetLastError();
                host = nullptr;
                if (hipHostMalloc(&host, bytes, hipHostMallocPortable) != hipSuccess) {
                    host = nullptr;
                    return false;
                }
            }
        }
        int now = 0;
        if (hipGetDevice(&now) != hipSuccess) return false;
        if (mapped && now != device) {
            if (hipHostGetDevicePointer(&dev, host, 0) != hipSuccess) {
                (void)hipGetLastError();
                dev = nullptr;
            }
            device = now;
        }
        return true;
    }
};

struct LaunchArgs {
    int vec4;           // every event's rows are 16-byte aligned float4 groups (d % 4 == 0)
    int n_events;
    int max_n;          // rows of the largest event
    int d;
    int dpad;
    int axes;           // binned coordinates (3 or 4)
    int dims[kMaxAxes]; // binned coordinates, axis 0 first (unused entries -1)
    float r;
    float r2;
    int K;
    int cell_div;
    unsigned long long edge_capacity;
    long long *src;
    long long *dst;
    hipStream_t stream;
    hipEvent_t *events;     // 8 events bracketing the 7 stages (without the one before the scatter when
                            // points are binned through tiles), or null
    int search_blocks;      // resident workgroups of the search kernel
    int search_prio;        // 1: the search grid is one round of resident workgroups
    int bounds_blocks;      // bounds partials per event (<= kBoundsBlocks)
    int bin_span;           // rows per share of the binning through tiles, or 0 (by atomics)
    int tile_points;        // points per tile aimed at
    EventDesc ev0;          // event 0, written to ws.ev by the first kernel when ev_from_arg
    int ev_from_arg;
    long long *edge_off_out;  // device [n_events + 2] for the edge ranges and status, or null (workspace)
    Report *report_out;       // device-visible pinned host report, or null (workspace)
};

// Enqueues the whole pipeline on a.stream; the report lands in ws.report and the
// per-event edge ranges in ws.edge_off.
hipError_t enqueue_build(const LaunchArgs &a, const Workspace &ws);

// Resident workgroups of the search kernel for rows padded to dpad (current device);
// sel: the variant for K below the list size, four: for four binned axes.
int search_blocks_for(int dpad, bool sel, bool four);

}  // namespace frnn
