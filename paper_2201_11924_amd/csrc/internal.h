// Internal declarations shared by the library's translation units (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/simsense.h"

namespace ss {

// Lanes that cooperate on one scanline: exactly one DPP row of a wave64, so
// every cross-lane step of the path recurrence is a row-local DPP operation.
constexpr int kLanesPerLine = 16;

// Disparities held by each lane; the padded disparity count is 16 * dpl.
int pick_dpl(int max_disp);
inline int padded_disp(int max_disp) { return kLanesPerLine * pick_dpl(max_disp); }
int census_bits(int cw, int ch, int mode);

// Path directions: 2 paths = horizontal pair, 4 adds the vertical pair, 8 adds
// the four diagonals (same order as the header documents).
extern const int kPathDx[8];
extern const int kPathDy[8];
int path_lines(int dx, int dy, int W, int H);
// Default lanes per horizontal line of the slots of a batch, the widest with W pixels a row,
// from its total_work (the sum of aggregate_work over them), and of one pair by the same rule
// but for the cases below.  More lanes shorten the chain of a row's steps, fewer spend less on
// the steps' cross-lane part.  Measured aggregation passes, 16 / 32 / 64 lanes, at the work
// per SIMD over a row's work (for one pair that is H / 8192 times twice the walks: W and the
// disparities stand in both):
//   0.66 (960x540, D = 96, 4 paths) 160 / 122 us;  1.3 (848x480, D = 128, 8) 169 / 143 / 187;
//   1.9 (1280x720, D = 128, 8) 271 / 308 / 334;
//   16 pairs of 1280x720, 2 paths, with the net: 2805 / 3043 / 3685.
int launch_lanes(int W, int dpad, int64_t total_work);
// One pair: rows alone (2 paths) of up to 192 disparities take the most lanes with which no
// SIMD has two waves, whole calls: 640x480 D = 128 99 / 72 / 65, 891x596 D = 96 179 / 141 /
// 159, 154x598 D = 160 64 / 51 / 56, 804x837 D = 96 174 / 140 / 156, 686x1052 D = 192 217 /
// 226 / 274, 1539x1041 D = 160 570 / 581 / 732, 1812x1307 D = 96 420 / 434 (with 256 the wider
// forms stay level: 686x871 285 / 219 / 224, 1190x1608 568 / 563 / 658).  4 paths that count
// census words of up to 192 disparities gain nothing from 32 lanes where the rows have more
// than one wave a SIMD (H > 1024) and rows and columns together (H + W / 2) more than two:
// 1920x1080 D = 192 (2040) 856 / 757, 1749x1160 (2034) 856 / 770, 1863x1120 (2051) 867 / 925,
// 2062x1080 (2111) 905 / 989, 2055x1200 D = 128 (2227) 689 / 762, 2379x1250 D = 192 1113 /
// 1141; but 3715x658 D = 256 (2515) 1589 / 1330.
int default_lanes(int W, int H, int dpad, int num_paths, bool costs, bool sums);
// The lanes a tuning stands for (asked; 0 the default).  64 cannot be asked for with 96
// disparities, which they do not divide, but are the default of launches short of rows
// (100x201, 2 paths: 27 us a call, with 32 lanes 29, with 16 36): there 32 stand for them, or
// every tuned handle would be slower than an untuned one.
int chosen_lanes(int asked, int dpad, int by_default);
int64_t aggregate_work(int W, int H, int dpad, int num_paths, bool sums);
// Whether the vertical and diagonal directions read a cost volume by default, rather than
// count census words.  Each of them reads it once, so a volume beyond the caches costs more
// than the counting, the sooner the more directions there are and the less is won by it:
// sums of two directions (sums) save half the planes, 64-bit words (wide) cost twice the
// counting, and so do 256 disparities of 8 directions.  Whole calls in us, volume / words:
//   8 directions, no sums: 960x540 D = 128 (66 MB) 272 / 281, D = 192 (100 MB) 414 / 396,
//   1280x720 D = 128 (118 MB) 461 / 454, 1600x1000 D = 128 (205 MB) 774 / 724, 1539x1041
//   D = 192 (308 MB) 1479 / 1072; D = 256: 1280x720 888 / 1095, 1920x1080 2220 / 2310;
//   with sums, 1280x720 D = 128: 405 / 458, 1920x1080 D = 256: 1660 / 2310.
//   4 directions: 1416x1048 D = 128 (190 MB) 0.91 (volume over words), 1755x1046 (235 MB) 1.05,
//   1439x741 D = 192 (205 MB) 0.94, 1565x782 (235 MB) 1.12, 1821x1086 D = 96 (190 MB) 1.01,
//   1804x1270 (220 MB) 1.08, 2389x1340 D = 64 (205 MB) 1.21, 2410x1620 (250 MB) 1.31; with
//   sums 1627x1056 D = 128 (220 MB) 1.05, 1920x1080 (265 MB) 601 / 556 us, D = 192 (398 MB) 873
//   / 756; with rows as sums too (below), 2400x1500 D = 96 831 / 882.
//   64-bit words: 1280x720 D = 128, 8 directions 498 / 938, 1920x1080 D = 192 1803 / 1890.
// Where columns are the longest chains and there are few of them, a launch waits for their
// steps, which counting makes longer, and not for memory (volume over words, 8 directions,
// no sums): 397x2051 D = 192 (156 MB) 0.86, 925x1139 D = 128 (135 MB) 0.97, 693x2160 D = 128
// (192 MB) 0.90, 1693x2826 D = 32 (153 MB) 1.15, 734x1615 D = 192 (228 MB) 1.01, 430x2766
// (228 MB) 0.89, 762x2892 (423 MB) 1.23; 4 directions: 701x3030
// D = 128 (272 MB) 0.90, 955x2481 D = 192 (455 MB) 1.26, with sums 805x4164 (644 MB) 0.84.
// And 4 directions of 256 disparities: 1050x960 (258 MB) 0.96, 1885x818 (395 MB) 1.06,
// 1605x1541 (633 MB) 1.29, 568x3646 (530 MB) 0.72, with sums 1050x960 0.90, 2032x676 (352 MB)
// 1.00, 1428x1473 (538 MB) 1.04.
bool default_costs(int W, int H, int dpad, int num_paths, bool wide, bool sums);
// Whether the horizontal directions are stored as sums by default: where the cost volume
// does not fit the 256 MB last-level cache, so that the aggregation waits for HBM, one
// buffer less is worth a third walk over the rows (1920x1080, D = 256: whole call 1762 ->
// 1682 us; 1280x720, D = 128: 423 -> 429; 16 pairs in a batch: no change).
bool default_row_sums(int W, int H, int dpad, int num_paths, bool wide, int hl);
bool horizontal_lanes_valid(int dpad, int hl);
// Disparities a lane of a line of `lanes` lanes holds: a whole number of words in
// memory (lanes past the padded count idle), or 1 or 2.
__host__ __device__ constexpr int lane_disparities(int dpad, int lanes)
{
    return dpad <= lanes ? 1 : dpad <= 2 * lanes ? 2 : dpad <= 4 * lanes ? 4 : dpad <= 8 * lanes ? 8 : dpad <= 12 * lanes ? 12 : 16;
}
// The same of a horizontal line: with 32-bit census words the 32 lanes of 192 disparities
// hold 6 each, an even lane storing its neighbour's with its own (8 each, with 8 lanes idle,
// take a third more instructions per step: 1280x720, D = 192, 4 directions 422 -> 403 us a
// call, 640x480, 8 directions 258 -> 248; three 16-bit stores a lane instead 407, 253).
__host__ __device__ constexpr int row_disparities(int dpad, int lanes, bool wide)
{
    return !wide && dpad == 6 * lanes && lanes == 32 ? 6 : lane_disparities(dpad, lanes);
}
// And of a vertical or diagonal line that counts census words: 96 disparities as 6 each.
__host__ __device__ constexpr int column_disparities(int dpad) { return dpad == 96 ? 6 : lane_disparities(dpad, kLanesPerLine); }
// lanes a horizontal line runs with when hl are asked for: as many as hold two or more
// disparities each, most of them in use
__host__ __device__ constexpr int effective_lanes(int dpad, int hl)
{
    return hl == 64 && dpad >= 96 ? 64 : hl >= 32 && dpad >= 64 ? 32 : kLanesPerLine;
}
// Estimated instructions per step of a line: about 4 per disparity a lane holds,
// plus the per-step line overhead (larger for lines spread over more than one DPP
// row).
__host__ __device__ constexpr int agg_step_cost(int dpl, int lanes_per_line) { return 4 * dpl + (lanes_per_line == 16 ? 12 : 18); }

// One slot's aggregation: its units in launch order.  A unit is one direction, or a
// direction with its opposite (pair: the buffer receives the sum of both path
// values); item i of a unit is the lines of one block: four waves' (one per SIMD of a
// compute unit), or for a pair two waves', each walked by two waves.
constexpr int kWavesPerItem = 4;
// Lines of an item of a vertical or diagonal direction whose columns count census words:
// neighbours in one image row at every clock (aggregate_impl.h, run_columns).
constexpr int kColumnLines = 16;
struct ColumnLines {
    int v0, n;           // column at clock 0 of line 0, and how many lines exist
    int begin, end;      // clocks at which any of them has a pixel
    int all_in, any_out; // and at which all of them have: from all_in to before any_out
};
__host__ __device__ inline ColumnLines column_lines(int dx, int item, int W, int H)
{
    constexpr int kLines = kColumnLines;
    auto lo = [](int a, int b) { return a < b ? a : b; };
    auto hi = [](int a, int b) { return a > b ? a : b; };
    ColumnLines g;
    const int total = dx == 0 ? W : W + H - 1;
    g.v0 = item * kLines - (dx > 0 ? H - 1 : 0);
    g.n = lo(kLines, total - item * kLines);
    const int v1 = g.v0 + g.n - 1;
    // line v has pixels at the clocks max(0, -v) .. min(H, W - v) - 1 (dx > 0),
    // max(0, v - W + 1) .. min(H, v + 1) - 1 (dx < 0)
    g.begin = dx == 0 ? 0 : hi(0, dx > 0 ? -v1 : g.v0 - W + 1);
    g.end = dx == 0 ? H : lo(H, dx > 0 ? W - g.v0 : v1 + 1);
    g.all_in = dx == 0 ? 0 : hi(0, dx > 0 ? -g.v0 : v1 - W + 1);
    g.any_out = dx == 0 ? H : lo(H, dx > 0 ? W - v1 : g.v0 + 1);
    return g;
}

struct AggregateArgs {
    const void *census_l, *census_r;  // uint32 words, or uint64 when bits > 32
    uint8_t *cost;       // cost volume the vertical and diagonal units read (null: they count census
                         // words, or there are none); for block matching the 16-bit block costs of
                         // every unit
    int row_costs;       // the horizontal units read it too (else the census words)
    int W, H, D, Dpad, bits, p1, p2;
    int nunits;
    int last_first;      // units from here on run after all others (they write over `cost`)
    int dx[8], dy[8], pair[8];
    int item_begin[9];   // first item index of each unit, prefix sums
    uint8_t *out[8];     // per-unit path values, W*H*Dpad values, d fastest
    int max_item_work;   // largest item work of the launch (issue priorities)
};
// whether there are vertical and diagonal units that count census words
inline bool counts_census(const AggregateArgs &a) { return !a.cost && a.nunits > 2; }
// Whether horizontal directions may be stored as sums too: 16 lanes per line and
// 32-bit census words (64-bit ones take more registers than a wave has).
__host__ __device__ constexpr bool row_pairs_built(int lanes, bool wide) { return lanes == kLanesPerLine && !wide; }
// Path buffers of a slot: one per direction, and one more for the cost volume where the
// directions need them all (no sums) and the caller can spare it.
constexpr int path_buffers(int num_paths, bool costs, bool sums, bool spare) { return num_paths + (costs && !sums && spare ? 1 : 0); }
// Whether a slot without that buffer keeps the volume in the last direction's and runs that
// direction after all others, in place, rather than counting census words along columns and
// diagonals: where the words are 64 bits or the disparities 256.  The no-allocation call
// with planes that fill its array, in us, in place / words: 64-bit, 250x230, D = 128 96 /
// 140; D = 256, 171x176 104 / 110; but 320x240, D = 96 102 / 72, 200x200, D = 192 99 / 81.
constexpr bool costs_in_place(int dpad, bool wide) { return wide || dpad == 256; }
// Fills a's units for the nbuffers `buffers` and hl lanes per horizontal line, from W, H
// and Dpad.  sums: opposite directions are stored as their sums (two path
// values must fit one value of the buffer); row_sums: the horizontal ones too.  Unit u
// fills buffers[u].  block: a.cost is the caller's and every unit reads it.
void plan_aggregation(AggregateArgs &a, int num_paths, bool costs, bool sums, bool row_sums, bool block, int hl,
                      uint8_t *const *buffers, int nbuffers);
int aggregate_item_work(const AggregateArgs &a, int unit, int item, int hl);

struct SelectArgs {
    const uint8_t *paths[8];  // path values or sums of two, 8-bit, or 16-bit when values16
    int values16;
    int nplanes;              // buffers to sum (the aggregation's units)
    int W, H, D, Dpad;
    int uniqueness_pct, lr_max_diff, subpixel;
    int small_values;     // every path value < 128 (bits + P2 <= 127), the first two buffers single ones
    uint8_t *disp_int;    // W*H
    uint16_t *cost_best;  // W*H
    uint16_t *cost_second;
    uint8_t *disp_right;
    float *disp_sub;      // before masking
    float *masked;        // masked sub-pixel disparity (0 = invalid)
    uint8_t *flags;       // bits 0..2
    int no_right;         // skip the right-image disparity (no LR check, disp_right unwritten)
};

struct PostArgs {
    const float *masked;
    const uint8_t *flags_in;
    int W, H, median;
    float fb;
    float *disp;     // may be null
    float *depth;    // may be null
    uint8_t *flags;  // may be null
};

hipError_t launch_ir_noise(const uint8_t *in, const float *gamma, const float *n, uint8_t *out,
                           int64_t count, hipStream_t s);
// (zero, nzero: words the census launch clears on the way, if a caller has any)
hipError_t launch_census(const uint8_t *img, int pitch, int W, int H, int cw, int ch, int mode,
                         void *out, bool out64, hipStream_t s, unsigned *zero = nullptr, int nzero = 0);
// both images of a pair in one launch (img1 may be null: img0 alone)
hipError_t launch_census_pair(const uint8_t *img0, const uint8_t *img1, int pitch, int W, int H, int cw, int ch,
                              int mode, void *out0, void *out1, bool out64, hipStream_t s, unsigned *zero = nullptr,
                              int nzero = 0);
// every slot of a batch phase, or a handle's own single slot
struct AggregateQueue {
    const AggregateArgs *slots;  // per pair slot (device)
    const uint32_t *items;       // slot << 20 | item, largest work first (device)
    int census;                  // the slots' vertical and diagonal units count census words
    const uint32_t *cost_items;  // slot << 20 | row of the slots whose costs go to a volume (device)
    int ncost, cost_width;       // their number, and the widest image among them
};
hipError_t launch_aggregate(const AggregateArgs &a, bool wide, int hl, hipStream_t s);
// grid: the items (one block each)
hipError_t launch_aggregate_queue(const AggregateQueue &q, int dpad, bool wide, int hl, int grid, hipStream_t s);
hipError_t launch_select(const SelectArgs &a, hipStream_t s);
hipError_t launch_post(const PostArgs &a, hipStream_t s);
// Semi-global block matching: the block-cost volume and the aggregation fed
// from it (16-bit path values, one block per line block).
constexpr int kMaxBlockHalf = 15;  // SGBM blocks are at most 31 x 31
// lanes per horizontal line of the block-cost-fed aggregation
__host__ __device__ constexpr int volume_horizontal_lanes(int dpad)
{
    return effective_lanes(dpad, dpad == 128 || dpad == 256 ? 64 : 32);
}
struct BlockCostArgs {
    const void *census_l, *census_r;  // uint32 words, or uint64 when bits > 32
    int W, H, D, bits, bw, bh;
    uint16_t *vol;                    // W*H*Dpad, d fastest
};
// cost of the padding disparities of a block-cost volume: no block cost plus P2
// exceeds it
constexpr int kBlockPadCost = 8191;
struct VolumeArgs {
    AggregateArgs a;  // cost: the block-cost volume; 16-bit path values
};
hipError_t launch_block_cost(const BlockCostArgs &a, int dpad, bool wide, hipStream_t s);
hipError_t launch_aggregate_volume(const VolumeArgs &a, hipStream_t s);

// x-flip of a census map (words of 4 or 8 bytes)
hipError_t launch_flip_census(const void *src, void *dst, int W, int H, bool wide, hipStream_t s);
// LR check against a full right-referenced run whose winners are given in
// x-flipped order (dint_m[y][W-1-xr] = dR(xr)): rewrites flag bit 1 and the
// masked disparity, and writes the right disparities
struct LRFullArgs {
    const uint8_t *dint, *dint_m;
    const float *disp_sub;
    uint8_t *flags;      // in: bits 0 and 2 of the left selection; out: bit 1 rewritten
    float *masked;
    uint8_t *disp_right;
    int W, H, lr;
};
hipError_t launch_lr_full(const LRFullArgs &a, hipStream_t s);

// batched forms: per-slot arguments in device memory, one block per item
// (slot << 20 | index), items in device memory
struct CensusJob {
    const uint8_t *img;
    int pitch, W, H, cw, ch, mode;
    void *out;
};
struct CensusBatch {
    const CensusJob *jobs;
    const uint32_t *items;
    int nitems, max_cw, max_ch;
};
struct SelectBatch {
    const SelectArgs *slots;
    const uint32_t *items;  // slot << 20 | row
    int nitems, max_width;
    int no_right;           // as SelectArgs::no_right, for every slot of the launch
};
constexpr int kPostTileRows = 16;  // rows of a batch's post tile (64 columns)
struct PostBatch {
    const PostArgs *slots;
    const uint32_t *items;  // slot << 20 | tile (64 x kPostTileRows, row-major)
    int nitems;
};
hipError_t launch_census_batch(const CensusBatch &b, bool out64, hipStream_t s);
hipError_t launch_select_batch(const SelectBatch &b, int dpad, int nplanes, bool small, hipStream_t s);
hipError_t launch_post_batch(const PostBatch &b, hipStream_t s);
int census_tiles(int W, int H);
struct PathSet {
    const uint8_t *p[8];
};
hipError_t launch_volume_sum(const PathSet &paths, int nplanes, bool values16, int W, int H, int D, int Dpad,
                             uint16_t *out, hipStream_t s);

// ---------------------------------------------------------------- handle
// Parameter validation (a simsense_status) and the handle's scratch layout: one
// block holding the census maps, the per-direction path values, the per-pixel
// results (and for lr_mode 1 a second set; for SGBM the block-cost volume),
// every piece 256-byte aligned.
int validate(const simsense_params *p);
struct Layout {
    size_t census, paths, per_px[7], total;
    int buffers;       // path buffers
    bool costs, sums;  // vertical and diagonal directions read a cost volume; opposite ones are stored as sums
    bool right_run;  // lr_mode 1: two more census maps and a second per-pixel set
    size_t volume;   // SGBM: the block-cost volume (16-bit, d fastest)
};
// (spare: with a buffer for the cost volume where the directions fill all others)
Layout layout(const simsense_params *p, bool spare);
bool sums_fit(const simsense_params *p);     // two path values fit one of the path buffers'
bool default_costs(const simsense_params *p);  // (above) for a handle's or a batch slot's parameters

// fields derived from the parameters; the buffers carved from `base` (l.total bytes)
void init_handle(simsense_handle *h, const simsense_params *params, const Layout &l);
void carve_scratch(simsense_handle *h, uint8_t *base, const Layout &l);
// the handle's aggregation units for its lane count (its buffers are set)
void plan_handle(simsense_handle *h);
// Work common to the compute entry points; each returns a simsense_status.
//  enqueue_match: census, aggregation and selection into the handle's scratch
//                 (d*, S1, S2, dR, sub-pixel, masked disparity, flags bits 0..2);
//  enqueue_post:  median + depth of a masked map into the caller's outputs.
//                 (volume_out, if set, receives the summed path costs S)
//                 (need_right = false: the learned form, which reads only d*, S1,
//                 S2 and the sub-pixel disparity, skips the right-image disparity)
int enqueue_match(simsense_handle *h, const uint8_t *left, const uint8_t *right, int pitch, hipStream_t s,
                  uint16_t *volume_out = nullptr, bool need_right = true);
int enqueue_post(simsense_handle *h, const float *masked, const uint8_t *flags_pre, const simsense_outputs *o,
                 hipStream_t s);
int profile_begin_call(simsense_handle *h);
void profile_end_call(simsense_handle *h);
void profile_mark(simsense_handle *h, int pass, bool end, hipStream_t s);

}  // namespace ss

struct simsense_handle {  // opaque to callers
    simsense_params p;
    int bits, Dpad, ndirs;
    int hlanes;  // lanes per horizontal scanline
    bool wide;
    // launch shape of the aggregation; for the sorted form, the work list (items
    // largest first, then the cost rows) and the argument block on the device
    simsense_batch_tuning tuning;
    int nitems, ncost;
    uint32_t *d_items;
    ss::AggregateArgs ag;  // the aggregation's units, set with the tuning
    ss::AggregateArgs *d_args;
    bool costs;    // the vertical and diagonal directions read a cost volume
    bool sums;     // opposite directions are stored as their sum
    bool row_sums; // the horizontal directions are stored as their sum
    // full right-referenced run (lr_mode 1): x-flipped census maps (the right
    // image's as the reference), that run's per-pixel results and its arguments
    void *census_ml, *census_mr;
    uint8_t *disp_int_m, *disp_right_m, *flags_m;
    uint16_t *cost_best_m, *cost_second_m;
    float *disp_sub_m, *masked_m;
    ss::AggregateArgs *d_args_m;
    // semi-global block matching: 16-bit path values fed from a block-cost volume
    bool sgbm;
    uint16_t *volume;
    void *block;
    void *census_l, *census_r;
    uint8_t *paths[9];
    int nbuffers;
    uint8_t *disp_int, *disp_right, *flags_pre;
    uint16_t *cost_best, *cost_second;
    float *disp_sub, *masked;
    hipStream_t last_stream;
    // profiling: call slots of 2 events per pass
    bool profiling;
    int prof_used;
    int prof_calls;
    double prof_ms[SIMSENSE_NUM_PASSES];
    hipEvent_t *prof_events;
};
