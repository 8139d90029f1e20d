// Host side of the aggregation pass: its units and items, and dispatch to the
// per-disparity-count instantiations (agg_dpl*.hip).
#include <algorithm>

#include "internal.h"

namespace ss {

hipError_t launch_agg_dpl1(const AggregateArgs *a, const AggregateQueue *q, int grid, int hl, bool wide, hipStream_t s);
hipError_t launch_agg_dpl2(const AggregateArgs *a, const AggregateQueue *q, int grid, int hl, bool wide, hipStream_t s);
hipError_t launch_agg_dpl4(const AggregateArgs *a, const AggregateQueue *q, int grid, int hl, bool wide, hipStream_t s);
hipError_t launch_agg_dpl6(const AggregateArgs *a, const AggregateQueue *q, int grid, int hl, bool wide, hipStream_t s);
hipError_t launch_agg_dpl8(const AggregateArgs *a, const AggregateQueue *q, int grid, int hl, bool wide, hipStream_t s);
hipError_t launch_agg_dpl12(const AggregateArgs *a, const AggregateQueue *q, int grid, int hl, bool wide, hipStream_t s);
hipError_t launch_agg_dpl16(const AggregateArgs *a, const AggregateQueue *q, int grid, int hl, bool wide, hipStream_t s);

namespace {
hipError_t launch_agg(const AggregateArgs *a, const AggregateQueue *q, int grid, int dpad, int hl, bool wide,
                      hipStream_t s)
{
    switch (dpad / kLanesPerLine) {
    case 1: return launch_agg_dpl1(a, q, grid, hl, wide, s);
    case 2: return launch_agg_dpl2(a, q, grid, hl, wide, s);
    case 4: return launch_agg_dpl4(a, q, grid, hl, wide, s);
    case 6: return launch_agg_dpl6(a, q, grid, hl, wide, s);
    case 8: return launch_agg_dpl8(a, q, grid, hl, wide, s);
    case 12: return launch_agg_dpl12(a, q, grid, hl, wide, s);
    case 16: return launch_agg_dpl16(a, q, grid, hl, wide, s);
    default: return hipErrorInvalidValue;
    }
}

int line_length(int dx, int dy, int l, int W, int H)
{
    if (dy == 0) return W;
    if (dx == 0) return H;
    if (l < W) return std::min(dx > 0 ? W - l : l + 1, H);
    return std::min(W, H - 1 - (l - W));
}

// lines of one item of a unit
int item_lines(const AggregateArgs &a, int unit, int hl)
{
    const int lanes = a.dy[unit] == 0 ? effective_lanes(a.Dpad, hl) : kLanesPerLine;
    return 64 / lanes * kWavesPerItem / (a.pair[unit] ? 2 : 1);
}
}  // namespace

bool horizontal_lanes_valid(int dpad, int hl)
{
    return (hl == 16 || hl == 32 || hl == 64) && dpad % hl == 0;
}

int64_t aggregate_work(int W, int H, int dpad, int num_paths, bool sums)
{
    const int walks = sums ? 2 * 2 + 3 * (num_paths - 2) : 2 * num_paths;  // twice the walks over the image
    return (int64_t)W * H / 4 * walks / 2 * agg_step_cost(lane_disparities(dpad, kLanesPerLine), kLanesPerLine);
}

constexpr int kSimds = 1024;

int launch_lanes(int W, int dpad, int64_t total_work)
{
    const int64_t row = (int64_t)W * agg_step_cost(lane_disparities(dpad, kLanesPerLine), kLanesPerLine);
    const int64_t per_simd = total_work / kSimds;
    return 10 * per_simd >= 16 * row ? 16 : 10 * per_simd >= 5 * row ? 32 : 64;
}

int default_lanes(int W, int H, int dpad, int num_paths, bool costs, bool sums)
{
    if (num_paths == 2 && dpad < 256) return H > kSimds ? 16 : 2 * H > kSimds ? 32 : 64;
    const int hl = launch_lanes(W, dpad, aggregate_work(W, H, dpad, num_paths, sums));
    return num_paths == 4 && !costs && dpad < 256 && hl == 32 && H > kSimds && H + W / 2 > 2 * kSimds ? 16 : hl;
}

int chosen_lanes(int asked, int dpad, int by_default)
{
    if (asked == 0) return by_default;
    return dpad == 96 && asked == 32 && by_default == 64 ? 64 : asked;
}

bool default_costs(int W, int H, int dpad, int num_paths, bool wide, bool sums)
{
    if (num_paths == 2) return false;
    const int64_t volume = (int64_t)W * H * dpad, kFew = 96000000, kTall = 192000000, kVast = 400000000;
    const int64_t kMany = dpad <= 64 ? 160000000 : dpad == 96 ? 190000000 : 228000000;
    if (wide || volume <= kFew) return true;
    const bool few_columns = H > W && num_paths * W < (volume <= kTall ? 8000 : 5700);
    if (few_columns && (sums || dpad == 256 || volume <= kVast)) return true;
    if (num_paths == 8) return sums || dpad == 256;
    if (dpad == 256) return sums || volume <= kVast;
    return volume <= kMany || (sums && default_row_sums(W, H, dpad, num_paths, wide,
                                                        default_lanes(W, H, dpad, num_paths, true, true)));
}

bool default_row_sums(int W, int H, int dpad, int num_paths, bool wide, int hl)
{
    return num_paths > 2 && row_pairs_built(effective_lanes(dpad, hl), wide) && (int64_t)W * H * dpad > (int64_t)256 << 20;
}

// Units.  Horizontal directions are units of their own unless row_sums (their lines
// are the longest chains: walking them one and a half times holds up the launch).  They
// count census bits themselves where that is one word a pixel, and read the volume where
// it is two (641x479, D = 100, full census: aggregation 215 -> 176 us; one word,
// 1280x720: 277 -> 289 us).  The cost volume takes the last path buffer: sums leave it
// free; otherwise, without a spare one, the direction that fills it runs after all others
// and replaces each cost by its path value (each is read once, before it is overwritten).
void plan_aggregation(AggregateArgs &a, int num_paths, bool costs, bool sums, bool row_sums, bool block, int hl,
                      uint8_t *const *buffers, int nbuffers)
{
    if (!block) a.cost = costs ? buffers[nbuffers - 1] : nullptr;
    a.row_costs = a.cost && (block || a.bits > 32);
    a.nunits = 0;
    for (int r = 0; r < num_paths; ++r) {
        const bool pair = sums && (kPathDy[r] != 0 || row_sums);
        if (pair && (kPathDy[r] < 0 || (kPathDy[r] == 0 && kPathDx[r] < 0))) continue;  // stored with its opposite
        const int u = a.nunits++;
        a.dx[u] = kPathDx[r];
        a.dy[u] = kPathDy[r];
        a.pair[u] = pair;
        a.out[u] = buffers[u];
    }
    a.last_first = a.cost && a.out[a.nunits - 1] == a.cost ? a.nunits - 1 : a.nunits;
    a.item_begin[0] = 0;
    a.max_item_work = 1;
    for (int u = 0; u < a.nunits; ++u) {
        const int lines = item_lines(a, u, hl), n = (path_lines(a.dx[u], a.dy[u], a.W, a.H) + lines - 1) / lines;
        a.item_begin[u + 1] = a.item_begin[u] + n;
        for (int i = 0; i < n; ++i) a.max_item_work = std::max(a.max_item_work, aggregate_item_work(a, u, i, hl));
    }
}

int aggregate_item_work(const AggregateArgs &a, int unit, int item, int hl)
{
    const int dx = a.dx[unit], dy = a.dy[unit], n = path_lines(dx, dy, a.W, a.H);
    const int lines = item_lines(a, unit, hl), lanes = dy == 0 ? effective_lanes(a.Dpad, hl) : kLanesPerLine;
    int len = 0;
    if (counts_census(a) && dy != 0) {
        const ColumnLines g = column_lines(dx, item, a.W, a.H);
        return (g.end - g.begin) * agg_step_cost(column_disparities(a.Dpad), lanes);
    }
    for (int l = item * lines; l < std::min(n, (item + 1) * lines); ++l) len = std::max(len, line_length(dx, dy, l, a.W, a.H));
    const int steps = a.pair[unit] ? 3 * len / 2 : len;  // of each wave, in a row
    return steps * agg_step_cost(dy == 0 ? row_disparities(a.Dpad, lanes, a.bits > 32) : lane_disparities(a.Dpad, lanes), lanes);
}

hipError_t launch_aggregate(const AggregateArgs &a, bool wide, int hl, hipStream_t s)
{
    return launch_agg(&a, nullptr, a.item_begin[a.last_first], a.Dpad, hl, wide, s);
}

hipError_t launch_aggregate_queue(const AggregateQueue &q, int dpad, bool wide, int hl, int grid, hipStream_t s)
{
    if (grid == 0) return hipSuccess;
    return launch_agg(nullptr, &q, grid, dpad, hl, wide, s);
}

}  // namespace ss
