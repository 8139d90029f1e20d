// Semi-global block matching (Sec. VI-D, the block-based cost mode: two pixels
// are compared through the neighbourhoods around them): the census Hamming
// costs summed over a block centred on the pixel (samples clamped to the image),
// aggregated by the same SGM recurrence with 16-bit path values.
//
// Two kernels: block_cost_kernel writes the block-cost volume (16-bit, d
// fastest, the path buffers' layout); aggregate_volume_kernel runs the path
// recurrence of every line from that volume, with the lines, steps and pairs of
// the census-fed aggregation.
#include "aggregate_impl.h"

namespace ss {

namespace {

// ---------------------------------------------------------------- block costs
// 16 pixels of one row per 256-thread block, one 16-lane row per pixel, DPL
// disparities per lane (lane l: l, l + 16, l + 32, ...).  The window rows come
// into LDS by direct-to-LDS loads,
// as many rows at once as fit a 12 KB tile (all of them for blocks up to
// 14 rows at D <= 128), so a block waits for memory once per tile rather than
// once per row.  A tile row holds the left census words the 16 windows cover
// and the right words they reach at every disparity; every sample is an LDS
// read.
template <int DPL, bool WIDE>
__global__ __launch_bounds__(256) void block_cost_kernel(BlockCostArgs a)
{
    using CW = CensusWord<WIDE>;
    using Word = typename CW::T;
    constexpr int kDpad = kLanesPerLine * DPL;
    constexpr int kWordDw = (int)sizeof(Word) / 4;
    constexpr int kLeftWords = 16 + 2 * kMaxBlockHalf;
    constexpr int kRowWords = kLeftWords + kLeftWords + kDpad - 1;  // left slots, then right slots
    constexpr int kRowDw = kRowWords * kWordDw;
    constexpr int kFit = 12288 / (kRowDw * 4);
    constexpr int kRows = kFit < 1 ? 1 : (kFit > 2 * kMaxBlockHalf + 1 ? 2 * kMaxBlockHalf + 1 : kFit);
    constexpr int kLoads = (kRows * kRowDw + 255) / 256;
    __shared__ __align__(16) uint32_t tile[kLoads * 256];
    const int tid = threadIdx.x, lane = tid & 15, px = tid >> 4;
    const int W = a.W, H = a.H, y = blockIdx.y, x0 = blockIdx.x * 16, x = x0 + px;
    // lane l sums disparities l, l + 16, l + 32, ...: for each of them the
    // 16 lanes of a pixel read 16 consecutive right words (no bank conflicts)
    const int hw = a.bw / 2, hh = a.bh / 2;
    // window columns (clamped to the image) and the right columns they reach;
    // right slot k holds column rlo + k (columns left of the image are never
    // counted: their samples cost the full bit count)
    const int xlo = max(x0 - hw, 0), rlo = xlo - (kDpad - 1);
    const uint32_t *cl = (const uint32_t *)a.census_l, *cr = (const uint32_t *)a.census_r;
    uint32_t acc[DPL];
#pragma unroll
    for (int j = 0; j < DPL; ++j) acc[j] = 0;
    const int xc = min(x, W - 1);
    const uint32_t bits = (uint32_t)a.bits;
    const bool inner = rlo >= 0;  // no sample reaches left of the image
    for (int r0 = -hh; r0 <= hh; r0 += kRows) {
        const int nrows = min(kRows, hh - r0 + 1);
        if (r0 > -hh) __syncthreads();  // the previous tile's reads are done
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int e = tid + 256 * k;  // dword of the tile
            if (e < nrows * kRowDw) {
                const int rr = e / kRowDw, rem = e - rr * kRowDw, idx = rem / kWordDw, h = rem - idx * kWordDw;
                const int row = min(max(y + r0 + rr, 0), H - 1);
                const bool left = idx < kLeftWords;
                const int col = min(max(left ? xlo + idx : rlo + (idx - kLeftWords), 0), W - 1);
                const uint32_t *src = (left ? cl : cr) + ((size_t)row * W + col) * kWordDw + h;
                __builtin_amdgcn_global_load_lds(src, &tile[256 * k + (tid & ~63)], 4, 0, 0);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        for (int rr = 0; rr < nrows; ++rr) {
            const Word *sl = (const Word *)tile + rr * kRowWords, *sr = sl + kLeftWords;
            for (int u = -hw; u <= hw; ++u) {
                const int cx = min(max(xc + u, 0), W - 1);
                const Word wl = sl[cx - xlo];
                const Word *rp = &sr[cx - lane - rlo];
                if (inner) {
#pragma unroll
                    for (int j = 0; j < DPL; ++j) acc[j] += CW::hamming(wl, rp[-16 * j]);
                } else {
#pragma unroll
                    for (int j = 0; j < DPL; ++j)
                        acc[j] += cx - lane - 16 * j >= 0 ? CW::hamming(wl, rp[-16 * j]) : bits;
                }
            }
        }
    }
    if (x < W) {
        uint16_t *o = a.vol + ((size_t)y * W + x) * kDpad + lane;
#pragma unroll
        for (int j = 0; j < DPL; ++j) o[16 * j] = (uint16_t)(lane + 16 * j < a.D ? acc[j] : (uint32_t)kBlockPadCost);
    }
}

// ---------------------------------------------------------------- aggregation
// The units' lines from the block-cost volume (16-bit path values): the horizontal
// ones singly, with volume_horizontal_lanes() lanes each (the longest chains: fewer
// disparities per lane shorten every step), the others in pairs.
template <int DPL>
__global__ __launch_bounds__(64 * kWavesPerItem) __attribute__((amdgpu_waves_per_eu(2, 2))) void aggregate_volume_kernel(VolumeArgs v)
{
    constexpr int kDpad = kLanesPerLine * DPL, HL = volume_horizontal_lanes(kDpad);
    constexpr int HD = lane_disparities(kDpad, HL), LD = lane_disparities(kDpad, kLanesPerLine);
    const AggregateArgs &a = v.a;
    int item = (int)blockIdx.x, unit = 0;
#pragma unroll
    for (int k = 1; k < 8; ++k) unit += (k < a.nunits && item >= a.item_begin[k]) ? 1 : 0;
    item -= a.item_begin[unit];
    const int w = uniform((int)threadIdx.x >> 6);
    const uint32_t p1 = both(a.p1), p2 = both(a.p2);
    const int dx = a.dx[unit], dy = a.dy[unit], nlines = line_count(dx, dy, a.W, a.H);
    if (dy == 0) {
        const int wave = item * kWavesPerItem + w;
        if (wave * (64 / HL) >= nlines) return;
        const WaveLines g = wave_lines<HL, 2 * kDpad>(dx, dy, wave, a.W, a.H, (int)threadIdx.x % HL * (2 * HD));
        run_single<kDpad, HD, HL, true>(VolumeSource<kDpad, HD, true>{a.cost}, a.out[unit], g, p1, p2, agg_step_cost(HD, HL),
                                        a.max_item_work);
    } else {
        const int wave = item * (kWavesPerItem / 2) + w / 2;
        const WaveLines g = wave_lines<kLanesPerLine, 2 * kDpad>(dx, dy, wave, a.W, a.H,
                                                                 (int)threadIdx.x % kLanesPerLine * (2 * LD));
        run_pair<kDpad, LD, kLanesPerLine, true, sum_steps(LD, true)>(
            VolumeSource<kDpad, LD, true>{a.cost}, a.out[unit], g, wave * (64 / kLanesPerLine) < nlines, (w & 1) != 0, p1, p2,
            agg_step_cost(LD, kLanesPerLine), a.max_item_work);
    }
}

template <int DPL>
hipError_t launch_sgbm_dpl(const BlockCostArgs *bc, const VolumeArgs *va, bool wide, hipStream_t s)
{
    if (bc) {
        dim3 grid((bc->W + 15) / 16, bc->H), block(256);
        if (wide) hipLaunchKernelGGL((block_cost_kernel<DPL, true>), grid, block, 0, s, *bc);
        else hipLaunchKernelGGL((block_cost_kernel<DPL, false>), grid, block, 0, s, *bc);
    } else {
        hipLaunchKernelGGL((aggregate_volume_kernel<DPL>), dim3(va->a.item_begin[va->a.nunits]), dim3(64 * kWavesPerItem), 0, s, *va);
    }
    return hipGetLastError();
}

hipError_t launch_sgbm(const BlockCostArgs *bc, const VolumeArgs *va, int dpad, bool wide, hipStream_t s)
{
    switch (dpad / kLanesPerLine) {
    case 1: return launch_sgbm_dpl<1>(bc, va, wide, s);
    case 2: return launch_sgbm_dpl<2>(bc, va, wide, s);
    case 4: return launch_sgbm_dpl<4>(bc, va, wide, s);
    case 6: return launch_sgbm_dpl<6>(bc, va, wide, s);
    case 8: return launch_sgbm_dpl<8>(bc, va, wide, s);
    case 12: return launch_sgbm_dpl<12>(bc, va, wide, s);
    case 16: return launch_sgbm_dpl<16>(bc, va, wide, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_block_cost(const BlockCostArgs &a, int dpad, bool wide, hipStream_t s)
{
    if (a.W < 1 || a.H < 1) return hipSuccess;
    return launch_sgbm(&a, nullptr, dpad, wide, s);
}

hipError_t launch_aggregate_volume(const VolumeArgs &a, hipStream_t s)
{
    return launch_sgbm(nullptr, &a, a.a.Dpad, false, s);
}

}  // namespace ss
