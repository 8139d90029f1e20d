// Semi-global block matching (Sec. VI-D, the block-based cost mode: two pixels
// are compared through the neighbourhoods around them): the census Hamming
// costs summed over a block centred on the pixel (samples clamped to the image),
// aggregated by the same SGM recurrence with 16-bit path values.
//
// Two passes: block_cost_rows_kernel (square blocks of 3 and 5) or block_cost_kernel
// writes the block-cost volume (16-bit, d fastest, the path buffers' layout);
// aggregate_volume_kernel runs the path recurrence of every line from that volume,
// with the lines, steps and pairs of the census-fed aggregation.
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

// Square blocks of 3 and 5, in images at least that wide: a lane takes DPL consecutive
// disparities of one pixel and walks down the image rows, keeping the sums over the
// block's columns of the last B rows in registers, so a row of a block is counted once
// instead of B times, and the words of the next row are in flight while this one is
// counted.  Words come straight from the census maps (a few MB, in cache): the
// DPL + B - 1 right words under a lane's block row are consecutive.  The tile form
// above reads every sample from LDS and is bound by that; this one is near the rate
// at which its volume can be written: 960x540, D = 128, 3x3 blocks 117 -> 36.6 us
// (133 MB, 3.6 TB/s).  Whole calls, 3x3 / 5x5: 1280x720 D = 128 1.31x / 1.64x,
// 640x480 D = 64 1.28x / 1.60x.
template <int DPL, bool WIDE, int B>
__global__ __launch_bounds__(256) void block_cost_rows_kernel(BlockCostArgs a, int seg)
{
    using CW = CensusWord<WIDE>;
    using Word = typename CW::T;
    constexpr int kDpad = kLanesPerLine * DPL, hw = B / 2, kRight = DPL - 1 + B;
    const int lane = threadIdx.x & 15, d0 = lane * DPL, W = a.W, H = a.H;
    // the last column of blocks first, then the others from the left: walks at the
    // image's sides take longest
    const int bx = blockIdx.y == 0 ? (int)gridDim.y - 1 : (int)blockIdx.y - 1;
    const int xw = bx * 16 + 4 * uniform((int)threadIdx.x >> 6);  // the wave's first pixel
    const int x = xw + (((int)threadIdx.x & 63) >> 4), y0 = (int)blockIdx.x * seg, y1 = min(y0 + seg, H);
    if (xw >= W) return;
    const Word *cl = (const Word *)a.census_l, *cr = (const Word *)a.census_r;
    uint32_t keep[DPL / 2 + DPL % 2], fill[DPL / 2 + DPL % 2];  // the padding disparities' cost
#pragma unroll
    for (int j = 0; j < DPL; j += 2) {
        const bool k0 = d0 + j < a.D, k1 = d0 + j + 1 < a.D;
        keep[j / 2] = (k0 ? 0xFFFFu : 0u) | (k1 ? 0xFFFF0000u : 0u);
        fill[j / 2] = (k0 ? 0u : (uint32_t)kBlockPadCost) | (k1 ? 0u : (uint32_t)kBlockPadCost << 16);
    }
    uint32_t sum[B][DPL];
    auto put = [&](int y) {
        uint32_t acc[DPL + 1];
        acc[DPL] = 0;
#pragma unroll
        for (int j = 0; j < DPL; ++j) {
            acc[j] = sum[0][j];
#pragma unroll
            for (int r = 1; r < B; ++r) acc[j] += sum[r][j];
        }
        uint16_t *o = a.vol + ((size_t)y * W + x) * kDpad + d0;
        if constexpr (DPL == 1) {
            *o = (uint16_t)((acc[0] & keep[0]) | fill[0]);
        } else {
            uint32_t v[DPL / 2];
#pragma unroll
            for (int j = 0; j < DPL; j += 2) v[j / 2] = ((acc[j] | acc[j + 1] << 16) & keep[j / 2]) | fill[j / 2];
            __builtin_memcpy(__builtin_assume_aligned(o, DPL % 8 == 0 ? 16 : DPL % 4 == 0 ? 8 : 4), v, sizeof(v));
        }
    };
    // rows y0 - hw .. y1 + hw - 1 in turn: load(y) gives a row's words, count() its sums
    auto walk = [&](auto load, auto count) {
        auto next = load(y0 - hw);
#pragma unroll
        for (int k = 0; k < B - 1; ++k) {
            const auto w = next;
            next = load(y0 - hw + k + 1);
            count(w, sum[k]);
        }
        for (int y = y0; y < y1; y += B) {
#pragma unroll
            for (int k = 0; k < B; ++k) {
                if (y + k >= y1) return;
                const auto w = next;
                next = load(y + k + hw + 1);
                count(w, sum[(k + B - 1) % B]);
                if (x < W) put(y + k);
            }
        }
    };
    auto row_of = [&](int y) { return (size_t)min(max(y, 0), H - 1) * W; };
    struct Row { Word l[B], r[kRight]; };
    // first of the B image columns that hold the window's samples, and column of r[0]
    const int xc = min(x, W - 1), xs = min(max(xc - hw, 0), W - B), c0 = xs - d0 - (DPL - 1);
    if (xw - hw >= kDpad - 1 && xw + 3 + hw < W) {  // every sample inside the image
        walk(
            [&](int y) {
                Row w;
                __builtin_memcpy(w.l, cl + row_of(y) + xs, sizeof(w.l));
                __builtin_memcpy(w.r, cr + row_of(y) + c0, sizeof(w.r));
                return w;
            },
            [&](const Row &w, uint32_t (&s)[DPL]) {
#pragma unroll
                for (int j = 0; j < DPL; ++j) {
                    s[j] = CW::hamming(w.l[0], w.r[DPL - 1 - j]);
#pragma unroll
                    for (int u = 1; u < B; ++u) s[j] += CW::hamming(w.l[u], w.r[u + DPL - 1 - j]);
                }
            });
    } else {
        // samples beyond a side repeat its column: each column counts as often as the
        // clamped window holds it; a right word left of the image differs in every bit
        uint32_t times[B];
#pragma unroll
        for (int c = 0; c < B; ++c) {
            times[c] = 0;
#pragma unroll
            for (int u = -hw; u <= hw; ++u) times[c] += min(max(xc + u, 0), W - 1) == xs + c ? 1u : 0u;
        }
        const Word all = (Word)~(Word)0 >> (8 * (int)sizeof(Word) - a.bits);
        Word left[kRight];
#pragma unroll
        for (int k = 0; k < kRight; ++k) left[k] = c0 + k < 0 ? all : 0;
        walk(
            [&](int y) {
                Row w;
                const size_t at = row_of(y);
                __builtin_memcpy(w.l, cl + at + xs, sizeof(w.l));
                if (at >= (size_t)kDpad) {  // left of the image lie words of the rows above
                    __builtin_memcpy(w.r, cr + at + c0, sizeof(w.r));
                } else {
#pragma unroll
                    for (int k = 0; k < kRight; ++k) {
                        w.r[k] = cr[max((int)at + c0 + k, 0)];
                        asm volatile("" : "+v"(w.r[k]));  // keeps the two forms of load apart
                    }
                }
                return w;
            },
            [&](const Row &w, uint32_t (&s)[DPL]) {
#pragma unroll
                for (int j = 0; j < DPL; ++j) {
                    s[j] = 0;
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        const int k = u + DPL - 1 - j;
                        s[j] += __umul24(times[u], CW::hamming((w.l[u] ^ w.r[k]) | left[k], 0));
                    }
                }
            });
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

// blocks of row walks a launch aims at
constexpr int kRowWalks = 2048;

template <int DPL>
hipError_t launch_sgbm_dpl(const BlockCostArgs *bc, const VolumeArgs *va, bool wide, hipStream_t s)
{
    if (bc) {
        dim3 grid((bc->W + 15) / 16, bc->H), block(256);
        if (bc->bw == bc->bh && (bc->bw == 3 || bc->bw == 5) && bc->W >= bc->bw) {
            // rows per walk: enough walks to fill the chip, few enough that the B - 1
            // rows a walk begins with stay a small part (960x540: 1024 blocks 64 us,
            // 2048 59 us, 4096 62 us)
            const int seg = std::min(std::max((int)((int64_t)grid.x * bc->H / kRowWalks), 4), 64);
            grid = dim3((bc->H + seg - 1) / seg, grid.x);
            if (bc->bw == 3 && wide) hipLaunchKernelGGL((block_cost_rows_kernel<DPL, true, 3>), grid, block, 0, s, *bc, seg);
            else if (bc->bw == 3) hipLaunchKernelGGL((block_cost_rows_kernel<DPL, false, 3>), grid, block, 0, s, *bc, seg);
            else if (wide) hipLaunchKernelGGL((block_cost_rows_kernel<DPL, true, 5>), grid, block, 0, s, *bc, seg);
            else hipLaunchKernelGGL((block_cost_rows_kernel<DPL, false, 5>), grid, block, 0, s, *bc, seg);
        } else if (wide) hipLaunchKernelGGL((block_cost_kernel<DPL, true>), grid, block, 0, s, *bc);
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
