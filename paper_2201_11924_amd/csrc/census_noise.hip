// IR noise model (Sec. VI-C, Eq. (7)) and census transform (Sec. VI-D).
#include "internal.h"

namespace ss {

// ---------------------------------------------------------------- IR noise
// out = clip(rint(gamma * in + n), 0, 255); product and sum are separately
// rounded fp32 operations, the integer decision is a round-half-even.
__global__ __launch_bounds__(256) void ir_noise_kernel(const uint8_t *__restrict__ in,
                                                       const float *__restrict__ gamma,
                                                       const float *__restrict__ n,
                                                       uint8_t *__restrict__ out, int64_t count)
{
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
        float v = __fadd_rn(__fmul_rn(gamma[i], (float)in[i]), n[i]);
        float r = rintf(v);
        r = r > 0.0f ? r : 0.0f;  // also maps NaN to 0
        r = r < 255.0f ? r : 255.0f;
        out[i] = (uint8_t)r;
    }
}

hipError_t launch_ir_noise(const uint8_t *in, const float *gamma, const float *n, uint8_t *out,
                           int64_t count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(ir_noise_kernel, dim3((unsigned)blocks), dim3(256), 0, s, in, gamma, n, out, count);
    return hipGetLastError();
}

// ---------------------------------------------------------------- census
// A 64x16 output tile per 256-thread block, four adjacent pixels of a row per thread;
// the tile plus its window halo is staged in LDS with clamp-to-edge addressing.  Bit k
// of a word is the k-th comparison of the window in row-major order:
//   full:               [I(p) > I(p+o)]       for every o != 0
//   center-symmetric:   [I(p+o) > I(p-o)]     for every o before the centre
constexpr int kCensusTx = 64, kCensusTy = 16, kCensusBlock = 256;

// any window: one byte from LDS per sample
template <typename Word>
__device__ __forceinline__ void census_tile(const uint8_t *__restrict__ img, int pitch, int W, int H, int cw, int ch,
                                            int mode, Word *__restrict__ out, int bx, int by, uint8_t *tile)
{
    const int rw = cw / 2, rh = ch / 2;
    const int tw = kCensusTx + cw - 1, th = kCensusTy + ch - 1;
    const int x0 = bx * kCensusTx - rw, y0 = by * kCensusTy - rh;
    for (int i = threadIdx.x; i < tw * th; i += kCensusBlock) {
        int ty = i / tw, tx = i - ty * tw;
        int gx = min(max(x0 + tx, 0), W - 1), gy = min(max(y0 + ty, 0), H - 1);
        tile[i] = img[(size_t)gy * pitch + gx];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kCensusTx * kCensusTy; i += kCensusBlock) {
        const int lx = i % kCensusTx, ly = i / kCensusTx;
        const int x = bx * kCensusTx + lx, y = by * kCensusTy + ly;
        if (x >= W || y >= H) continue;
        // window centre inside the tile
        const int cx = lx + rw, cy = ly + rh;
        Word word = 0;
        int k = 0;
        if (mode == 0) {
            // offsets before the centre: every row above it, then the left half of its row
            for (int oy = -rh; oy <= 0; ++oy) {
                const int oxe = oy < 0 ? rw : -1;
                const uint8_t *pa = &tile[(cy + oy) * tw + cx];
                const uint8_t *pb = &tile[(cy - oy) * tw + cx];
                for (int ox = -rw; ox <= oxe; ++ox) {
                    word |= (Word)(pa[ox] > pb[-ox]) << k;
                    ++k;
                }
            }
        } else {
            const int c = tile[cy * tw + cx];
            for (int oy = -rh; oy <= rh; ++oy)
                for (int ox = -rw; ox <= rw; ++ox) {
                    if (ox == 0 && oy == 0) continue;
                    word |= (Word)(c > tile[(cy + oy) * tw + cx + ox]) << k;
                    ++k;
                }
        }
        out[(size_t)y * W + x] = word;
    }
}

// A window size and mode fixed at compile time.  The pass is bound by its LDS reads
// when every sample is one (62 byte reads per pixel of a 7x9 window: 1280x720 pair
// 13.0 us), so a thread reads the three words of each window row that its four pixels
// share (27 reads for four pixels) and compares bytes out of registers: the
// difference of two selected bytes is one instruction, and its sign bit is shifted
// into the word by a second (v_alignbit), from the last comparison down.  A call at
// 1280x720 got 6.5 us shorter, 16 pairs of that size 168 -> 78 us, 641x479 with the
// full census 19 -> 6.4 us.  What is left is the arithmetic: two instructions of
// about 4.4 cycles each per comparison (51 us of the 78).
constexpr int kCensusHalo = 4;                                    // columns staged left and right of the tile
constexpr int kCensusRow = (kCensusTx + 2 * kCensusHalo) / 4;     // words per staged row

// offset of the k-th comparison's (first) sample
template <int CW, int CH, int MODE>
__device__ __forceinline__ void census_offset(int k, int &oy, int &ox)
{
    const int i = MODE == 1 && k >= CW * CH / 2 ? k + 1 : k;  // the full census skips the centre
    oy = -(CH / 2) + i / CW;
    ox = -(CW / 2) + i % CW;
}

template <typename Word, int CW, int CH, int MODE>
__device__ __forceinline__ void census_tile_fixed(const uint8_t *__restrict__ img, int pitch, int W, int H,
                                                  Word *__restrict__ out, int bx, int by, uint32_t *tile)
{
    constexpr int rh = CH / 2, th = kCensusTy + CH - 1, kRow = kCensusRow;
    constexpr int kBits = MODE == 0 ? (CW * CH - 1) / 2 : CW * CH - 1;
    static_assert(CW / 2 <= kCensusHalo && kBits <= 8 * (int)sizeof(Word), "window too wide");
    const int x0 = bx * kCensusTx, y0 = by * kCensusTy;
    for (int i = threadIdx.x; i < kRow * th; i += kCensusBlock) {
        const int ty = i / kRow, gx = x0 - kCensusHalo + 4 * (i - ty * kRow);
        const uint8_t *row = img + (size_t)min(max(y0 - rh + ty, 0), H - 1) * pitch;
        uint32_t v;
        if (gx >= 0 && gx + 3 < W) {
            __builtin_memcpy(&v, row + gx, 4);
        } else {
            v = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) v |= (uint32_t)row[min(max(gx + b, 0), W - 1)] << (8 * b);
        }
        tile[i] = v;
    }
    __syncthreads();
    const int q = threadIdx.x % (kCensusTx / 4), ly = threadIdx.x / (kCensusTx / 4);
    const int x = x0 + 4 * q, y = y0 + ly;
    if (x >= W || y >= H) return;
    uint32_t w[CH][3];  // columns x - 4 .. x + 7 of the window's rows
#pragma unroll
    for (int r = 0; r < CH; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) w[r][c] = tile[(ly + r) * kRow + q + c];
    auto sample = [&](int p, int oy, int ox) -> uint32_t {
        const int col = kCensusHalo + p + ox;
        return (w[rh + oy][col / 4] >> (8 * (col % 4))) & 0xFFu;
    };
    Word words[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        uint32_t lo = 0, hi = 0;
#pragma unroll
        for (int k = kBits - 1; k >= 0; --k) {
            int oy, ox;
            census_offset<CW, CH, MODE>(k, oy, ox);
            // the sign of the difference is [a > b]
            const uint32_t d = MODE == 0 ? sample(p, -oy, -ox) - sample(p, oy, ox) : sample(p, oy, ox) - sample(p, 0, 0);
            if (k >= 32) hi = __builtin_amdgcn_alignbit(hi, d, 31);
            else lo = __builtin_amdgcn_alignbit(lo, d, 31);
        }
        words[p] = (Word)lo;
        if constexpr (sizeof(Word) == 8) words[p] |= (Word)hi << 32;
    }
    Word *o = out + (size_t)y * W + x;
    if (x + 3 < W) {
        __builtin_memcpy(o, words, sizeof(words));
    } else {
#pragma unroll
        for (int p = 0; p < 3; ++p)
            if (x + p < W) o[p] = words[p];
    }
}

// the windows with a compiled form; others take the general loop
template <typename Word>
__device__ __forceinline__ void census_any(const uint8_t *img, int pitch, int W, int H, int cw, int ch, int mode,
                                           Word *out, int bx, int by, uint32_t *tile)
{
    if (mode == 0) {
        if (cw == 7 && ch == 9) return census_tile_fixed<Word, 7, 9, 0>(img, pitch, W, H, out, bx, by, tile);
        if (cw == 9 && ch == 7) return census_tile_fixed<Word, 9, 7, 0>(img, pitch, W, H, out, bx, by, tile);
        if (cw == 5 && ch == 5) return census_tile_fixed<Word, 5, 5, 0>(img, pitch, W, H, out, bx, by, tile);
        if (cw == 7 && ch == 7) return census_tile_fixed<Word, 7, 7, 0>(img, pitch, W, H, out, bx, by, tile);
        if constexpr (sizeof(Word) == 8)
            if (cw == 9 && ch == 9) return census_tile_fixed<Word, 9, 9, 0>(img, pitch, W, H, out, bx, by, tile);
    } else {
        if (cw == 5 && ch == 5) return census_tile_fixed<Word, 5, 5, 1>(img, pitch, W, H, out, bx, by, tile);
        if constexpr (sizeof(Word) == 8)
            if (cw == 7 && ch == 9) return census_tile_fixed<Word, 7, 9, 1>(img, pitch, W, H, out, bx, by, tile);
    }
    census_tile<Word>(img, pitch, W, H, cw, ch, mode, out, bx, by, (uint8_t *)tile);
}

// one launch for one or two images of the same size (blockIdx.z picks the image)
template <typename Word>
__global__ __launch_bounds__(kCensusBlock) void census_kernel(const uint8_t *__restrict__ img0,
                                                              const uint8_t *__restrict__ img1, int pitch, int W, int H,
                                                              int cw, int ch, int mode, Word *__restrict__ out0,
                                                              Word *__restrict__ out1, unsigned *zero, int nzero)
{
    extern __shared__ uint32_t tile[];
    if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && (int)threadIdx.x < nzero) zero[threadIdx.x] = 0u;
    const bool second = blockIdx.z != 0;
    census_any<Word>(second ? img1 : img0, pitch, W, H, cw, ch, mode, second ? out1 : out0, blockIdx.x, blockIdx.y, tile);
}

// batch form: one block per (job, tile) item; tile = by * ceil(W / kCensusTx) + bx
template <typename Word>
__global__ __launch_bounds__(kCensusBlock) void census_batch_kernel(CensusBatch b)
{
    extern __shared__ uint32_t tile[];
    const uint32_t it = b.items[blockIdx.x];
    const CensusJob &j = b.jobs[it >> 20];
    const int t = (int)(it & 0xFFFFFu), tx = (j.W + kCensusTx - 1) / kCensusTx;
    census_any<Word>(j.img, j.pitch, j.W, j.H, j.cw, j.ch, j.mode, (Word *)j.out, t % tx, t / tx, tile);
}

// LDS of a launch: the general form's bytes or the fixed one's words, whichever is more
static size_t census_lds(int cw, int ch)
{
    const int row = kCensusTx + cw - 1 > 4 * kCensusRow ? kCensusTx + cw - 1 : 4 * kCensusRow;
    return ((size_t)row * (kCensusTy + ch - 1) + 3) / 4 * 4;
}

hipError_t launch_census_batch(const CensusBatch &b, bool out64, hipStream_t s)
{
    if (b.nitems == 0) return hipSuccess;
    const size_t lds = census_lds(b.max_cw, b.max_ch);
    if (out64) hipLaunchKernelGGL(census_batch_kernel<uint64_t>, dim3(b.nitems), dim3(kCensusBlock), lds, s, b);
    else hipLaunchKernelGGL(census_batch_kernel<uint32_t>, dim3(b.nitems), dim3(kCensusBlock), lds, s, b);
    return hipGetLastError();
}

int census_tiles(int W, int H) { return ((W + kCensusTx - 1) / kCensusTx) * ((H + kCensusTy - 1) / kCensusTy); }

hipError_t launch_census_pair(const uint8_t *img0, const uint8_t *img1, int pitch, int W, int H, int cw, int ch,
                              int mode, void *out0, void *out1, bool out64, hipStream_t s, unsigned *zero, int nzero)
{
    if (nzero < 0 || nzero > kCensusBlock || (nzero > 0 && !zero)) return hipErrorInvalidValue;
    dim3 grid((W + kCensusTx - 1) / kCensusTx, (H + kCensusTy - 1) / kCensusTy, img1 ? 2 : 1);
    dim3 block(kCensusBlock);
    const size_t lds = census_lds(cw, ch);
    if (out64)
        hipLaunchKernelGGL(census_kernel<uint64_t>, grid, block, lds, s, img0, img1, pitch, W, H, cw, ch, mode,
                           (uint64_t *)out0, (uint64_t *)out1, zero, nzero);
    else
        hipLaunchKernelGGL(census_kernel<uint32_t>, grid, block, lds, s, img0, img1, pitch, W, H, cw, ch, mode,
                           (uint32_t *)out0, (uint32_t *)out1, zero, nzero);
    return hipGetLastError();
}

hipError_t launch_census(const uint8_t *img, int pitch, int W, int H, int cw, int ch, int mode, void *out,
                         bool out64, hipStream_t s, unsigned *zero, int nzero)
{
    return launch_census_pair(img, nullptr, pitch, W, H, cw, ch, mode, out, nullptr, out64, s, zero, nzero);
}

}  // namespace ss
