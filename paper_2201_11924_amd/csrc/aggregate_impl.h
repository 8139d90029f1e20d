// Semi-global path aggregation kernels (included by the per-disparity-count
// translation units agg_dpl*.hip, which instantiate them in parallel builds,
// and by sgbm.hip for the 16-bit block costs).
//
// Semi-global path aggregation (Sec. VI-D; the SGM recurrence of Hirschmueller,
// which the paper cites):
//   L_r(p,d) = C(p,d) + min(L_r(p-r,d), L_r(p-r,d+-1) + P1, m + P2) - m,
//   m = min_k L_r(p-r,k),  C(p,d) = popcount(cL(p) ^ cR(p - d)).
//
// Every scanline of every direction is an independent chain of steps.  A line's
// D-vector is held by LPL lanes of one wave (16: one DPP row, so a wave runs four
// lines), DPL consecutive disparities per lane, two disparities per register: the
// values are integers far below 2^16, so packed 16-bit adds and minima give exactly
// the 32-bit results at half the instructions.  Register j of a lane holds
// disparities d0 + j and d0 + j + DPL/2, so the d-1 / d+1 neighbours of a register
// are the neighbouring registers, and only the two edge registers take a DPP move.
//
// The lanes keep un-normalised sums
//   U(p,d) = C(p,d) + min(U(p-r,d), U(p-r,d+-1) + P1, u + P2),  u = min_k U(p-r,k),
// for which induction gives L_r(p,d) = U(p,d) - u exactly, so a step that stores
// nothing needs no normalisation; U is brought back to U - u every 8 or 16 steps
// (16-bit block costs, whose sums grow faster, every step).  All values
// stay below 0x7C00, where 16-bit patterns order the same as half floats and as
// integers, so three-way minima use v_pk_minimum3_f16 (no value is ever a NaN
// or changed by it).
//
// No LDS; a wave owns its lines alone, or shares them with one other (below).
//
// Two kinds of unit:
//  * single: one direction, its path values stored as bytes.
//  * pair: a direction and its opposite, whose lines are the same pixels; the SUM of
//    both path values is stored, so that one byte per pixel and disparity is written,
//    and read by the selection, instead of two (both passes are bound by that
//    traffic: stores alone reach 4.1 TB/s on this GPU).  The price is a third walk of
//    arithmetic (run_pair).  Needs sums of two path values to fit a byte:
//    bits + P2 <= 127.
// Vertical and diagonal units read the matching costs from a volume of bytes that
// cost_kernel wrote (1 byte per pixel and disparity, in the path buffers' layout):
// recomputing them from the census words costs 4.7 SIMD cycles more per disparity
// and step than unpacking a byte.  Costs where x - d < 0 are `bits`, and 255 where
// d >= D, so the steps need no border case.  Where no buffer is left for the volume they
// count 32-bit words after all (run_columns), and so they do where the volume is too large
// for the caches and little is won by it (default_costs).  Horizontal units count the bits of
// 32-bit census words themselves (a lane's right words slide by one column per step:
// the pixels of a segment share all but a few), which saves the reads.
#pragma once
#include <algorithm>
#include <type_traits>
#include <utility>

#include "internal.h"

namespace ss {

namespace {

// ---------------------------------------------------------------- small pieces
typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x3_t __attribute__((ext_vector_type(3)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// the neighbour value of a disparity outside the line: above every real value
// plus P1, and the largest pattern that is a finite half float
constexpr uint32_t kNone = 0x7BFF7BFFu;

// DPP controls (GFX9 encoding)
constexpr int kRowShl1 = 0x101, kRowShr1 = 0x111;
constexpr int kRowRor1 = 0x121, kRowRor2 = 0x122, kRowRor4 = 0x124, kRowRor8 = 0x128;
constexpr int kQuadOdd = 0xF5;  // lanes 1, 1, 3, 3 of each four
constexpr int kWaveShl1 = 0x130, kWaveShr1 = 0x138;

__device__ __forceinline__ u16x2_t h2(uint32_t v) { return __builtin_bit_cast(u16x2_t, v); }
__device__ __forceinline__ uint32_t w1(u16x2_t v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ uint32_t pk_add(uint32_t a, uint32_t b) { return w1(h2(a) + h2(b)); }
__device__ __forceinline__ uint32_t pk_sub(uint32_t a, uint32_t b) { return w1(h2(a) - h2(b)); }
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) { return w1(__builtin_elementwise_min(h2(a), h2(b))); }
__device__ __forceinline__ uint32_t pk_min3(uint32_t a, uint32_t b, uint32_t c)
{
    const f16x2_t m = __builtin_elementwise_minimum(__builtin_bit_cast(f16x2_t, a), __builtin_bit_cast(f16x2_t, b));
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_minimum(m, __builtin_bit_cast(f16x2_t, c)));
}
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b) { return w1(__builtin_elementwise_max(h2(a), h2(b))); }
__device__ __forceinline__ uint32_t pk_max3(uint32_t a, uint32_t b, uint32_t c)
{
    const f16x2_t m = __builtin_elementwise_maximum(__builtin_bit_cast(f16x2_t, a), __builtin_bit_cast(f16x2_t, b));
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_maximum(m, __builtin_bit_cast(f16x2_t, c)));
}
// a 16-bit value in both halves
__device__ __forceinline__ uint32_t both(uint32_t v) { return w1(u16x2_t{(uint16_t)v, (uint16_t)v}); }

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t old, uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, 0xF, 0xF, false);
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_rot(uint32_t v)
{
    // (the caller replaces what lanes without a source receive, if there are any)
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

template <typename T>
__device__ __forceinline__ T *uniform(T *p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (T *)(((uint64_t)hi << 32) | lo);
}

// f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>)
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// buffer resource word 3 for raw byte buffers (GFX9 family); offsets at or past
// the size are dropped (stores) or read as zero (loads): a lane off its line passes
// kOff instead of branching
constexpr int kBufferWord3 = 0x00020000;
constexpr uint32_t kOff = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t open_buffer(const void *base)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, 0x7FFFFFFF, kBufferWord3);
}

// Cache policy of the path-value stores: non-temporal (NT).  Only the selection
// reads them back; stored with the default policy they leave the last-level caches
// full of dirty lines whose write-back then competes with the selection's reads
// (measured on the 8-buffer form: selection 241 -> 185 us).
constexpr int kStoreAux = 2;

// ---------------------------------------------------------------- lanes of a line
// LPL lanes of which the first ACTIVE hold the line's disparities (the others
// idle: nothing they hold reaches an active lane)
template <int LPL, int ACTIVE>
struct LineOps {
    // value of the previous / next lane (the line's end lanes get kNone)
    static __device__ __forceinline__ uint32_t from_prev(uint32_t v, int lane)
    {
        if constexpr (LPL == 16) return dpp_mov<kRowShr1>(kNone, v);
        else if constexpr (LPL == 64) return dpp_mov<kWaveShr1>(kNone, v);
        else {
            const uint32_t r = dpp_rot<kWaveShr1>(v);  // (every lane takes part in the move)
            return lane == 0 ? kNone : r;
        }
    }
    static __device__ __forceinline__ uint32_t from_next(uint32_t v, int lane)
    {
        if constexpr (LPL == 16 && ACTIVE == LPL) return dpp_mov<kRowShl1>(kNone, v);
        else if constexpr (LPL == 64 && ACTIVE == LPL) return dpp_mov<kWaveShl1>(kNone, v);
        else {
            const uint32_t r = dpp_rot<LPL == 16 ? kRowShl1 : kWaveShl1>(v);
            return lane == ACTIVE - 1 ? kNone : r;
        }
    }
    // minimum over the line's lanes, in every lane of the line: a DPP row's minimum
    // by rotations, then rows exchanged in pairs (permlane16 swap) and, for a
    // whole-wave line, halves (permlane32 swap)
    static __device__ __forceinline__ uint32_t line_min(uint32_t v, int lane)
    {
        if constexpr (ACTIVE < LPL) v = lane < ACTIVE ? v : 0xFFFFu;
        v = min(v, dpp_rot<kRowRor8>(v));
        v = min(v, dpp_rot<kRowRor4>(v));
        v = min(v, dpp_rot<kRowRor2>(v));
        v = min(v, dpp_rot<kRowRor1>(v));
        if constexpr (LPL >= 32) {
            const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
            v = min((uint32_t)s[0], (uint32_t)s[1]);
        }
        if constexpr (LPL == 64) {
            const auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
            v = min((uint32_t)s[0], (uint32_t)s[1]);
        }
        return v;
    }
};

// ---------------------------------------------------------------- a lane's values
// DPL values of a lane in memory (bytes, or 16-bit words for V16) and in N packed
// registers.  Bytes: register j = disparities (j, j + N); 16-bit: (2j, 2j + 1), the
// order in memory.  DPL = 1 uses the low half only.
template <int DPL, bool V16>
struct Lane {
    static_assert(DPL <= 2 || DPL % 4 == 0 || (DPL == 6 && !V16), "two disparities per register, whole words in memory (6: 16-bit pieces)");
    static constexpr int N = DPL == 1 ? 1 : DPL / 2;
    static constexpr int kBytes = DPL * (V16 ? 2 : 1);
    static constexpr int NW = (kBytes + 3) / 4;  // words in memory

    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, uint32_t off, int soff, uint32_t (&w)[NW])
    {
        if constexpr (kBytes == 1) {
            w[0] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(rs, off, soff, 0);
        } else if constexpr (kBytes == 2) {
            w[0] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off, soff, 0);
        } else {
            static_assert(kBytes % 4 == 0, "");
            static_for<(NW + 3) / 4>([&](auto ic) {
                constexpr int i = 4 * decltype(ic)::value, n = NW - i < 4 ? NW - i : 4;
                if constexpr (n == 1) {
                    w[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, off + 4 * i, soff, 0);
                } else if constexpr (n == 2) {
                    const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(rs, off + 4 * i, soff, 0);
                    w[i] = v[0]; w[i + 1] = v[1];
                } else if constexpr (n == 3) {
                    const u32x3_t v = __builtin_amdgcn_raw_buffer_load_b96(rs, off + 4 * i, soff, 0);
                    w[i] = v[0]; w[i + 1] = v[1]; w[i + 2] = v[2];
                } else {
                    const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(rs, off + 4 * i, soff, 0);
                    w[i] = v[0]; w[i + 1] = v[1]; w[i + 2] = v[2]; w[i + 3] = v[3];
                }
            });
        }
    }

    template <int AUX>
    static __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t rs, uint32_t off, int soff, const uint32_t (&w)[NW])
    {
        if constexpr (kBytes == 1) {
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)w[0], rs, off, soff, AUX);
        } else if constexpr (kBytes == 2) {
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)w[0], rs, off, soff, AUX);
        } else if constexpr (kBytes == 6) {
            // an even lane stores its next lane's six bytes too (three words, aligned)
            const uint32_t a = dpp_rot<kQuadOdd>(w[0]), b = dpp_rot<kQuadOdd>(w[1]);
            __builtin_amdgcn_raw_buffer_store_b96(u32x3_t{w[0], w[1] | a << 16, __builtin_amdgcn_alignbit(b, a, 16)}, rs,
                                                  (threadIdx.x & 1 ? kOff : off) + soff, 0, AUX);
        } else {
            static_for<(NW + 3) / 4>([&](auto ic) {
                constexpr int i = 4 * decltype(ic)::value, n = NW - i < 4 ? NW - i : 4;
                // (stores of more than 8 bytes take the whole offset in the address
                // register: the next instructions may overwrite their data registers
                // while a busy memory pipe still reads them, and the compiler keeps the
                // wait states for that only where the scalar offset is a constant;
                // measured wrong values at 1920x1080, D = 256 with a register there)
                if constexpr (n == 1) __builtin_amdgcn_raw_buffer_store_b32(w[i], rs, off + 4 * i, soff, AUX);
                else if constexpr (n == 2)
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{w[i], w[i + 1]}, rs, off + 4 * i, soff, AUX);
                else if constexpr (n == 3)
                    __builtin_amdgcn_raw_buffer_store_b96(u32x3_t{w[i], w[i + 1], w[i + 2]}, rs, off + soff + 4 * i, 0, AUX);
                else
                    __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{w[i], w[i + 1], w[i + 2], w[i + 3]}, rs,
                                                           off + soff + 4 * i, 0, AUX);
            });
        }
    }

    // register j from the loaded words
    template <int J>
    static __device__ __forceinline__ uint32_t get(const uint32_t (&w)[NW])
    {
        if constexpr (V16 || DPL == 1) {
            return w[J];
        } else {
            constexpr int a = J, b = J + N;
            constexpr uint32_t sel = (uint32_t)(a % 4) | 0x0C00u | ((uint32_t)(4 + b % 4) << 16) | 0x0C000000u;
            return __builtin_amdgcn_perm(w[b / 4], w[a / 4], sel);
        }
    }

    // the words of N registers whose halves are below 256 (bytes beyond stay inside
    // their own halves: every byte is selected, never shifted in)
    static __device__ __forceinline__ void pack(const uint32_t (&r)[N], uint32_t (&w)[NW])
    {
        if constexpr (V16 || DPL == 1) {
            static_for<N>([&](auto j) { w[j] = r[j]; });
        } else if constexpr (DPL == 2) {
            w[0] = __builtin_amdgcn_perm(r[0], r[0], 0x0C0C0200u);
        } else if constexpr (DPL == 6) {
            const uint32_t p = __builtin_amdgcn_perm(r[1], r[0], 0x06020400u);
            w[0] = __builtin_amdgcn_perm(r[2], p, 0x02040100u);
            w[1] = __builtin_amdgcn_perm(r[2], p, 0x0C0C0603u);
        } else {
            static_assert(N % 2 == 0, "");
            uint32_t p[N / 2];  // lo bytes of registers 2i, 2i + 1, then their hi bytes
            static_for<N / 2>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                p[i] = __builtin_amdgcn_perm(r[2 * i + 1], r[2 * i], 0x06020400u);
            });
            if constexpr (NW == 1) {
                w[0] = p[0];
            } else {
                static_for<NW>([&](auto kc) {  // 16-bit pieces 2k, 2k + 1: the low halves of p, then the high halves
                    constexpr int a = 2 * decltype(kc)::value, b = a + 1, M = N / 2;
                    constexpr uint32_t sa = a < M ? 0x0100u : 0x0302u, sb = b < M ? 0x05040000u : 0x07060000u;
                    w[kc] = __builtin_amdgcn_perm(p[b % M], p[a % M], sa | sb);
                });
            }
        }
    }
};

// One line's state and one step of the recurrence.
template <int DPL, int LPL, int ACTIVE, bool V16>
struct Line {
    using LV = Lane<DPL, V16>;
    using LO = LineOps<LPL, ACTIVE>;
    static constexpr int N = LV::N;
    uint32_t U[N];  // un-normalised sums (V16: normalised path values)
    uint32_t u;     // the line's minimum of U, in the low half

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int j = 0; j < N; ++j) U[j] = 0;
        u = 0;
    }

    // U becomes C + min(...): add(j, t) returns t plus the costs of register j
    template <typename ADD>
    __device__ __forceinline__ void step(uint32_t p1, uint32_t p2, int lane, ADD add)
    {
        uint32_t P[N], low[N], up[N];
#pragma unroll
        for (int j = 0; j < N; ++j) P[j] = pk_add(U[j], p1);
        const uint32_t prev = LO::from_prev(P[N - 1], lane), next = LO::from_next(P[0], lane);
        if constexpr (DPL == 1) {
            low[0] = prev;
            up[0] = next;
        } else if constexpr (V16) {  // register j = (2j, 2j + 1)
#pragma unroll
            for (int j = 0; j < N; ++j) low[j] = __builtin_amdgcn_alignbit(P[j], j > 0 ? P[j - 1] : prev, 16);
#pragma unroll
            for (int j = 0; j < N; ++j) up[j] = j < N - 1 ? low[j + 1] : __builtin_amdgcn_alignbit(next, P[j], 16);
        } else {  // register j = (j, j + N)
            low[0] = __builtin_amdgcn_alignbit(P[N - 1], prev, 16);
#pragma unroll
            for (int j = 1; j < N; ++j) low[j] = P[j - 1];
#pragma unroll
            for (int j = 0; j < N - 1; ++j) up[j] = P[j + 1];
            up[N - 1] = __builtin_amdgcn_alignbit(next, P[0], 16);
        }
        const uint32_t cap = pk_add(both(u), p2);
        const uint32_t ub = both(u);
#pragma unroll
        for (int j = 0; j < N; ++j) {
            uint32_t t = pk_min(pk_min3(U[j], low[j], up[j]), cap);
            if constexpr (V16) t = pk_sub(t, ub);
            low[j] = t;
        }
        static_for<N>([&](auto j) { U[j] = add(j, low[j]); });
        uint32_t m = U[0];
        if constexpr (N % 2 == 0) m = pk_min(m, U[1]);
#pragma unroll
        for (int j = N % 2 == 0 ? 2 : 1; j < N; j += 2) m = pk_min3(m, U[j], U[j + 1]);
        m = DPL == 1 ? m & 0xFFFFu : min(m & 0xFFFFu, m >> 16);
        u = LO::line_min(m, lane);
    }

    // brings U back to U - u
    __device__ __forceinline__ void rebase()
    {
        if constexpr (!V16) {
            const uint32_t ub = both(u);
#pragma unroll
            for (int j = 0; j < N; ++j) U[j] = pk_sub(U[j], ub);
            u = 0;
        }
    }
    // what a step that starts from minimum u adds to a path value
    static __device__ __forceinline__ uint32_t base(uint32_t u) { return V16 ? 0u : u; }
};

// ---------------------------------------------------------------- geometry
// Lines of a direction: first pixel and length of line l.
__device__ __forceinline__ void line_start(int dx, int dy, int l, int W, int H, int &x, int &y, int &len)
{
    if (dy == 0) {
        x = dx > 0 ? 0 : W - 1;
        y = l;
        len = W;
    } else if (dx == 0) {
        x = l;
        y = dy > 0 ? 0 : H - 1;
        len = H;
    } else if (l < W) {  // enters through the top / bottom row
        x = l;
        y = dy > 0 ? 0 : H - 1;
        len = min(dx > 0 ? W - l : l + 1, H);
    } else {  // enters through the side column
        const int j = l - W;
        x = dx > 0 ? 0 : W - 1;
        y = dy > 0 ? j + 1 : H - 2 - j;
        len = min(W, H - 1 - j);
    }
}

// A wave's lines: the first pixel (elements of the image) all offsets count from,
// each lane's byte offset from it, its line's length, the shortest and longest
// length, and the image step per clock.  Lanes past the direction's last line repeat
// that line (they load and store the same values at the same places, in lockstep).
struct WaveLines {
    int64_t base;
    uint32_t off;
    int len, minlen, maxlen, step;
};

__device__ __forceinline__ int line_count(int dx, int dy, int W, int H) { return dy == 0 ? H : dx == 0 ? W : W + H - 1; }

// (wave: a running number over the direction's waves, below the last line's)
template <int LPL, int DPADB>
__device__ __forceinline__ WaveLines wave_lines(int dx, int dy, int wave, int W, int H, int lane_bytes)
{
    constexpr int kLines = 64 / LPL;
    const int nlines = line_count(dx, dy, W, H);
    WaveLines g;
    g.minlen = 1 << 30;
    g.maxlen = 0;
    g.base = (int64_t)1 << 60;
    int64_t mine = 0;
    const int sub = (int)(threadIdx.x & 63) / LPL;
#pragma unroll
    for (int i = 0; i < kLines; ++i) {
        int x, y, len;
        line_start(dx, dy, min(wave * kLines + i, nlines - 1), W, H, x, y, len);
        const int64_t at = (int64_t)y * W + x;
        g.base = at < g.base ? at : g.base;
        g.minlen = min(g.minlen, len);
        g.maxlen = max(g.maxlen, len);
        if (sub == i) {
            mine = at;
            g.len = len;
        }
    }
    g.off = lane_bytes < DPADB ? (uint32_t)(mine - g.base) * DPADB + lane_bytes : kOff;  // idle lanes: nowhere
    g.step = dy * W + dx;
    return g;
}

// Issue priority from a wave's remaining work relative to the launch's largest:
// the waves sharing a SIMD then drain in order of remaining work and finish
// together instead of the longest running on alone.
__device__ __forceinline__ void set_priority(int remaining, int max_work)
{
    if (remaining > max_work / 100 * 43) __builtin_amdgcn_s_setprio(3);
    else if (remaining > max_work / 100 * 21) __builtin_amdgcn_s_setprio(2);
    else if (remaining > max_work / 100 * 7) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

// The S pixels of a line from index q*S on, walked forwards or (back) backwards, in a
// buffer of path-layout values: the resource of their first address in memory, and
// each step's scalar offset from it.
struct Segment {
    __amdgpu_buffer_rsrc_t rs;
    int stride;  // bytes per pixel of the line in memory order (>= 0)
    bool down;   // the walk runs against memory order
};
template <int S, int DPADB>
__device__ __forceinline__ Segment segment(const uint8_t *buf, const WaveLines &g, int q, bool back)
{
    const bool neg = g.step < 0;
    const int64_t first = g.base + (int64_t)(q * S + (neg ? S - 1 : 0)) * g.step;
    return Segment{open_buffer(buf + first * DPADB), (neg ? -g.step : g.step) * DPADB, neg != back};
}
// offset of the walk's step s
template <int S>
__device__ __forceinline__ int at_step(const Segment &b, int s)
{
    return (b.down ? S - 1 - s : s) * b.stride;
}
// the line index of the walk's step s of segment q
template <int S>
__device__ __forceinline__ int index_of(int q, int s, bool back)
{
    return q * S + (back ? S - 1 - s : s);
}

// ---------------------------------------------------------------- where costs come from
// A source loads what S pixels' costs need (Raw) and adds a register's costs to a step.
// WHOLE: every pixel of the segment exists on every line of the wave, and its costs
// need no care; otherwise pixels that do not exist cost nothing, which leaves a line's
// state before its first pixel as it is.

// A cost volume in the path buffers' layout.
template <int DPAD, int DPL, bool V16>
struct VolumeSource {
    using LV = Lane<DPL, V16>;
    static constexpr int kSeg = 4, kRing = 4;
    const uint8_t *vol;
    template <int S>
    struct Raw {
        uint32_t w[S][LV::NW];  // in walking order
    };
    template <int S>
    __device__ __forceinline__ bool whole(const WaveLines &g, int qa, int qb) const
    {
        return min(qa, qb) >= 0 && (max(qa, qb) + 1) * S <= g.minlen;
    }
    template <bool WHOLE, int S, class B>
    __device__ __forceinline__ void load(const WaveLines &g, int q, B back, Raw<S> &raw) const
    {
        const Segment b = segment<S, DPAD * (V16 ? 2 : 1)>(vol, g, q, back);
        static_for<S>([&](auto s) {
            LV::load(b.rs, WHOLE || (uint32_t)index_of<S>(q, s, back) < (uint32_t)g.len ? g.off : kOff, at_step<S>(b, s), raw.w[s]);
        });
    }
    template <bool WHOLE, int S, int J, class B>
    __device__ __forceinline__ uint32_t add(const Raw<S> &raw, int s, int, B, uint32_t t) const
    {
        return pk_add(t, LV::template get<J>(raw.w[s]));
    }
};

template <bool WIDE>
struct CensusWord;
template <>
struct CensusWord<false> {
    using T = uint32_t;
    static __device__ __forceinline__ uint32_t hamming(T a, T b) { return __popc(a ^ b); }
};
template <>
struct CensusWord<true> {
    using T = uint64_t;
    static __device__ __forceinline__ uint32_t hamming(T a, T b) { return __popcll(a ^ b); }
};

// N consecutive words of a census map from word `at` on, 16 bytes per load (as many
// whole loads as hold them; the words after are other words of the scratch)
template <bool WIDE, int N>
__device__ __forceinline__ void load_words(__amdgpu_buffer_rsrc_t rs, int at, typename CensusWord<WIDE>::T (&w)[N])
{
    constexpr int kPer = WIDE ? 2 : 4;
    static_for<(N + kPer - 1) / kPer>([&](auto ic) {
        constexpr int i = decltype(ic)::value * kPer;
        const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(rs, (at + i) * (16 / kPer), 0, 0);
        static_for<kPer>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            if constexpr (i + k < N) {
                if constexpr (WIDE) w[i + k] = ((uint64_t)v[2 * k + 1] << 32) | v[2 * k];
                else w[i + k] = v[k];
            }
        });
    });
}
// the same one word at a time, each at its own clamped position (segments that
// touch the image's ends)
template <bool WIDE, int N>
__device__ __forceinline__ void load_words_clamped(__amdgpu_buffer_rsrc_t rs, int at, int last,
                                                   typename CensusWord<WIDE>::T (&w)[N])
{
    static_for<N>([&](auto i) {
        const int p = min(max(at + i, 0), last);
        if constexpr (WIDE) {
            const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(rs, p * 8, 0, 0);
            w[i] = ((uint64_t)v[1] << 32) | v[0];
        } else {
            w[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, p * 4, 0, 0);
        }
    });
}

// Horizontal lines from the census words: the S pixels of a segment need S left words
// and, per lane, the S + DPL - 1 right words of columns x - d0 - j, consecutive words
// of a row.  The walk's direction is a constant (B: std::integral_constant): words sit
// in registers in memory order.  (wave: as wave_lines)
template <int DPAD, int DPL, int LPL, bool WIDE>
struct RowSource {
    using CW = CensusWord<WIDE>;
    using Word = typename CW::T;
    // (8 pixels of a lane with many disparities share more words: 24 loaded for 8
    // steps instead of 16 for 4; 1280x720, D = 128: 429 -> 423 us a call)
    static constexpr int kSeg = DPL <= 4 ? 4 : 8, kRing = DPL <= 4 ? 4 : 2;
    __amdgpu_buffer_rsrc_t rl, rr;  // from the wave's first row on
    int row, last;                  // the lane's row (words), the maps' last word
    int W, D, d0;
    uint32_t bits;
    template <int S>
    struct Raw {
        Word l[S], r[S + DPL - 1];
    };
    __device__ __forceinline__ RowSource(const void *cl, const void *cr, int wave, int W_, int H, int D_, uint32_t bits_)
        : W(W_), D(D_), bits(bits_)
    {
        constexpr int kLines = 64 / LPL;
        const int y0 = wave * kLines, y = min(y0 + (int)(threadIdx.x & 63) / LPL, H - 1);
        rl = open_buffer((const Word *)cl + (int64_t)y0 * W);
        rr = open_buffer((const Word *)cr + (int64_t)y0 * W);
        row = (y - y0) * W;
        last = (H - y0) * W - 1;
        d0 = (int)threadIdx.x % LPL * DPL;
    }
    template <int S>
    __device__ __forceinline__ bool whole(const WaveLines &, int qa, int qb) const
    {
        return D == DPAD && min(qa, qb) * S >= DPAD - 1 && (max(qa, qb) + 1) * S <= W;
    }
    template <bool WHOLE, int S, class B>
    __device__ __forceinline__ void load(const WaveLines &, int q, B, Raw<S> &raw) const
    {
        const int left = row + q * S, right = left - d0 - (DPL - 1);
        if constexpr (WHOLE) {
            load_words<WIDE>(rl, left, raw.l);
            load_words<WIDE>(rr, right, raw.r);
        } else {
            load_words_clamped<WIDE>(rl, left, last, raw.l);
            load_words_clamped<WIDE>(rr, right, last, raw.r);
        }
    }
    template <bool WHOLE, int S, int J, class B>
    __device__ __forceinline__ uint32_t add(const Raw<S> &raw, int s, int q, B, uint32_t t) const
    {
        const int i = B::value ? S - 1 - s : s;  // the pixel within the segment
        auto cost = [&](int j) -> uint32_t {
            const uint32_t c = CW::hamming(raw.l[i], raw.r[i + DPL - 1 - j]);
            if constexpr (WHOLE) {
                return c;
            } else {
                const int x = q * S + i;
                return x >= W ? 0u : d0 + j >= D ? 255u : d0 + j <= x ? c : bits;
            }
        };
        // (each half takes its own count: no carry between them)
        t += cost(J);
        if constexpr (DPL > 1) t += cost(J + DPL / 2) << 16;
        return t;
    }
};

// A wave keeps a ring of kRing segments of kSeg steps' costs, loaded kRing - 1 ahead:
// vector loads and stores complete in issue order, so waiting for a load also waits for
// the stores issued before it, and stores take longer.  The ring is unrolled (16 steps a
// block, each slot in fixed registers); longer rings cost more instruction cache than
// they gain (32 steps a block: 54 -> 72 us at 320x240, 24 steps: no change).

// ---------------------------------------------------------------- one direction from the cost volume
template <int DPAD, int DPL, int LPL, bool V16>
__device__ __forceinline__ void run_single(const VolumeSource<DPAD, DPL, V16> &src, uint8_t *out, const WaveLines &g, uint32_t p1, uint32_t p2,
                                           int cost, int max_work)
{
    using LV = Lane<DPL, V16>;
    using L = Line<DPL, LPL, DPAD / DPL, V16>;
    using SRC = VolumeSource<DPAD, DPL, V16>;
    constexpr int S = SRC::kSeg, R = SRC::kRing, kDpadB = DPAD * (V16 ? 2 : 1), N = LV::N;
    const int lane = (int)threadIdx.x % LPL;
    L line;
    line.clear();
    const int nseg = (g.maxlen + S - 1) / S;
    typename SRC::template Raw<S> ring[R];
    auto block = [&](auto wc, int k) {
        constexpr bool WHOLE = decltype(wc)::value;
        static_for<R>([&](auto r) {
            if (!WHOLE && k + r >= nseg) return;
            src.template load<WHOLE>(g, k + r + R - 1, false, ring[(r + R - 1) % R]);
            const Segment o = segment<S, kDpadB>(out, g, k + r, false);
            static_for<S>([&](auto s) {
                const uint32_t ub = both(L::base(line.u));
                line.step(p1, p2, lane, [&](auto j, uint32_t t) {
                    return src.template add<WHOLE, S, decltype(j)::value>(ring[r], s, 0, false, t);
                });
                uint32_t v[N], m[LV::NW];
#pragma unroll
                for (int j = 0; j < N; ++j) v[j] = V16 ? line.U[j] : pk_sub(line.U[j], ub);
                LV::pack(v, m);
                LV::template store<kStoreAux>(o.rs, WHOLE || (k + r) * S + s < g.len ? g.off : kOff, at_step<S>(o, s), m);
            });
        });
        line.rebase();
    };
    static_for<R - 1>([&](auto r) { src.template load<false>(g, r, false, ring[r]); });
    for (int k = 0; k < nseg; k += R) {
        set_priority((g.maxlen - k * S) * cost, max_work);
        if ((k + 2 * R - 1) * S <= g.minlen) block(std::true_type{}, k);
        else block(std::false_type{}, k);
    }
}

// ---------------------------------------------------------------- a direction and its opposite
// Two waves share a group of lines: wave `back` 0 walks them forwards, 1 backwards.
// Each first walks its own half without storing values, only its state before every
// segment of SUMS steps (in the slot of the segment's first pixel of `out`); after a
// barrier it walks on through the other's half: there, per segment, it recomputes the
// other direction's values from the state the other wave stored, keeps them in
// registers, walks the segment itself and stores the sums.  Three steps of work per
// pixel in all, one and a half per wave in a row.
// (live: the wave has lines; all waves of a block meet at the barrier)
template <int DPAD, int DPL, int LPL, bool V16, int SUMS, class SRC, class B>
__device__ __forceinline__ void run_pair(const SRC &src, uint8_t *out, const WaveLines &g, bool live, B back, uint32_t p1,
                                         uint32_t p2, int cost, int max_work)
{
    using LV = Lane<DPL, V16>;
    using L = Line<DPL, LPL, DPAD / DPL, V16>;
    constexpr int kDpadB = DPAD * (V16 ? 2 : 1), N = LV::N, NW = LV::NW;
    const int lane = (int)threadIdx.x % LPL;
    const int nseg = (g.maxlen + SUMS - 1) / SUMS;
    const int half = back ? nseg - nseg / 2 : nseg / 2;  // segments of the wave's own half
    L mine;
    mine.clear();
    if (live) {
        constexpr int S = SRC::kSeg, R = SRC::kRing, kPer = SUMS / S;
        static_assert(SUMS % S == 0 && (R * S) % SUMS == 0, "states fall on load segments");
        typename SRC::template Raw<S> ring[R];
        const int nall = nseg * kPer, nload = half * kPer;
        auto seg = [&](int k) { return back ? nall - 1 - k : k; };  // load segment k of the walk
        auto block = [&](auto wc, int k) {
            constexpr bool WHOLE = decltype(wc)::value;
            static_for<R>([&](auto r) {
                if (!WHOLE && k + r >= nload) return;
                src.template load<WHOLE>(g, seg(k + r + R - 1), back, ring[(r + R - 1) % R]);
                const int here = seg(k + r);
                static_for<S>([&](auto s) {
                    mine.step(p1, p2, lane, [&](auto j, uint32_t t) {
                        return src.template add<WHOLE, S, decltype(j)::value>(ring[r], s, here, back, t);
                    });
                });
                if constexpr ((r + 1) * S % SUMS == 0) {
                    // the state before the walk's next segment.  (Values of padding
                    // disparities can exceed a byte: 255 is still above every real
                    // value plus P2 - P1, so the clamp changes no real one.)
                    const uint32_t ub = both(mine.u);
                    uint32_t v[N], m[NW];
#pragma unroll
                    for (int j = 0; j < N; ++j) {
                        v[j] = pk_sub(mine.U[j], ub);
                        if constexpr (!V16) {
                            mine.U[j] = v[j];
                            v[j] = pk_min(v[j], 0x00FF00FFu);
                        }
                    }
                    if constexpr (!V16) mine.u = 0;
                    LV::pack(v, m);
                    const int next = (k + r + 1) / kPer, q = back ? nseg - 1 - next : next;
                    const Segment o = segment<SUMS, kDpadB>(out, g, q, false);
                    LV::template store<0>(o.rs, next < half && (WHOLE || q * SUMS < g.len) ? g.off : kOff, at_step<SUMS>(o, 0), m);
                }
            });
        };
        static_for<R - 1>([&](auto r) { src.template load<false>(g, seg(r), back, ring[r]); });
        for (int k = 0; k < nload; k += R) {
            set_priority((3 * nseg * SUMS / 2 - k * S) * cost, max_work);
            const int ahead = k + 2 * R - 2;  // the block's last load
            if (k + R <= nload && ahead < nall && src.template whole<S>(g, seg(k), seg(ahead))) block(std::true_type{}, k);
            else block(std::false_type{}, k);
        }
    }
    // the states are in memory before the other wave reads them
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (!live) return;

    constexpr int S = SUMS;
    auto seg = [&](int k) { return back ? nseg - 1 - k : k; };  // segment k of the walk
    using Raw = typename SRC::template Raw<S>;
    Raw ring[2];
    uint32_t states[2][NW];
    auto load = [&](auto wc, int k, Raw &w, uint32_t (&m)[NW]) {
        constexpr bool WHOLE = decltype(wc)::value;
        if (!WHOLE && k >= nseg) return;
        const int q = seg(k);
        src.template load<WHOLE>(g, q, back, w);
        // (the other wave starts from zeros in its first segment, this walk's last)
        const Segment o = segment<S, kDpadB>(out, g, q, false);
        LV::load(o.rs, WHOLE || (k < nseg - 1 && q * S < g.len) ? g.off : kOff, at_step<S>(o, 0), m);
    };
    auto sums = [&](auto wc, int k, const Raw &w, const uint32_t (&state)[NW]) {
        constexpr bool WHOLE = decltype(wc)::value;
        const int q = seg(k);
        L other;
        uint32_t F[S][N], fu[S];
        static_for<N>([&](auto j) { other.U[j] = LV::template get<j>(state); });
        other.u = 0;  // a state is normalised
        static_for<S>([&](auto sc) {
            constexpr int s = S - 1 - decltype(sc)::value;
            fu[s] = L::base(other.u);
            other.step(p1, p2, lane, [&](auto j, uint32_t t) {
                return src.template add<WHOLE, S, decltype(j)::value>(w, s, q, back, t);
            });
#pragma unroll
            for (int j = 0; j < N; ++j) F[s][j] = other.U[j];
        });
        const Segment o = segment<S, kDpadB>(out, g, q, back);
        static_for<S>([&](auto s) {
            const uint32_t sub = both(L::base(mine.u) + fu[s]);
            mine.step(p1, p2, lane, [&](auto j, uint32_t t) {
                return src.template add<WHOLE, S, decltype(j)::value>(w, s, q, back, t);
            });
            uint32_t v[N], m[NW];
#pragma unroll
            for (int j = 0; j < N; ++j) v[j] = V16 ? pk_add(mine.U[j], F[s][j]) : pk_sub(pk_add(mine.U[j], F[s][j]), sub);
            LV::pack(v, m);
            LV::template store<kStoreAux>(o.rs, WHOLE || index_of<S>(q, s, back) < g.len ? g.off : kOff, at_step<S>(o, s), m);
        });
        mine.rebase();
    };
    auto block = [&](auto wc, int k) {
        constexpr bool WHOLE = decltype(wc)::value;
        load(wc, k + 1, ring[1], states[1]);
        sums(wc, k, ring[0], states[0]);
        if (!WHOLE && k + 1 >= nseg) return;
        load(wc, k + 2, ring[0], states[0]);
        sums(wc, k + 1, ring[1], states[1]);
    };
    load(std::false_type{}, half, ring[0], states[0]);
    for (int k = half; k < nseg; k += 2) {
        set_priority(2 * (nseg - k) * S * cost, max_work);
        if (k + 2 < nseg - 1 && src.template whole<S>(g, seg(k), seg(k + 2))) block(std::true_type{}, k);
        else block(std::false_type{}, k);
    }
}

// ---------------------------------------------------------------- one horizontal direction from census words
// Horizontal lines (rows), HDIR +1 left to right, -1 right to left.  At column x a
// lane needs the right words of columns x - d0 - j, j < DPL: one new word per step,
// at columns that advance with x, so a segment's S new words are S consecutive
// words of the row.
template <int DPAD, int DPL, int LPL, bool WIDE, int HDIR>
__device__ __forceinline__ void run_horizontal(const void *cl, const void *cr, uint8_t *out, int wave, int W, int H, int D,
                                               uint32_t bits, uint32_t p1, uint32_t p2, int cost, int max_work)
{
    using LV = Lane<DPL, false>;
    using L = Line<DPL, LPL, DPAD / DPL, false>;
    using CW = CensusWord<WIDE>;
    using Word = typename CW::T;
    constexpr int S = 4, R = 4, N = LV::N, kDpad = DPAD, kLines = 64 / LPL;
    const int lane = (int)threadIdx.x % LPL, d0 = lane * DPL;
    const WaveLines g = wave_lines<LPL, kDpad>(HDIR, 0, wave, W, H, lane * DPL);
    const int y0 = wave * kLines, y = min(y0 + (int)(threadIdx.x & 63) / LPL, H - 1);
    // resources from the wave's first row on (a lane's offset stays below 4 rows)
    const __amdgpu_buffer_rsrc_t rl = open_buffer((const Word *)cl + (int64_t)y0 * W);
    const __amdgpu_buffer_rsrc_t rr = open_buffer((const Word *)cr + (int64_t)y0 * W);
    const int row = (y - y0) * W, last = (H - y0) * W - 1;  // the lane's row, the map's last word
    const int nseg = (W + S - 1) / S;
    // left words of segment k: columns lx .. lx + S - 1 in memory order; right words:
    // the S columns that enter the lane's window, in memory order
    auto lcol = [&](int k) { return HDIR > 0 ? k * S : W - S - k * S; };
    auto rcol = [&](int k) { return HDIR > 0 ? k * S - d0 : W - S - k * S - d0 - (DPL - 1); };
    // (uniform: true when no lane reads outside its row and no pixel of the segment
    // has x - d < 0)
    auto inside = [&](int k) { return HDIR > 0 ? k * S >= kDpad - 1 && (k + 1) * S <= W : W - (k + 1) * S >= kDpad - 1; };
    auto load = [&](auto wc, int k, Word (&wl)[S], Word (&wr)[S]) {
        if constexpr (decltype(wc)::value) {
            load_words<WIDE>(rl, row + lcol(k), wl);
            load_words<WIDE>(rr, row + rcol(k), wr);
        } else {
            load_words_clamped<WIDE>(rl, row + lcol(k), last, wl);
            load_words_clamped<WIDE>(rr, row + rcol(k), last, wr);
        }
    };
    L line;
    line.clear();
    // window: entry i of the S + DPL - 1 words a segment uses, in the order they
    // enter; the last DPL - 1 of a segment are the first of the next
    Word carry[DPL];
#pragma unroll
    for (int i = 0; i < DPL; ++i) carry[i] = 0;
    if constexpr (HDIR < 0) {
        // columns W - 1 - d0 - i, i < DPL - 1, have entered before the first step
#pragma unroll
        for (int i = 0; i < DPL - 1; ++i) {
            Word v[1];
            load_words_clamped<WIDE>(rr, row + W - 1 - d0 - i, last, v);
            carry[i] = v[0];
        }
    }
    const bool padded = D < kDpad;
    Word left[R][S], rights[R][S];
    auto run = [&](auto wc, int k, const Word (&wl)[S], const Word (&wr)[S]) {
        constexpr bool WHOLE = decltype(wc)::value;
        // words in the order they enter the lane's window
        Word win[S + DPL - 1];
#pragma unroll
        for (int i = 0; i < DPL - 1; ++i) win[i] = carry[i];
#pragma unroll
        for (int s = 0; s < S; ++s) win[DPL - 1 + s] = HDIR > 0 ? wr[s] : wr[S - 1 - s];
#pragma unroll
        for (int i = 0; i < DPL - 1; ++i) carry[i] = win[S + i];
        const Segment o = segment<S, kDpad>(out, g, k, false);
        static_for<S>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            const int x = HDIR > 0 ? k * S + s : W - 1 - k * S - s;
            const Word l = HDIR > 0 ? wl[s] : wl[S - 1 - s];
            // the lane's disparity j compares with window entry: HDIR > 0, newest is
            // column x - d0 (j = 0); HDIR < 0, newest is x - d0 - (DPL - 1)
            auto hamming = [&](int j) -> uint32_t {
                const uint32_t c = CW::hamming(l, HDIR > 0 ? win[s + DPL - 1 - j] : win[s + j]);
                if constexpr (!WHOLE) return d0 + j < D ? (j <= x - d0 ? c : bits) : 255u;
                return c;
            };
            const uint32_t ub = both(line.u);
            line.step(p1, p2, lane, [&](auto j, uint32_t t) {
                // (each half takes its own count: no carry between them)
                t += hamming(j);
                if constexpr (DPL > 1) t += hamming(j + N) << 16;
                return t;
            });
            uint32_t v[N], m[LV::NW];
#pragma unroll
            for (int j = 0; j < N; ++j) v[j] = pk_sub(line.U[j], ub);
            LV::pack(v, m);
            LV::template store<kStoreAux>(o.rs, WHOLE || k * S + s < W ? g.off : kOff, at_step<S>(o, s), m);
        });
    };
    auto block = [&](auto wc, int k) {
        constexpr bool WHOLE = decltype(wc)::value;
        static_for<R>([&](auto r) {
            if (!WHOLE && k + r >= nseg) return;
            constexpr int next = (r + R - 1) % R;
            load(wc, k + r + R - 1, left[next], rights[next]);
            run(wc, k + r, left[r], rights[r]);
        });
        line.rebase();
    };
    static_for<R - 1>([&](auto r) { load(std::false_type{}, r, left[r], rights[r]); });
    for (int k = 0; k < nseg; k += R) {
        set_priority((W - k * S) * cost, max_work);
        if (!padded && inside(k) && inside(k + 2 * R - 2)) block(std::true_type{}, k);
        else block(std::false_type{}, k);
    }
}

// ---------------------------------------------------------------- columns and diagonals from census words
// A block's 16 neighbouring lines of a vertical or diagonal direction.  At every clock
// they lie in one image row and 16 consecutive columns: line i of item k is the one
// that would enter the image's first row (of the walk) at column v = v0 + i, and a
// diagonal that enters through a side column starts at a later clock (until then its
// costs are 0, which leave its state as it is).  So the words the block needs for a
// clock are 16 left ones and Dpad + 15 right ones, and those of 16 clocks a tile in LDS;
// the next tile's words are on their way, in registers, while one is walked.  Bound by
// the issue of a step: 56 instructions at 96 disparities, 87 at 192, a third more at the
// image's sides.  Words read a clock ahead, counts that accumulate and packed border
// tests: 320x240, D = 96, 8 directions 88 -> 71 us a call, 1920x1080, D = 192 1326 -> 1290.
template <typename T>
using lds_t = __attribute__((address_space(3))) T;
__device__ __forceinline__ uint32_t lds_address(const uint32_t *p) { return (uint32_t)(uint64_t)(const lds_t<uint32_t> *)p; }

constexpr int kTileClocks = 16;
// words of a tile: per clock Dpad + 15 right ones, then per clock 16 left ones
constexpr int column_tile_words(int dpad) { return kTileClocks * (dpad + kColumnLines - 1 + kColumnLines); }

template <int DPAD, int DPL>
__device__ __forceinline__ void run_columns(const void *cl, const void *cr, uint8_t *out, int item, int dx, int dy, int W, int H,
                                            int D, uint32_t bits, uint32_t p1, uint32_t p2, int cost, int max_work,
                                            uint32_t (*tile)[column_tile_words(DPAD)])
{
    using LV = Lane<DPL, false>;
    using L = Line<DPL, kLanesPerLine, DPAD / DPL, false>;
    using CW = CensusWord<false>;
    constexpr int T = kTileClocks, N = LV::N, kL = kColumnLines, kR = DPAD + kL - 1;  // left and right words of a clock
    constexpr int kRows = T / kWavesPerItem, kRl = (kR + 63) / 64;                     // clocks a wave loads; loads of one
    static_assert(kL == 64 / kLanesPerLine * kWavesPerItem && kRows * kL == 64, "a lane, a left word of the wave's clocks");
    const int lane64 = (int)threadIdx.x & 63, lane = (int)threadIdx.x % kLanesPerLine, line = (int)threadIdx.x / kLanesPerLine;
    const int w = uniform((int)threadIdx.x >> 6), d0 = lane * DPL;
    const ColumnLines g = column_lines(dx, item, W, H);
    // this lane's line: its first clock and its length
    const int v = g.v0 + line, first = dx == 0 ? 0 : max(0, dx > 0 ? -v : v - W + 1);
    const int len = line < g.n ? (dx == 0 ? H : min(H, dx > 0 ? W - v : v + 1)) - first : 0;
    const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc((void *)cl, 0, W * H * 4, kBufferWord3);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void *)cr, 0, W * H * 4, kBufferWord3);
    const int step = dy * W + dx;
    // word index of column v0 + dx c of clock c's row
    auto at = [&](int c) { return (dy > 0 ? c : H - 1 - c) * W + g.v0 + dx * c; };
    uint32_t nr[kRows][kRl], nl;
    // (positions outside an image row are other words of the map, or past it zeros: they
    // only reach costs that are replaced and pixels that do not exist.  Positions before
    // the map are clamped: a wrapped register plus an instruction's offset is no offset.)
    auto fetch = [&](int c) {
        const int base = at(c + kRows * w);
#pragma unroll
        for (int i = 0; i < kRows; ++i)
#pragma unroll
            for (int m = 0; m < kRl; ++m)
                nr[i][m] = __builtin_amdgcn_raw_buffer_load_b32(rr, max((base + i * step - (DPAD - 1) + 64 * m + lane64) * 4, 0), 0, 0);
        nl = __builtin_amdgcn_raw_buffer_load_b32(rl, max((base + lane64 / kL * step + lane64 % kL) * 4, 0), 0, 0);
    };
    auto keep = [&](uint32_t *t) {
#pragma unroll
        for (int i = 0; i < kRows; ++i)
#pragma unroll
            for (int m = 0; m < kRl; ++m)
                if (64 * (m + 1) <= kR || lane64 < kR - 64 * m) t[(kRows * w + i) * kR + 64 * m + lane64] = nr[i][m];
        t[T * kR + kRows * w * kL + lane64] = nl;
    };
    // LDS traffic of the waves ordered; stores on their way are not waited for
    auto meet = [&] {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // (idle lanes read the last active lane's words)
    const int left_at = T * kR + line, right_at = line + DPAD - DPL - min(d0, DPAD - DPL);
    const uint32_t off = d0 < DPAD ? (uint32_t)(line * DPAD + d0) : kOff;
    uint32_t pad[N];  // at least this for the padding disparities, nothing for the others
#pragma unroll
    for (int j = 0; j < N; ++j) pad[j] = (d0 + j < D ? 0u : 255u) | (DPL > 1 && d0 + j + N >= D ? 255u << 16 : 0u);
    const uint32_t bits2 = both(bits);
    L state;
    state.clear();
    // EDGE: a line without a pixel at some clock, or a cost where x - d < 0
    auto walk = [&](auto edge, auto padded, int c, const uint32_t *t) {
        constexpr bool EDGE = decltype(edge)::value, PAD = decltype(padded)::value;
        const bool neg = step < 0;
        const __amdgpu_buffer_rsrc_t rs = open_buffer(out + (int64_t)(at(c) + (neg ? (T - 1) * step : 0)) * DPAD);
        const int stride = (neg ? -step : step) * DPAD;
        // the next clock's words are read before this one's step.  (The addresses are kept
        // running and opaque: as large constants off one base they took an add per read.)
        uint32_t al = lds_address(t + left_at), ar = lds_address(t + right_at);
        uint32_t left[2], right[2][DPL];
        auto read = [&](uint32_t &l, uint32_t (&r)[DPL]) {
            l = *(const lds_t<uint32_t> *)al;
#pragma unroll
            for (int k = 0; k < DPL; ++k) r[k] = ((const lds_t<uint32_t> *)ar)[k];
            al += kL * 4;
            ar += kR * 4;
            asm volatile("" : "+v"(al), "+v"(ar));
        };
        read(left[0], right[0]);
        static_for<T>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            if constexpr (s + 1 < T) read(left[(s + 1) & 1], right[(s + 1) & 1]);
            const uint32_t l = left[s & 1], (&r)[DPL] = right[s & 1];
            const bool on = (uint32_t)(c + s - first) < (uint32_t)len;
            // disparities d0 + j with j < lim stay inside the right image; the others' costs are
            // raised to `bits`: 64 (j + 1 - lim), or 0, is at least that
            const int lim = v + dx * (c + s) - d0 + 1;
            const uint32_t lim64 = EDGE ? both((uint32_t)min(max(lim, 0), DPL) * 64) : 0u, live = on ? ~0u : 0u;
            auto hamming = [&](int j) { return CW::hamming(l, r[DPL - 1 - j]); };
            const uint32_t ub = both(state.u);
            state.step(p1, p2, lane, [&](auto jc, uint32_t x) {
                constexpr int j = decltype(jc)::value;
                // (each half takes its own count: no carry between them)
                if constexpr (EDGE || PAD) {
                    uint32_t n = hamming(j);
                    if constexpr (DPL > 1) n |= hamming(j + N) << 16;
                    if constexpr (EDGE) {
                        const u16x2_t beyond = __builtin_elementwise_sub_sat(u16x2_t{64 * (j + 1), 64 * (j + 1 + N)}, h2(lim64));
                        n = pk_max3(n, pk_min(w1(beyond), bits2), pad[j]) & live;
                    } else {
                        n = pk_max(n, pad[j]);
                    }
                    return pk_add(x, n);
                } else {
                    x += hamming(j);
                    asm("" : "+v"(x));  // counted onto the sum, not added to it afterwards
                    if constexpr (DPL > 1) x += hamming(j + N) << 16;
                    return x;
                }
            });
            uint32_t o[N], m[LV::NW];
#pragma unroll
            for (int j = 0; j < N; ++j) o[j] = pk_sub(state.U[j], ub);
            LV::pack(o, m);
            LV::template store<kStoreAux>(rs, !EDGE || on ? off : kOff, (neg ? T - 1 - s : s) * stride, m);
        });
        state.rebase();
    };
    fetch(g.begin);
    keep(tile[0]);
    meet();
    for (int c = g.begin, b = 0; c < g.end; c += T, b ^= 1) {
        set_priority((g.end - c) * cost, max_work);
        // (the last tile's look-ahead is not used)
        fetch(c + T);
        const bool inside = g.n == kColumnLines && c >= g.all_in && c + T <= g.any_out &&
                            g.v0 + (dx < 0 ? -(c + T - 1) : dx * c) >= DPAD - 1;
        if (inside && D == DPAD) walk(std::false_type{}, std::false_type{}, c, tile[b]);
        else if (inside) walk(std::false_type{}, std::true_type{}, c, tile[b]);
        else walk(std::true_type{}, std::true_type{}, c, tile[b]);
        keep(tile[b ^ 1]);
        meet();
    }
}

// ---------------------------------------------------------------- matching costs
// The cost volume: byte popcount(cL(x) ^ cR(x - d)) per pixel and disparity, d
// fastest; `bits` where x - d < 0 and 255 (above every path value a real one can be
// compared with) where d >= D.  A thread makes 16 disparities of two adjacent
// pixels (17 right words from LDS for 32 values) and stores 16 bytes for each.
// Bound by the volume's stores, which keep the default cache policy: the
// aggregation reads the volume several times, from the last-level cache when it
// fits there.
constexpr int kCostDisp = 16;
__host__ __device__ constexpr int cost_pairs(int dpad) { return 256 / (dpad / kCostDisp); }  // pixel pairs per block
constexpr int cost_tiles(int dpad, int W) { return (W + 2 * cost_pairs(dpad) - 1) / (2 * cost_pairs(dpad)); }  // per row

template <int DPL, bool WIDE>
__device__ __forceinline__ void cost_tile(const AggregateArgs &a, int y, int tile, typename CensusWord<WIDE>::T *lds)
{
    using CW = CensusWord<WIDE>;
    using Word = typename CW::T;
    constexpr int kDpad = kLanesPerLine * DPL, kChunks = kDpad / kCostDisp, kPairs = cost_pairs(kDpad), kPx = 2 * kPairs;
    const int W = uniform(a.W), D = uniform(a.D);
    const int x0 = tile * kPx;
    if (x0 >= W) return;  // (the widest image of a batch sets the grid)
    const Word *cl = uniform((const Word *)a.census_l) + (int64_t)y * W;
    const Word *cr = uniform((const Word *)a.census_r) + (int64_t)y * W;
    // right words of columns x0 - (Dpad - 1) .. x0 + kPx - 1
    for (int i = threadIdx.x; i < kDpad - 1 + kPx; i += 256) lds[i] = cr[min(max(x0 - (kDpad - 1) + i, 0), W - 1)];
    __syncthreads();
    const int c = (int)threadIdx.x % kChunks, p = (int)threadIdx.x / kChunks;
    const int x = x0 + 2 * p, d0 = c * kCostDisp;
    if (p >= kPairs || x >= W) return;
    const Word l0 = cl[x], l1 = cl[min(x + 1, W - 1)];
    // window word i: column x + 1 - d0 - i; pixel 0 uses 1 + j, pixel 1 uses j
    Word r[kCostDisp + 1];
#pragma unroll
    for (int i = 0; i <= kCostDisp; ++i) r[i] = lds[2 * p + kDpad - d0 - i];
    uint32_t w0[4], w1v[4];
    const bool edge = D < kDpad || x0 < kDpad - 1;
    const uint32_t bits = a.bits;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t v0 = 0, v1 = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int j = 4 * q + b;
            uint32_t c0 = CW::hamming(l0, r[j + 1]), c1 = CW::hamming(l1, r[j]);
            if (edge) {
                c0 = d0 + j < D ? (x - d0 - j >= 0 ? c0 : bits) : 255u;
                c1 = d0 + j < D ? (x + 1 - d0 - j >= 0 ? c1 : bits) : 255u;
            }
            v0 |= c0 << (8 * b);
            v1 |= c1 << (8 * b);
        }
        w0[q] = v0;
        w1v[q] = v1;
    }
    uint8_t *o = uniform(a.cost) + ((int64_t)y * W + x) * kDpad + d0;
    *(__attribute__((address_space(1))) u32x4_t *)o = u32x4_t{w0[0], w0[1], w0[2], w0[3]};
    if (x + 1 < W) *(__attribute__((address_space(1))) u32x4_t *)(o + kDpad) = u32x4_t{w1v[0], w1v[1], w1v[2], w1v[3]};
}

template <int DPL>
constexpr int cost_lds_words() { return kLanesPerLine * DPL + 2 * cost_pairs(kLanesPerLine * DPL); }

template <int DPL, bool WIDE>
__global__ __launch_bounds__(256) void cost_kernel(AggregateArgs a)
{
    __shared__ typename CensusWord<WIDE>::T lds[cost_lds_words<DPL>()];
    cost_tile<DPL, WIDE>(a, (int)blockIdx.y, (int)blockIdx.x, lds);
}

// batch form: one item per (slot, row)
template <int DPL, bool WIDE>
__global__ __launch_bounds__(256) void cost_queue_kernel(AggregateQueue q)
{
    __shared__ typename CensusWord<WIDE>::T lds[cost_lds_words<DPL>()];
    const uint32_t it = __builtin_amdgcn_readfirstlane(q.cost_items[blockIdx.x]);
    cost_tile<DPL, WIDE>(q.slots[it >> 20], (int)(it & 0xFFFFFu), (int)blockIdx.y, lds);
}

// ---------------------------------------------------------------- the aggregation launch
// Steps between two states of a pair: 8, or 4 where the forward values of 8 steps
// would not fit the registers.
constexpr int sum_steps(int dpl, bool v16) { return v16 && dpl >= 12 ? 4 : 8; }

// One block of four waves: the lines of item `item` of the slot (a running number
// over its units).  A block's waves have about the same work and land on the four
// SIMDs of a unit.
template <int DPL, bool WIDE, int HL>
__device__ __forceinline__ void aggregate_item(const AggregateArgs &a, int item)
{
    constexpr int kDpad = kLanesPerLine * DPL, LD = lane_disparities(kDpad, kLanesPerLine), HD = row_disparities(kDpad, HL, WIDE);
    const int nunits = uniform(a.nunits);
    int unit = 0;
#pragma unroll
    for (int k = 1; k < 8; ++k) unit += (k < nunits && item >= a.item_begin[k]) ? 1 : 0;
    unit = uniform(unit);
    item = uniform(item - a.item_begin[unit]);
    const int w = uniform((int)threadIdx.x >> 6);
    const int dx = uniform(a.dx[unit]), dy = uniform(a.dy[unit]);
    uint8_t *out = uniform(a.out[unit]);
    const int W = uniform(a.W), H = uniform(a.H), max_work = uniform(a.max_item_work);
    const int nlines = line_count(dx, dy, W, H);
    const uint32_t p1 = both(uniform(a.p1)), p2 = both(uniform(a.p2));
    const bool pair = uniform(a.pair[unit]) != 0;
    const int wave = pair ? item * (kWavesPerItem / 2) + w / 2 : item * kWavesPerItem + w;
    if (dy == 0) {
        constexpr int cost = agg_step_cost(HD, HL);
        const bool live = wave * (64 / HL) < nlines;
        const void *cl = uniform(a.census_l), *cr = uniform(a.census_r);
        const int D = uniform(a.D);
        const uint32_t bits = uniform(a.bits);
        if constexpr (row_pairs_built(HL, WIDE))
            if (pair) {
                const WaveLines g = wave_lines<HL, kDpad>(1, 0, wave, W, H, (int)threadIdx.x % HL * HD);
                const RowSource<kDpad, HD, HL, WIDE> src(cl, cr, wave, W, H, D, bits);
                constexpr int kSums = sum_steps(HD, false);
                if (w & 1) run_pair<kDpad, HD, HL, false, kSums>(src, out, g, live, std::true_type{}, p1, p2, cost, max_work);
                else run_pair<kDpad, HD, HL, false, kSums>(src, out, g, live, std::false_type{}, p1, p2, cost, max_work);
                return;
            }
        if (!live) return;
        if constexpr (WIDE)
            if (uniform(a.row_costs)) {
                const WaveLines g = wave_lines<HL, kDpad>(dx, 0, wave, W, H, (int)threadIdx.x % HL * HD);
                return run_single<kDpad, HD, HL, false>(VolumeSource<kDpad, HD, false>{uniform(a.cost)}, out, g, p1, p2, cost,
                                                        max_work);
            }
        if (dx > 0) run_horizontal<kDpad, HD, HL, WIDE, 1>(cl, cr, out, wave, W, H, D, bits, p1, p2, cost, max_work);
        else run_horizontal<kDpad, HD, HL, WIDE, -1>(cl, cr, out, wave, W, H, D, bits, p1, p2, cost, max_work);
    } else {
        constexpr int cost = agg_step_cost(LD, kLanesPerLine), kLines = 64 / kLanesPerLine;
        const bool live = wave * kLines < nlines;
        const int lane = (int)threadIdx.x % kLanesPerLine;
        const WaveLines g = wave_lines<kLanesPerLine, kDpad>(dx, dy, wave, W, H, lane * LD);
        const VolumeSource<kDpad, LD, false> src{uniform(a.cost)};
        if (pair)
            run_pair<kDpad, LD, kLanesPerLine, false, sum_steps(LD, false)>(src, out, g, live, (w & 1) != 0, p1, p2, cost, max_work);
        else if (live)
            run_single<kDpad, LD, kLanesPerLine, false>(src, out, g, p1, p2, cost, max_work);
    }
}

// One block of four waves where no unit reads a cost volume: single directions only.
template <int DPL, int HL>
__device__ __forceinline__ void census_item(const AggregateArgs &a, int item,
                                            uint32_t (*tile)[column_tile_words(kLanesPerLine * DPL)])
{
    constexpr int kDpad = kLanesPerLine * DPL, LD = column_disparities(kDpad), HD = row_disparities(kDpad, HL, false);
    const int nunits = uniform(a.nunits);
    int unit = 0;
#pragma unroll
    for (int k = 1; k < 8; ++k) unit += (k < nunits && item >= a.item_begin[k]) ? 1 : 0;
    unit = uniform(unit);
    item = uniform(item - a.item_begin[unit]);
    const int dx = uniform(a.dx[unit]), dy = uniform(a.dy[unit]);
    uint8_t *out = uniform(a.out[unit]);
    const int W = uniform(a.W), H = uniform(a.H), D = uniform(a.D), max_work = uniform(a.max_item_work);
    const uint32_t p1 = both(uniform(a.p1)), p2 = both(uniform(a.p2)), bits = uniform(a.bits);
    const void *cl = uniform(a.census_l), *cr = uniform(a.census_r);
    if (dy == 0) {
        constexpr int cost = agg_step_cost(HD, HL);
        const int wave = item * kWavesPerItem + uniform((int)threadIdx.x >> 6);
        if (wave * (64 / HL) >= H) return;
        if (dx > 0) run_horizontal<kDpad, HD, HL, false, 1>(cl, cr, out, wave, W, H, D, bits, p1, p2, cost, max_work);
        else run_horizontal<kDpad, HD, HL, false, -1>(cl, cr, out, wave, W, H, D, bits, p1, p2, cost, max_work);
    } else {
        run_columns<kDpad, LD>(cl, cr, out, item, dx, dy, W, H, D, bits, p1, p2, agg_step_cost(LD, kLanesPerLine), max_work, tile);
    }
}

// (three waves per SIMD: 1920x1080, D = 192, 8 directions 1345 / 1326 / 1432 us a call with
// two / three / four)
template <int DPL, int HL>
__global__ __launch_bounds__(64 * kWavesPerItem) __attribute__((amdgpu_waves_per_eu(3, 3))) void census_aggregate_kernel(AggregateArgs a)
{
    __shared__ __align__(16) uint32_t tile[2][column_tile_words(kLanesPerLine * DPL)];
    census_item<DPL, HL>(a, (int)blockIdx.x, tile);
}

template <int DPL, int HL>
__global__ __launch_bounds__(64 * kWavesPerItem) __attribute__((amdgpu_waves_per_eu(3, 3))) void census_aggregate_queue_kernel(AggregateQueue q)
{
    __shared__ __align__(16) uint32_t tile[2][column_tile_words(kLanesPerLine * DPL)];
    const uint32_t it = __builtin_amdgcn_readfirstlane(q.items[blockIdx.x]);
    census_item<DPL, HL>(q.slots[it >> 20], (int)(it & 0xFFFFFu), tile);
}

// Registers for two waves per SIMD: a step is a serial chain, and the scheduler fills
// its gaps with other steps' work when it has the registers (2 waves with up to 256
// registers beat 3 with 168).
template <int DPL, bool WIDE, int HL>
__global__ __launch_bounds__(64 * kWavesPerItem) __attribute__((amdgpu_waves_per_eu(2, 2))) void aggregate_kernel(AggregateArgs a, int first)
{
    aggregate_item<DPL, WIDE, HL>(a, first + (int)blockIdx.x);
}

// items (slot << 20 | item) in launch order, largest estimated work first
template <int DPL, bool WIDE, int HL>
__global__ __launch_bounds__(64 * kWavesPerItem) __attribute__((amdgpu_waves_per_eu(2, 2))) void aggregate_queue_kernel(AggregateQueue q)
{
    const uint32_t it = __builtin_amdgcn_readfirstlane(q.items[blockIdx.x]);
    aggregate_item<DPL, WIDE, HL>(q.slots[it >> 20], (int)(it & 0xFFFFFu));
}

// Launches the costs (when a unit reads them) and the lines of one slot (a) or of
// every slot of a queue (q): nitems blocks.  A unit that writes over the cost volume (a slot
// alone) runs after everything else has read it: the remaining blocks, in a launch of
// their own.
template <int DPL, bool WIDE, int HL>
hipError_t launch_aggregation(const AggregateArgs *a, const AggregateQueue *q, int nitems, hipStream_t s)
{
    constexpr int kDpad = kLanesPerLine * DPL;
    const dim3 block(64 * kWavesPerItem);
    if (a ? counts_census(*a) : q->census != 0) {
        if constexpr (WIDE) return hipErrorInvalidValue;
        else if (a) hipLaunchKernelGGL((census_aggregate_kernel<DPL, HL>), dim3(nitems), block, 0, s, *a);
        else hipLaunchKernelGGL((census_aggregate_queue_kernel<DPL, HL>), dim3(nitems), block, 0, s, *q);
    } else if (a) {
        const int rest = a->item_begin[a->nunits] - nitems;
        if (a->cost) hipLaunchKernelGGL((cost_kernel<DPL, WIDE>), dim3(cost_tiles(kDpad, a->W), a->H), dim3(256), 0, s, *a);
        if (nitems > 0) hipLaunchKernelGGL((aggregate_kernel<DPL, WIDE, HL>), dim3(nitems), block, 0, s, *a, 0);
        if (rest > 0) hipLaunchKernelGGL((aggregate_kernel<DPL, WIDE, HL>), dim3(rest), block, 0, s, *a, nitems);
    } else {
        if (q->ncost > 0)
            hipLaunchKernelGGL((cost_queue_kernel<DPL, WIDE>), dim3(q->ncost, cost_tiles(kDpad, q->cost_width)), dim3(256), 0, s, *q);
        hipLaunchKernelGGL((aggregate_queue_kernel<DPL, WIDE, HL>), dim3(nitems), block, 0, s, *q);
    }
    return hipGetLastError();
}

template <int DPL, bool WIDE>
hipError_t launch_aggregation_lanes(const AggregateArgs *a, const AggregateQueue *q, int grid, int hl, hipStream_t s)
{
    constexpr int kDpad = kLanesPerLine * DPL;
    hl = effective_lanes(kDpad, hl);
    if constexpr (effective_lanes(kDpad, 32) == 32)
        if (hl == 32) return launch_aggregation<DPL, WIDE, 32>(a, q, grid, s);
    if constexpr (effective_lanes(kDpad, 64) == 64)
        if (hl == 64) return launch_aggregation<DPL, WIDE, 64>(a, q, grid, s);
    return launch_aggregation<DPL, WIDE, 16>(a, q, grid, s);
}

}  // namespace

}  // namespace ss
