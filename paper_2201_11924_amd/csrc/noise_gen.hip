// On-device IR noise for simulated cameras (Sec. VI-C): the multiplicative
// speckle gamma and the additive thermal noise n of Eq. (7), drawn on the GPU
// (Eq. (8) and the fit of Sec. VII-C give the distributions; Table X's noise
// scale s maps gamma -> 1 + s (gamma - 1) and n -> s n), then applied to the
// clean image in the same pass, so a rendered IR pair goes to the census with
// no host round trip.
//
// Random numbers: Philox4x32-10 (Salmon et al., SC'11), counter (pixel, stream,
// attempt, 0), key (seed low, seed high); uniforms from the top 23 bits,
// ((x >> 9) + 0.5) 2^-23; normals by Box-Muller and the gamma by the method of
// Marsaglia and Tsang (2000), both in double precision and rounded to float32.
#include <math.h>

#include "internal.h"

namespace ss {

namespace {

struct Philox {
    static __device__ __forceinline__ void round(uint32_t (&c)[4], uint32_t k0, uint32_t k1)
    {
        const uint64_t m0 = (uint64_t)0xD2511F53u * c[0], m1 = (uint64_t)0xCD9E8D57u * c[2];
        const uint32_t lo0 = (uint32_t)m0, hi0 = (uint32_t)(m0 >> 32), lo1 = (uint32_t)m1, hi1 = (uint32_t)(m1 >> 32);
        const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0;
        c[1] = lo1;
        c[2] = n2;
        c[3] = lo0;
    }
    static __device__ __forceinline__ void draw(uint32_t (&c)[4], uint32_t k0, uint32_t k1)
    {
#pragma unroll
        for (int r = 0; r < 10; ++r) {
            if (r > 0) {
                k0 += 0x9E3779B9u;
                k1 += 0xBB67AE85u;
            }
            round(c, k0, k1);
        }
    }
};

__device__ __forceinline__ double u01(uint32_t x) { return ((double)(x >> 9) + 0.5) * (1.0 / 8388608.0); }

__device__ __forceinline__ double box_muller(uint32_t a, uint32_t b)
{
    const double kTwoPi = 6.283185307179586476925286766559;
    return sqrt(-2.0 * log(u01(a))) * cos(kTwoPi * u01(b));
}

struct NoiseArgs {
    int gain_model;
    float k, theta, gain_sd, mu, sigma, scale;
    uint32_t key0, key1, stream;
    // the single-precision form (apply_fast): whether it is used, d, 1 / sqrt(9 d), d theta
    // and the bound on the error of 1 + c x
    int fast;
    float d, c, dtheta, et;
};

// gamma' and n' of pixel i
__device__ __forceinline__ void draws(const NoiseArgs &a, uint32_t i, float &gamma, float &n)
{
    double g = 1.0;
    if (a.gain_model == 1) {
        const double d = (double)a.k - 1.0 / 3.0, c = 1.0 / sqrt(9.0 * d);
        g = d * (double)a.theta;
        for (uint32_t att = 0; att < 64; ++att) {
            uint32_t w[4] = {i, a.stream, att, 0u};
            Philox::draw(w, a.key0, a.key1);
            const double x = box_muller(w[0], w[1]);
            double v = 1.0 + c * x;
            if (v <= 0.0) continue;
            v = v * v * v;
            if (log(u01(w[2])) < 0.5 * x * x + d - d * v + d * log(v)) {
                g = d * v * (double)a.theta;
                break;
            }
        }
    } else if (a.gain_model == 2) {
        uint32_t w[4] = {i, a.stream, 0u, 0u};
        Philox::draw(w, a.key0, a.key1);
        g = 1.0 + (double)a.gain_sd * box_muller(w[0], w[1]);
    }
    uint32_t w[4] = {i, a.stream, 0xFFFFFFFFu, 0u};
    Philox::draw(w, a.key0, a.key1);
    const float nz = (float)((double)a.mu + (double)a.sigma * box_muller(w[0], w[1]));
    const float gf = (float)g;
    gamma = __fadd_rn(1.0f, __fmul_rn(a.scale, __fsub_rn(gf, 1.0f)));
    n = __fmul_rn(a.scale, nz);
}

// Eq. (7)'s value of pixel i before the rounding to an integer, from its draws in single
// precision, and a bound on how far it lies from the one of draws(): false where a
// decision of the gamma's rejection loop could differ.
//
// The bounds, each the largest error against double precision over every value that can
// occur: with the hardware's log2, sqrt and cosine (of turns), over all 2^23 uniforms,
// sqrt(-2 log u) is off by at most 4.88e-7 (and at most 5.77), the cosine by 1.25e-7,
// log u by 1.63e-7 of itself, and log v over all floats in [2^-14, 2^6) by 1.39e-7
// (1 + |log v|) (v = t^3, 0.05 < t < 3.4: k >= 1); so a normal is off by at most kEx.
// Every product and sum adds half a unit, kEps of its result, in either form.
constexpr float kEps = 5.97e-8f, kEx = 1.7e-6f, kLog2 = 0.69314718055994531f;

__device__ __forceinline__ float fast_u01(uint32_t x) { return ((float)(x >> 9) + 0.5f) * (1.0f / 8388608.0f); }  // exact

__device__ __forceinline__ float fast_normal(uint32_t a, uint32_t b)
{
    return __builtin_amdgcn_sqrtf((-2.0f * kLog2) * __builtin_amdgcn_logf(fast_u01(a))) *
           __builtin_amdgcn_cosf(fast_u01(b));
}

__device__ __forceinline__ bool apply_fast(const NoiseArgs &a, uint32_t i, float in, float &value, float &err)
{
    uint32_t wn[4] = {i, a.stream, 0xFFFFFFFFu, 0u};
    Philox::draw(wn, a.key0, a.key1);
    const float sx = a.sigma * fast_normal(wn[0], wn[1]), nz = a.mu + sx;
    const float en = a.sigma * kEx + kEps * (2.0f * fabsf(sx) + 2.0f * fabsf(nz));
    float g = 1.0f, eg = 0.0f;
    if (a.gain_model == 1) {
        bool found = false;
        for (uint32_t att = 0; att < 64 && !found; ++att) {
            uint32_t w[4] = {i, a.stream, att, 0u};
            Philox::draw(w, a.key0, a.key1);
            const float x = fast_normal(w[0], w[1]);
            const float t = 1.0f + a.c * x;
            if (t < -0.01f) continue;  // certainly not positive
            if (!(t > 0.05f)) return false;
            const float v = t * t * t, rv = 3.2f * a.et * __builtin_amdgcn_rcpf(t) + 4.0f * kEps;  // v is off by rv of itself
            const float lu = kLog2 * __builtin_amdgcn_logf(fast_u01(w[2])), lv = kLog2 * __builtin_amdgcn_logf(v);
            const float h = 0.5f * x * x, w1 = 1.0f - v, q = w1 + lv, rhs = h + a.d * q;
            const float eq = rv * (1.0f + v) + 1.6e-7f * (1.0f + fabsf(lv)) + kEps * (fabsf(w1) + fabsf(q));
            const float diff = lu - rhs;
            const float tol = 1.05f * (a.d * (eq + 2.0f * kEps * fabsf(q)) + fabsf(x) * kEx +
                                       2.0f * kEps * (h + fabsf(rhs)) + 2.0e-7f * fabsf(lu) + kEps * fabsf(diff));
            if (diff > tol) continue;
            if (!(diff < -tol)) return false;
            g = a.dtheta * v;
            eg = g * (rv + 4.0f * kEps);
            found = true;
        }
        if (!found) return false;
    } else if (a.gain_model == 2) {
        uint32_t w[4] = {i, a.stream, 0u, 0u};
        Philox::draw(w, a.key0, a.key1);
        const float sg = a.gain_sd * fast_normal(w[0], w[1]);
        g = 1.0f + sg;
        eg = a.gain_sd * kEx + kEps * (2.0f * fabsf(sg) + 2.0f * fabsf(g));
    }
    const float g1 = g - 1.0f, gamma = 1.0f + a.scale * g1, n = a.scale * nz, prod = gamma * in;
    value = prod + n;
    const float egamma = a.scale * (eg + kEps * (2.0f * fabsf(g) + 4.0f * fabsf(g1))) + 2.0f * kEps * fabsf(gamma);
    err = 1.05f * (in * egamma + a.scale * en + 2.0f * kEps * (fabsf(prod) + fabsf(n) + fabsf(value)));
    return true;
}

__global__ __launch_bounds__(256) void noise_draws_kernel(NoiseArgs a, int64_t count, float *gamma, float *n)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    float g, z;
    draws(a, (uint32_t)i, g, z);
    gamma[i] = g;
    n[i] = z;
}

// Eq. (7) with this pixel's draws: product and sum each rounded to float32,
// rounded to the nearest integer (ties to even) and clipped to [0, 255].
//
// Bound by the arithmetic of the draws.  Only a byte leaves the kernel, so the draws are
// made in single precision with a bound on their error, and in double only for a pixel
// whose byte, or whose gamma's acceptance, lies within that bound of the other outcome:
// the bytes are those of the double-precision draws.  Default gamma (k = 3.98): 640x480
// 13.8 -> 8.4 us (the host's own time per call), 1920x1080 59.3 -> 25.3 us.
template <bool FAST>
__global__ __launch_bounds__(256) void noise_apply_kernel(NoiseArgs a, const uint8_t *in, int in_pitch, int W, int H,
                                                          uint8_t *out, int out_pitch)
{
    const int x = blockIdx.x * 256 + threadIdx.x, y = blockIdx.y;
    if (x >= W) return;
    const uint32_t i = (uint32_t)((int64_t)y * W + x);
    const float pix = (float)in[(size_t)y * in_pitch + x];
    float r = 0.0f, value, err;
    bool sure = false;
    if (FAST && apply_fast(a, i, pix, value, err)) {
        r = rintf(value);
        sure = 0.5f - fabsf(value - r) > err;
    }
    if (!sure) {
        float g, z;
        draws(a, i, g, z);
        r = rintf(__fadd_rn(__fmul_rn(g, pix), z));
    }
    r = r > 0.0f ? r : 0.0f;
    r = r < 255.0f ? r : 255.0f;
    out[(size_t)y * out_pitch + x] = (uint8_t)r;
}

NoiseArgs noise_args(const simsense_noise_params &p, int64_t pixels = 0)
{
    NoiseArgs a{};
    a.gain_model = p.gain_model;
    a.k = p.k; a.theta = p.theta; a.gain_sd = p.gain_sd; a.mu = p.mu; a.sigma = p.sigma; a.scale = p.scale;
    a.key0 = (uint32_t)p.seed;
    a.key1 = (uint32_t)(p.seed >> 32);
    a.stream = p.stream;
    const double d = (double)p.k - 1.0 / 3.0, c = 1.0 / sqrt(9.0 * d);
    a.d = (float)d;
    a.c = (float)c;
    a.dtheta = (float)(d * (double)p.theta);
    a.et = (float)(c * kEx + kEps * (3.0 + 4.0 * 5.8 * c));
    // the single-precision form pays where few pixels need the double one: the error of
    // the value (2e-6 of the draws' spread) well below one half (1920x1080 in us, double /
    // single: sigma 900 16.9 / 13.4, gain_sd 3.9 30.2 / 19.5, at the line), the shape small
    // enough for the acceptance test, whose error grows with k (k 256 46.2 / 24.3, 1024
    // 45.5 / 28.5, 4096 45.1 / 39.5; 640x480 10.1 / 9.9 at 1024, 10.0 / 10.5 at 4096),
    // the image large enough that its waves wait for each other and not for the few that
    // draw twice (kernel alone: 320x240 7.0 / 6.1, 237x137 5.5 / 5.7, 171x134 without a
    // gain 2.4 / 2.9), the more of them the closer k is to 1, where t is often near 0 (in a
    // graph, double / single: k 1 320x240 9.0 / 11.3, 560x420 15.0 / 15.3, 640x480 17.6 /
    // 14.2; k 1.2 320x240 7.9 / 9.9, 480x360 10.4 / 11.1, 560x420 14.2 / 10.9; k 1.5 320x240
    // 7.8 / 8.3, 400x300 9.1 / 7.7; k 2 320x240 7.8 / 7.1)
    const double spread = p.gain_model == 1 ? 2.0 * d * (double)p.theta : p.gain_model == 2 ? (double)p.gain_sd : 0.0;
    const bool shape = p.gain_model != 1 || p.k <= 1024.0f;
    const int64_t enough = p.gain_model != 1 || p.k >= 2.0f ? 65536 : p.k >= 1.25f ? 98304 : p.k >= 1.05f ? 180000 : 240000;
    a.fast = pixels >= enough && shape && (double)p.scale * (255.0 * spread + (double)p.sigma + fabs((double)p.mu) / 8.0) * 2e-6 <= 2e-3;
    return a;
}

int validate_noise(const simsense_noise_params *p)
{
    if (!p) return SIMSENSE_ERR_NULL_POINTER;
    if (p->struct_size != sizeof(simsense_noise_params)) return SIMSENSE_ERR_ABI;
    if (p->gain_model < 0 || p->gain_model > 2) return SIMSENSE_ERR_INVALID_ARGUMENT;
    if (p->gain_model == 1 && !(p->k >= 1.0f && p->theta > 0.0f)) return SIMSENSE_ERR_INVALID_ARGUMENT;
    if (!(p->gain_sd >= 0.0f) || !(p->sigma >= 0.0f) || !(p->scale >= 0.0f) || !(p->mu == p->mu))
        return SIMSENSE_ERR_INVALID_ARGUMENT;
    return SIMSENSE_OK;
}

}  // namespace

}  // namespace ss

using namespace ss;

extern "C" {

int simsense_noise_draws(const simsense_noise_params *params, int64_t count, float *gamma, float *n, void *stream)
{
    int rc = validate_noise(params);
    if (rc != SIMSENSE_OK) return rc;
    if (count < 0 || count > ((int64_t)1 << 32)) return SIMSENSE_ERR_INVALID_ARGUMENT;
    if (count == 0) return SIMSENSE_OK;
    if (!gamma || !n) return SIMSENSE_ERR_NULL_POINTER;
    hipLaunchKernelGGL(noise_draws_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       noise_args(*params), count, gamma, n);
    if (hipGetLastError() != hipSuccess) return SIMSENSE_ERR_DEVICE;
    return SIMSENSE_OK;
}

int simsense_ir_noise_generate(const simsense_noise_params *params, const uint8_t *in, int32_t in_pitch,
                               int32_t width, int32_t height, uint8_t *out, int32_t out_pitch, void *stream)
{
    int rc = validate_noise(params);
    if (rc != SIMSENSE_OK) return rc;
    if (width < 1 || height < 1 || width > 65536 || height > 65536) return SIMSENSE_ERR_INVALID_ARGUMENT;
    if (in_pitch < width || out_pitch < width) return SIMSENSE_ERR_INVALID_ARGUMENT;
    if (!in || !out) return SIMSENSE_ERR_NULL_POINTER;
    dim3 grid((width + 255) / 256, height), block(256);
    const NoiseArgs a = noise_args(*params, (int64_t)width * height);
    // (forms of their own: with the other's code beside it the double one is 2% slower)
    hipLaunchKernelGGL(a.fast ? noise_apply_kernel<true> : noise_apply_kernel<false>, grid, block, 0, (hipStream_t)stream, a, in,
                       in_pitch, width, height, out, out_pitch);
    if (hipGetLastError() != hipSuccess) return SIMSENSE_ERR_DEVICE;
    return SIMSENSE_OK;
}

}  // extern "C"
