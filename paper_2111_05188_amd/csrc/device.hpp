// Device helpers for gfx950: Philox4x32-10, Box-Muller, bf16 rounding,
// 64-lane wavefront reductions and scans.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tpk {

constexpr int WAVE = 64;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).  Ten rounds; each round
// multiplies counter words 0 and 2 by the two Philox multipliers, and the new
// counter is (hi(M1*c2)^c1^k0, lo(M1*c2), hi(M0*c0)^c3^k1, lo(M0*c0)).  The
// key is bumped by the two Weyl increments before every round but the first.
// ---------------------------------------------------------------------------
struct U4 {
    uint32_t x, y, z, w;
};

__device__ __forceinline__ U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1)
{
    constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
    constexpr uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += W0;
            k1 += W1;
        }
        const uint32_t hi0 = __umulhi(M0, c.x), lo0 = M0 * c.x;
        const uint32_t hi1 = __umulhi(M1, c.z), lo1 = M1 * c.z;
        c = U4{hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0};
    }
    return c;
}

// Top 23 bits, centred in their cell: exact in fp32, strictly inside (0,1).
__device__ __forceinline__ float uniform_open01(uint32_t w)
{
    return ((float)(w >> 9) + 0.5f) * (1.0f / 8388608.0f);
}

// log(u) for uniform_open01's u.  u = 2^k m, m in [sqrt(1/2), sqrt(2)), f = m - 1:
// k ln 2 + f + f^2 Q(f), Q fitted to log(1 + f) for the least relative error
// (2^-27 before rounding); ln 2 in two parts, the first short enough that its
// product with k is exact.  Within 0.91 ulp and without bias (mean error 6e-10
// of the value), where the library's logf is 2.6e-8 too small on average: that
// bias adds up in a log-density over many stocks.
__device__ __forceinline__ float log_open01(float u)
{
    float m = __builtin_amdgcn_frexp_mantf(u);   // [1/2, 1)
    int k = __builtin_amdgcn_frexp_expf(u);
    const bool low = m < 0.707106781f;
    m = low ? 2.0f * m : m;
    const float kf = (float)(low ? k - 1 : k), f = m - 1.0f;
    float q = -0x1.383c86p-4f;
    q = fmaf(q, f, 0x1.084d76p-3f);
    q = fmaf(q, f, -0x1.0f3750p-3f);
    q = fmaf(q, f, 0x1.2270b4p-3f);
    q = fmaf(q, f, -0x1.542750p-3f);
    q = fmaf(q, f, 0x1.99a400p-3f);
    q = fmaf(q, f, -0x1.000428p-2f);
    q = fmaf(q, f, 0x1.555550p-2f);
    q = fmaf(q, f, -0x1.fffff8p-2f);
    const float hi = kf * 0x1.62e4p-1f, a = hi + f, al = f - (a - hi);
    return a + fmaf(kf, 0x1.7f7d1cp-20f, fmaf(f * f, q, al));
}

// Box & Muller (1958): two independent N(0,1) draws from two uniforms.  The
// angle is taken in half turns: exact, where a product with 2 pi would round.
// Errors against 64 bits (2-norm, relative), with logf and the sine and cosine
// of the rounded product -> so: the draws 1.43e-7 -> 4.4e-8, a log-density
// of 5, 30, 100 stocks 5.7e-8, 3.1e-8, 2.9e-8 -> 4.4e-8, 2.8e-8, 2.5e-8
// (with logf and half turns 5.2e-8, 3.5e-8, 3.2e-8: the rounded product's
// bias had hidden logf's).
__device__ __forceinline__ void box_muller(float u0, float u1, float &z0,
                                           float &z1)
{
    const float rad = sqrtf(-2.0f * log_open01(u0));
    float s, c;
    sincospif(2.0f * u1, &s, &c);
    z0 = rad * c;
    z1 = rad * s;
}

// The same with the hardware transcendentals: v_log_f32 (log2), v_sqrt_f32,
// and v_sin_f32 / v_cos_f32, whose argument is in revolutions, so the
// uniform u1 is the angle / 2 pi as it stands.  Close to fp32 precision, not
// correctly rounded: used where the draws feed a bf16 actor, whose
// tolerance is far wider.
__device__ __forceinline__ void box_muller_hw(float u0, float u1, float &z0, float &z1)
{
    // -2 ln u0 = -2 ln(2) log2(u0)
    const float rad = __builtin_amdgcn_sqrtf(-1.38629436111989061f * __builtin_amdgcn_logf(u0));
    z0 = rad * __builtin_amdgcn_cosf(u1);
    z1 = rad * __builtin_amdgcn_sinf(u1);
}

// ---------------------------------------------------------------------------
// Wavefront collectives (all 64 lanes active), built on DPP lane moves:
// row_shr:k shifts within 16-lane rows, row_bcast:15 / row_bcast:31 carry
// row totals into the following rows.  A lane whose DPP source does not
// exist (or whose row is masked off) receives 0.
// ---------------------------------------------------------------------------
enum : int { DPP_ROW_SHR = 0x110, DPP_ROW_BCAST15 = 0x142, DPP_ROW_BCAST31 = 0x143 };

template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ double dpp_f64(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROWS, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Inclusive prefix sum across the 64 lanes in lane order (Hillis-Steele in
// rows of 16, then row totals carried forward).
__device__ __forceinline__ double wave_inclusive_scan(double v)
{
    v += dpp_f64<DPP_ROW_SHR + 1>(v);
    v += dpp_f64<DPP_ROW_SHR + 2>(v);
    v += dpp_f64<DPP_ROW_SHR + 4>(v);
    v += dpp_f64<DPP_ROW_SHR + 8>(v);
    v += dpp_f64<DPP_ROW_BCAST15, 0xA>(v);
    v += dpp_f64<DPP_ROW_BCAST31, 0xC>(v);
    return v;
}

__device__ __forceinline__ double lane_value(double v, int lane)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ int lane_value(int v, int lane)
{
    return __builtin_amdgcn_readlane(v, lane);
}

__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Orders this wave's LDS writes before the reads that other lanes of it make
// after (and its reads before the next writes).  One wave's LDS operations
// complete in order, so it costs no instruction: it keeps the compiler from
// moving them over one another.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum over the 64 lanes (same value returned to every lane).
__device__ __forceinline__ double wave_sum(double v)
{
    return lane_value(wave_inclusive_scan(v), WAVE - 1);
}

// fp32 -> bf16, IEEE round to nearest even (v_cvt_pk_bf16_f32 on gfx950).
__device__ __forceinline__ __bf16 to_bf16(float x) { return (__bf16)x; }

// tanh(x) = 2 / (1 + exp(-2x)) - 1 with the hardware exp2 and reciprocal;
// the argument comes in as e2 = -2 log2(e) x (one fma with a pre-scaled
// bias).  Absolute error of a few 1e-7 (cancellation near 0 leaves the fp32
// rounding of 1), far below the bf16 rounding the result goes through.
constexpr float NEG_2LOG2E = -2.8853900817779268f;

__device__ __forceinline__ float tanh_from_e2(float e2)
{
    return fmaf(2.0f, __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(e2)), -1.0f);
}

// tanh of |x| < 1: x + x^3 P(x^2), P fitted to tanh for the least relative error
// (2^-27 before rounding), odd in x and exact at 0.
__device__ __forceinline__ float tanh_below_1(float ax)
{
    const float u = ax * ax;
    float p = -0x1.77dca8p-12f;
    p = fmaf(p, u, 0x1.2da4bap-9f);
    p = fmaf(p, u, -0x1.0460b0p-7f);
    p = fmaf(p, u, 0x1.60098cp-6f);
    p = fmaf(p, u, -0x1.b96222p-5f);
    p = fmaf(p, u, 0x1.110be2p-3f);
    p = fmaf(p, u, -0x1.55553cp-2f);
    return fmaf(ax * u, p, ax);
}

// tanh to fp32 precision without a branch (NaN stays NaN, -0 stays -0).  From
// 1 on 1 - 2 / (e + 1), e = exp(2 |x|): elo carries the rounding of the
// exponent's argument, dlo also that of e + 1, and one Newton step brings them
// into the quotient; past 10 tanh is 1 in fp32.  Over every fp32 value the
// error is at most 0.98 ulp, and no larger than the library tanhf's (1.41) in
// any binade.  SKIP: a wave whose arguments are all below 1 takes the
// polynomial alone (a year of values of the 30-stock daily workload, fp32
// critic of 256: 741 us without, 717 with it; the rollout's layers, where
// several tiles interleave, are faster without).
template <bool SKIP = false>
__device__ __forceinline__ float tanh_f32(float x)
{
    constexpr double LOG2E2 = 2.88539008177792681472;   // 2 log2(e)
    constexpr float HI = (float)LOG2E2, LO = (float)(LOG2E2 - (double)HI);
    const float ax = fabsf(x), small = tanh_below_1(ax);
    if (SKIP && __ballot(!(ax < 1.0f)) == 0) return copysignf(small, x);
    const float y = ax > 10.0f ? 10.0f : ax, yh = y * HI;
    const float yl = fmaf(y, LO, fmaf(y, HI, -yh));
    const float e = __builtin_amdgcn_exp2f(yh), elo = e * (yl * 0.693147181f);
    const float d = e + 1.0f, dlo = (1.0f - (d - e)) + elo;
    const float r = __builtin_amdgcn_rcpf(d);
    const float q = fmaf(fmaf(-dlo, r, fmaf(-d, r, 1.0f)), r, r);
    const float large = fmaf(-2.0f, q, 1.0f);
    return copysignf(ax < 1.0f ? small : large, x);
}

// The same for a result that is rounded to bf16 next, without the corrections
// from 1 on: at most 1.35 ulp of fp32 (still below tanhf's 1.41), 2e-5 of a
// bf16 ulp.
template <bool SKIP = false>
__device__ __forceinline__ float tanh_for_bf16(float x)
{
    const float ax = fabsf(x), small = tanh_below_1(ax);
    if (SKIP && __ballot(!(ax < 1.0f)) == 0) return copysignf(small, x);
    const float e = __builtin_amdgcn_exp2f(-NEG_2LOG2E * ax);
    const float large = fmaf(-2.0f, __builtin_amdgcn_rcpf(e + 1.0f), 1.0f);
    return copysignf(ax < 1.0f ? small : large, x);
}

}  // namespace tpk
