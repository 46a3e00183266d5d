// hmc_device.hpp -- device-side building blocks shared by the HMC kernels.
//
// Counter-based random numbers (Philox4x32-10, Salmon et al., SC'11), the
// uniform and normal maps of the ABI (include/hmc.h), wavefront reductions,
// and the per-chain accept / dual-averaging step.  gfx950 only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hmc {

// ---------------------------------------------------------------------------
// Philox4x32-10: ten rounds of two 32x32->64 multiplies; round multipliers
// and Weyl key increments from the SC'11 paper (Sec. 3.2, Table 2).
// ---------------------------------------------------------------------------
struct Key {
    uint32_t k0, k1;
};

__host__ __device__ inline Key make_key(uint64_t seed) {
    return Key{(uint32_t)(seed & 0xffffffffu), (uint32_t)(seed >> 32)};
}

__device__ __forceinline__ uint4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, Key key) {
    uint32_t k0 = key.k0, k1 = key.k1;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // each 32 x 32 -> 64-bit product as one v_mad_u64_u32 (instead of a
        // separate low and high multiply, both quarter-rate)
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
        const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        // three-way xor in one instruction (the compiler pairs the uniform key with
        // the other terms and takes two)
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32(hi1, c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32(hi0, c3, k1, 0x96);
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return make_uint4(c0, c1, c2, c3);
}

enum : uint32_t { TAG_MOMENTUM = 0, TAG_ACCEPT = 1, TAG_SWAP = 2 };

// (k + 1/2) 2^-23 with k the top 23 bits: exact in binary32 and binary64.
__device__ __forceinline__ float u23_f32(uint32_t w) {
    return fmaf((float)(w >> 9), 0x1p-23f, 0x1p-24f);
}
__device__ __forceinline__ double u23_f64(uint32_t w) {
    return ((double)(w >> 9) + 0.5) * 0x1p-23;
}

// Box-Muller on one pair: r = sqrt(-2 log u1), angle = 2 pi u2 (sincospi of 2 u2,
// exact argument).  Runs of many chains are bound by the vector instructions of
// their draws, so the FP32 logarithm and root leave out what u in [2^-24, 1 -
// 2^-24] cannot need (subnormals, scaling, infinities): log u is log2 u times ln 2
// in two parts (Cody and Waite 1980) with the first product's rounding recovered by an
// FMA (Dekker 1971), the root one Newton step from 1 / sqrt with its residual by an
// FMA (Markstein 1990).  For each of the 2^23 values of u both are bit for bit logf
// and the correctly rounded sqrtf as this compiler builds them (all are compared in
// tests/device_check.hip).  16384 chains of diagonal D = 1000 FP32, 20 transitions:
// 910 -> 750 us together with log_uniform52_below.
__device__ __forceinline__ float sqrt_m2log(float u) {
    const float y = __builtin_amdgcn_logf(u);               // log2
    const float hi = 0x1.62e42ep-1f, lo = 0x1.efa39ep-25f;  // ln 2 = hi + lo
    const float p = y * hi;
    const float x = -2.0f * fmaf(y, hi, fmaf(y, lo, fmaf(y, hi, -p)));
    const float r = __builtin_amdgcn_rsqf(x), g = x * r;
    return fmaf(fmaf(-g, g, x), 0.5f * r, g);
}
__device__ __forceinline__ void box_muller(uint32_t wa, uint32_t wb, float& z0, float& z1) {
    const float r = sqrt_m2log(u23_f32(wa));
    const float a = fmaf((float)(wb >> 9), 0x1p-22f, 0x1p-23f), h = 0.5f * a;
    // facts that shorten the reduction of sincospif's argument
    __builtin_assume(a > 0.0f && a < 2.0f);
    __builtin_assume(__builtin_isfinite(a) && __builtin_isfinite(h));
    float s, c;
    sincospif(a, &s, &c);
    z0 = r * c;
    z1 = r * s;
}
__device__ __forceinline__ void box_muller(uint32_t wa, uint32_t wb, double& z0, double& z1) {
    const double u = u23_f64(wa), a = 2.0 * u23_f64(wb), h = 0.5 * a;
    __builtin_assume(u > 0.0 && u < 1.0 && a > 0.0 && a < 2.0);
    __builtin_assume(__builtin_isfinite(u) && __builtin_isfinite(a) && __builtin_isfinite(h));
    const double r2 = -2.0 * log(u);
    __builtin_assume(r2 > 0.0 && __builtin_isfinite(r2));
    const double r = sqrt(r2);
    double s, c;
    sincospi(a, &s, &c);
    z0 = r * c;
    z1 = r * s;
}

// Four momenta of chain c at transition t for dimensions 4*block .. 4*block+3.
// need_hi = false when dimensions 4*block+2 and +3 lie beyond D: the second
// Box-Muller pair is then not evaluated (its values would be discarded; the
// first pair does not depend on it) and z[2], z[3] are set to 0.
template <typename T>
__device__ __forceinline__ void momentum4(Key key, uint32_t chain, uint32_t t, uint32_t block, T z[4],
                                          bool need_hi = true) {
    const uint4 w = philox(chain, t, block, TAG_MOMENTUM, key);
    box_muller(w.x, w.y, z[0], z[1]);
    if (need_hi) {
        asm volatile("" ::: );   // keeps the pair behind the branch (not computed and selected)
        box_muller(w.z, w.w, z[2], z[3]);
    } else {
        z[2] = (T)0;
        z[3] = (T)0;
    }
}

// log of the uniform ((w0>>6) 2^26 + (w1>>6) + 1/2) 2^-52 of block
// (chain, t, 0, tag), in FP64: the Metropolis test (tag ACCEPT) and the
// replica-exchange test (tag SWAP).
__device__ __forceinline__ double log_uniform52(Key key, uint32_t chain, uint32_t t, uint32_t tag) {
    const uint4 w = philox(chain, t, 0u, tag, key);
    const double k = (double)(w.x >> 6) * 67108864.0 + (double)(w.y >> 6);
    return log((k + 0.5) * 0x1p-52);
}
__device__ __forceinline__ double log_accept_uniform(Key key, uint32_t chain, uint32_t t) {
    return log_uniform52(key, chain, t, TAG_ACCEPT);
}

// log_uniform52(key, chain, t, tag) < thr, the logarithm in FP64 only where it
// decides: the uniform lies below 1, so thr >= 0 holds without it, and FP32's
// log2 is within 2e-7 of log u relatively plus 6e-8 from rounding u, an order
// below the margin.  NaN compares false, as before.
__device__ __forceinline__ bool log_uniform52_below(Key key, uint32_t chain, uint32_t t, uint32_t tag, double thr) {
    if (thr >= 0.0) return true;
    const uint4 w = philox(chain, t, 0u, tag, key);
    const double k = (double)(w.x >> 6) * 67108864.0 + (double)(w.y >> 6);
    const double u = (k + 0.5) * 0x1p-52;
    const double la = (double)(__builtin_amdgcn_logf((float)u) * 0.693147180559945f);
    const double d = thr - la;
    if (fabs(d) > fma(-4e-6, la, 4e-6)) return d > 0.0;
    return log(u) < thr;
}
__device__ __forceinline__ bool accept_below(Key key, uint32_t chain, uint32_t t, double lar) {
    return log_uniform52_below(key, chain, t, TAG_ACCEPT, lar);
}

// ---------------------------------------------------------------------------
// Reductions across a power-of-two group of G lanes (G <= 64) of a wavefront.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// v of the lane and of lane ^ 32, added (v_permlane32_swap of a register with
// itself gives [lo, lo] and [hi, hi]).
__device__ __forceinline__ double xor32_sum(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    return __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])) +
           __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}
// Sum of rows 2k and 2k+1 (k = 0, 1), in both rows: lane and lane ^ 16.
__device__ __forceinline__ double rows2_sum(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    const double a = __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0]));
    const double b = __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
    return a + b;
}
// A butterfly over lane ^ G/2, .., lane ^ 1 in registers, where a step by
// ds_bpermute waits for the LDS: fused diagonal D = 333, 1000 chains, 320
// transitions 1128 -> 1054 us, logistic NUTS 1000 x 25 3415 -> 3228 us, bitwise the
// same.  After the step of 8 the values of lanes l and l ^ 8 of a 16-lane row are
// equal, so rotating the row by 4 meets the partner l ^ 4.
template <int G>
__device__ __forceinline__ double group_sum(double v) {
    if constexpr (G == 64) v = xor32_sum(v);
    if constexpr (G >= 32) v = rows2_sum(v);
    if constexpr (G >= 16) {
        v += dpp_f64<0x128>(v);                        // row_ror 8
        v += dpp_f64<0x124>(v);                        // row_ror 4
    } else if constexpr (G == 8) {
        v += __shfl_xor(v, 4, 64);
    }
    if constexpr (G >= 4) v += dpp_f64<0x4E>(v);       // quad_perm [2,3,0,1]
    if constexpr (G >= 2) v += dpp_f64<0xB1>(v);       // quad_perm [1,0,3,2]
    return v;
}

template <typename T>
__device__ __forceinline__ T as_state(float v);
template <>
__device__ __forceinline__ float as_state<float>(float v) { return v; }
template <>
__device__ __forceinline__ double as_state<double>(float v) { return (double)v; }

// BF16 <-> FP32 (round to nearest even; inputs finite).
__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
    return __uint_as_float(((uint32_t)b) << 16);
}
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// ---------------------------------------------------------------------------
// Per-chain decision (Metropolis-Hastings on dH) and dual averaging
// (Hoffman & Gelman 2014, eq. 6).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double log_accept_ratio_of(double dh) {
    // -dH, with NaN and +inf dH mapped to -inf (reject)
    return (isnan(dh) || (isinf(dh) && dh > 0.0)) ? -INFINITY : -dh;
}

struct DualAvg {
    double hbar, log_eps_bar, mu;
};

// The factors of iteration m that do not depend on the chain: the averaging
// weight 1/(m + t0), the shrinkage sqrt(m)/gamma and the iterate weight m^-kappa.
struct DaConst {
    double w, k, eta;
};
__device__ __forceinline__ DaConst dual_avg_const(double m, double gamma, double t0, double kappa) {
    return DaConst{1.0 / (m + t0), sqrt(m) / gamma, pow(m, -kappa)};
}

// Iteration with accept statistic alpha; returns the new log step size.
__device__ __forceinline__ double dual_avg_apply(DualAvg& s, const DaConst& c, double alpha, double delta) {
    s.hbar = (1.0 - c.w) * s.hbar + c.w * (delta - alpha);
    const double log_eps = s.mu - c.k * s.hbar;
    s.log_eps_bar = c.eta * log_eps + (1.0 - c.eta) * s.log_eps_bar;
    return log_eps;
}

// Multiplicative rule (SimpleStepSizeAdaptation example of the wrapper
// pattern): grow after a transition whose accept statistic is above the
// target, shrink otherwise.
__device__ __forceinline__ double simple_adapt(double eps, double alpha, double target, double rate) {
    return alpha > target ? eps * (1.0 + rate) : eps / (1.0 + rate);
}

// Iteration m >= 1 with accept statistic alpha; returns the new log step size.
__device__ __forceinline__ double dual_avg_update(DualAvg& s, double m, double alpha, double delta,
                                                  double gamma, double t0, double kappa) {
    return dual_avg_apply(s, dual_avg_const(m, gamma, t0, kappa), alpha, delta);
}

// Control block of the plain/graph path (device resident, written by a
// one-thread kernel so that a captured graph can be replayed unchanged).
struct Ctrl {
    uint64_t t;               // current transition index
    uint64_t t_begin;         // first transition of the current sample_chain call
    int64_t n_burnin;
    int64_t n_results;
    int32_t adapt;
    int32_t adapt_kind;       // HMC_ADAPT_DUAL_AVERAGING or HMC_ADAPT_SIMPLE
    double target_accept, gamma, t0, kappa, rate;
    void* samples;            // [R, C, D] state dtype or null
    double* tr_step;
    uint8_t* tr_acc;
    double* tr_lar;
    double* tr_logp;
    uint8_t* out_acc;         // hmc_step outputs ([C] / [C, D]) or null
    double* out_lar;
    double* out_logp;
    void* out_xprop;
    void* out_pprop;
    double* out_dh;
};

}  // namespace hmc
