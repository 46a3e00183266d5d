// device_check.hip -- the shortened forms of the draws (csrc/hmc_device.hpp) beside
// the functions they stand for, counted by tests/test_gpu_draws.py.
#include <math.h>

#include "../paper_2002_01184_amd/csrc/hmc_device.hpp"

namespace {

// thread i: u of the top 23 bits i; mismatches of u, of sqrt(-2 log u) and of the pair
// of normals for a second word that changes with i
__global__ void k_box_muller(uint32_t* bad) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x, w = i << 9, w2 = (i * 2654435761u) & ~0x1ffu;
    const float u = hmc::u23_f32(w), ref = sqrtf(-2.0f * logf(u));
    if (u != ((float)(w >> 9) + 0.5f) * 0x1p-23f) atomicAdd(bad, 1u);
    if (__float_as_uint(hmc::sqrt_m2log(u)) != __float_as_uint(ref)) atomicAdd(bad + 1, 1u);
    float z0, z1, s, c;
    hmc::box_muller(w, w2, z0, z1);
    sincospif(2.0f * (((float)(w2 >> 9) + 0.5f) * 0x1p-23f), &s, &c);
    if (__float_as_uint(z0) != __float_as_uint(ref * c) || __float_as_uint(z1) != __float_as_uint(ref * s))
        atomicAdd(bad + 2, 1u);
}

// thread i: the uniform of chain i against n thresholds: its logarithm plus off[j], and
// fixed[j]; mismatches with the comparison in FP64
__global__ void k_below(hmc::Key key, uint32_t t, const double* off, const double* fixed, int n, uint32_t* bad) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    const double lu = hmc::log_uniform52(key, i, t, hmc::TAG_ACCEPT);
    for (int j = 0; j < n; ++j) {
        const double thr = lu + off[j];
        if (hmc::accept_below(key, i, t, thr) != (lu < thr)) atomicAdd(bad, 1u);
        if (hmc::accept_below(key, i, t, fixed[j]) != (lu < fixed[j])) atomicAdd(bad + 1, 1u);
    }
}

}  // namespace

extern "C" int check_box_muller(uint32_t* bad) {
    hipLaunchKernelGGL(k_box_muller, dim3((1u << 23) / 256), dim3(256), 0, 0, bad);
    return (int)hipGetLastError();
}

// blocks of 256 chains
extern "C" int check_below(uint64_t seed, uint32_t t, const double* off, const double* fixed, int n, uint32_t blocks,
                           uint32_t* bad) {
    hipLaunchKernelGGL(k_below, dim3(blocks), dim3(256), 0, 0, hmc::make_key(seed), t, off, fixed, n, bad);
    return (int)hipGetLastError();
}
