// Largest errors of the float32 clock functions against the float64 ones, on the device
// (tests/test_gpu_clock_error.py).  out: one uint32 per kernel, float bits, zeroed by the caller.
#include <hip/hip_runtime.h>

#include "../paper_2609_21858_amd/csrc/psd_device.hpp"

namespace {

__device__ void max_into(uint32_t* out, double err) {
    float e = (float)err;
    for (int off = 32; off > 0; off >>= 1) e = fmaxf(e, __shfl_xor(e, off));
    if ((threadIdx.x & 63) == 0) atomicMax(out, __float_as_uint(e));  // (errors are not negative)
}

// -ln U of every uniform (a word's low 9 bits are not used), relative.
__global__ void exp1_error(uint32_t* out) {
    const uint32_t w = (blockIdx.x * blockDim.x + threadIdx.x) << 9;
    const double e = psd::exp1_f64(w);
    max_into(out, fabs((double)psd::exp1_f32(w) - e) / e);
}

// ln x of every float in [2^-44, 2^8), absolute.
__global__ void ln_error(uint32_t* out) {
    const uint32_t mantissa = blockIdx.x * blockDim.x + threadIdx.x;
    double err = 0.0;
    for (int ex = 127 - 44; ex < 127 + 8; ++ex) {
        const float x = __uint_as_float(((uint32_t)ex << 23) | mantissa);
        err = fmax(err, fabs((double)psd::ln_f32(x) - log((double)x)));
    }
    max_into(out, err);
}

// Tree clocks of one random (token, slot) per thread, relative.
__global__ void tree_error(uint32_t* out, uint32_t V, uint32_t seed) {
    const psd::Words w = psd::philox(blockIdx.x * blockDim.x + threadIdx.x, 0u, 0u, 7u, seed, V);
    const uint32_t v = w.w0 % V, slot = w.w1 % 32u;
    const double e = psd::tree_clock_f64(V, slot, v, w.w2, w.w3);
    max_into(out, fabs((double)psd::tree_clock_f32(V, slot, v, w.w2, w.w3) - e) / e);
}

}  // namespace

extern "C" {
int clock_error_exp1(uint32_t* out, hipStream_t s) {
    exp1_error<<<dim3(1 << 15), dim3(256), 0, s>>>(out);
    return (int)hipGetLastError();
}
int clock_error_ln(uint32_t* out, hipStream_t s) {
    ln_error<<<dim3(1 << 15), dim3(256), 0, s>>>(out);
    return (int)hipGetLastError();
}
int clock_error_tree(uint32_t* out, uint32_t V, uint32_t seed, hipStream_t s) {
    tree_error<<<dim3(1 << 14), dim3(256), 0, s>>>(out, V, seed);
    return (int)hipGetLastError();
}
}
