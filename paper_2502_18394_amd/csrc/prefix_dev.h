// Device helpers shared by the Prefix-FFT cache kernels.
#pragma once
#include "common.h"
#include "prefix.h"

namespace spectre {

constexpr int kSweepBins = 128;   // bins of one head per workgroup of a pass over the half spectra

template <typename T>
__device__ __forceinline__ float load_scalar(const T *p, size_t i);
template <>
__device__ __forceinline__ float load_scalar<float>(const float *p, size_t i) { return p[i]; }
template <>
__device__ __forceinline__ float load_scalar<uint16_t>(const uint16_t *p, size_t i) {
    return __uint_as_float((uint32_t)p[i] << 16);
}

// (a b) mod N for a, b < N <= 2^17 without 64-bit division.
__device__ __forceinline__ unsigned mul_mod(unsigned a, unsigned b, int N) {
    if ((N & (N - 1)) == 0) return (a * b) & (unsigned)(N - 1);
    return (((a * (b >> 9)) % (unsigned)N) * 512u + a * (b & 511u)) % (unsigned)N;
}

// Ring rows of the tokens whose updates are pending, or of the tokens of one appended batch, as a kernel argument.
struct PendingSlots {
    int n;
    int slot[kMaxBatch];
};

// table index of bin k_start for a root index `mult` per bin, and its advance over 8 bins
__device__ __forceinline__ void index_walk(unsigned k_start, unsigned mult, int N, unsigned &m, unsigned &step) {
    if ((N & (N - 1)) == 0) {
        step = (8u * mult) & (unsigned)(N - 1);
        m = (k_start * mult) & (unsigned)(N - 1);
    } else {
        step = (unsigned)((8ull * mult) % (unsigned)N);
        m = (unsigned)(((unsigned long long)k_start * mult) % (unsigned)N);
    }
}

}  // namespace spectre
