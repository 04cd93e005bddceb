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

// The complex transform Z of z = v_even + j v_odd separates into the two real channels' half spectra,
// X_even[k] = (Z_k + conj Z_{N-k})/2, X_odd[k] = (Z_k - conj Z_{N-k})/(2j).
__device__ __forceinline__ float4 untangle_pair(float2 zk, float2 zn) {
    float4 o;
    o.x = 0.5f * (zk.x + zn.x);
    o.y = 0.5f * (zk.y - zn.y);
    o.z = 0.5f * (zk.y + zn.y);
    o.w = -0.5f * (zk.x - zn.x);
    return o;
}

// The inverse with the gate applied: Y_c[k] = g_k X_c[k] for k <= N/2 (real parts only at DC and Nyquist: `real`),
// Hermitian-extended, then Z_k = Y_even[k] + j Y_odd[k] and Z_{N-k} = conj(Y_even[k]) + j conj(Y_odd[k]), times s.
struct TangledPair {
    float2 k, n;
};
__device__ __forceinline__ TangledPair tangle_pair(float4 x, float2 gk, bool real, float s) {
    float2 ya = cmul(gk, make_float2(x.x, x.y)), yb = cmul(gk, make_float2(x.z, x.w));
    if (real) {
        ya.y = 0.f;
        yb.y = 0.f;
    }
    return {make_float2((ya.x - yb.y) * s, (ya.y + yb.x) * s), make_float2((ya.x + yb.y) * s, (yb.x - ya.y) * s)};
}

}  // namespace spectre
