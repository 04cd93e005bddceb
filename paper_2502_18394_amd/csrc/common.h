// Shared device helpers of the SPECTRE HIP kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace spectre {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// float2 + and - are HIP's own component-wise operators.
__host__ __device__ __forceinline__ float2 cmul(float2 a, float2 b) {   // a * b
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__host__ __device__ __forceinline__ float2 cmulc(float2 a, float2 b) {  // a * conj(b)
    return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
__host__ __device__ __forceinline__ float2 cconj(float2 a) { return make_float2(a.x, -a.y); }

// p + at bytes, p the same in every lane and at the lane's own: the address is formed from a scalar base, without a product.
template <typename T, typename At>
__device__ __forceinline__ T *lane_pointer(T *p, At at) {
    typedef typename std::conditional<std::is_const<T>::value, const char, char>::type byte_t;
    return reinterpret_cast<T *>(reinterpret_cast<byte_t *>(p) + at);
}

// Streaming accesses for data that is touched once per kernel (the cache rows of a decode sweep,
// the transform scratch): non-temporal loads and stores, which this GPU moves about 8 % faster
// than plain ones when both directions stream.
typedef float f32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 stream_load(const float4 *p) {
    const f32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void stream_store(float4 *p, float4 v) {
    const f32x4_t w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, reinterpret_cast<f32x4_t *>(p));
}
__device__ __forceinline__ float2 stream_load(const float2 *p) {
    const f32x2_t v = __builtin_nontemporal_load(reinterpret_cast<const f32x2_t *>(p));
    return make_float2(v.x, v.y);
}
__device__ __forceinline__ void stream_store(float2 *p, float2 v) {
    const f32x2_t w = {v.x, v.y};
    __builtin_nontemporal_store(w, reinterpret_cast<f32x2_t *>(p));
}

// Stores that go through the L2 at once.  What a kernel leaves dirty there, up to 4 MB on each of the eight XCDs, is written back
// when it ends and before the next one starts, with nothing beside it; written through, it leaves while the kernel still
// works.  For scratch the next kernel reads, of whole 128-byte lines per wave instruction, in launches that have memory to
// themselves (streaming stores instead cost 3 to 5 %, the next kernel reads the scratch).  Where the scratch is about what the
// L2s hold together, the next kernel finds it there after plain stores: each user's rule leaves that range out, with both sides measured.
constexpr size_t kL2Bytes = (size_t)32 << 20;
template <typename T>
__device__ __forceinline__ void through_store(T *p, T v) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "one or two words");
    if constexpr (sizeof(T) == 8)
        __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    else
        __hip_atomic_store(reinterpret_cast<unsigned int *>(p), __builtin_bit_cast(unsigned int, v), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
// The same for 16 bytes at byte `at` of the `bytes` from a base that is the same in every lane.
typedef unsigned int u32x4_store_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void through_store16(void *base, unsigned bytes, unsigned at, u32x4_store_t v) {
    constexpr int kRaw = 0x00027000, kDeviceScope = 16;              // 32-bit elements without a format; the sc1 bit
    __builtin_amdgcn_raw_buffer_store_b128(v, __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)bytes, kRaw), (int)at, 0, kDeviceScope);
}

// Two adjacent channels (2c, 2c+1) of one token row travel as one complex number
// (even channel = real part).  Storage types: float2 for fp32 rows, one 32-bit
// word holding two bfloat16 for bf16 rows.
// Loads of two elements from where callers only promise the alignment of one (the instruction is the same).
typedef float f32x2_elem_t __attribute__((ext_vector_type(2), aligned(4)));
typedef double f64x2_elem_t __attribute__((ext_vector_type(2), aligned(8)));
typedef uint32_t bf16x2_elem_t __attribute__((aligned(2)));
typedef float f32x4_elem_t __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t bf16x4_elem_t __attribute__((ext_vector_type(2), aligned(2)));

struct IoF32 {
    typedef float2 pair_t;
    static constexpr int kBytes = 4;
    __device__ static __forceinline__ float2 unpack(pair_t p) { return p; }
    __device__ static __forceinline__ pair_t pack(float2 v) { return v; }
    __device__ static __forceinline__ pair_t zero() { return make_float2(0.f, 0.f); }
    __device__ static __forceinline__ pair_t load_elements(const pair_t *p) {
        const f32x2_elem_t v = *reinterpret_cast<const f32x2_elem_t *>(p);
        return make_float2(v.x, v.y);
    }
    typedef f32x4_t quad_t;                                          // two adjacent pairs
    __device__ static __forceinline__ quad_t load_quad(const pair_t *p) { return *reinterpret_cast<const f32x4_elem_t *>(p); }
    __device__ static __forceinline__ float4 unpack_quad(quad_t q) { return make_float4(q.x, q.y, q.z, q.w); }
    __device__ static __forceinline__ pair_t load_stream(const pair_t *p) { return stream_load(p); }
    __device__ static __forceinline__ void store_stream(pair_t *p, pair_t v) { stream_store(p, v); }
};
struct IoBf16 {
    typedef uint32_t pair_t;
    static constexpr int kBytes = 2;
    __device__ static __forceinline__ float2 unpack(pair_t w) {
        return make_float2(__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u));
    }
    __device__ static __forceinline__ pair_t pack(float2 v) {   // round to nearest even
        f32x2_t f = {v.x, v.y};
        bf16x2_t b = __builtin_convertvector(f, bf16x2_t);
        return __builtin_bit_cast(uint32_t, b);
    }
    __device__ static __forceinline__ pair_t zero() { return 0u; }
    __device__ static __forceinline__ pair_t load_elements(const pair_t *p) { return *reinterpret_cast<const bf16x2_elem_t *>(p); }
    typedef uint32_t quad_t __attribute__((ext_vector_type(2)));
    __device__ static __forceinline__ quad_t load_quad(const pair_t *p) { return *reinterpret_cast<const bf16x4_elem_t *>(p); }
    __device__ static __forceinline__ float4 unpack_quad(quad_t q) {
        const float2 a = unpack(q.x), b = unpack(q.y);
        return make_float4(a.x, a.y, b.x, b.y);
    }
    __device__ static __forceinline__ pair_t load_stream(const pair_t *p) { return __builtin_nontemporal_load(p); }
    __device__ static __forceinline__ void store_stream(pair_t *p, pair_t v) { __builtin_nontemporal_store(v, p); }
};

}  // namespace spectre
