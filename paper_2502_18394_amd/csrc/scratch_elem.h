// Element of the transform scratch: one complex number per channel pair, as two fp32 (the default) or, on request
// for bf16 rows, as two bfloat16 in a 32-bit word (half the bytes of every exchange between the three kernels;
// the arithmetic stays fp32).
#pragma once
#include "common.h"

namespace spectre {

struct ScrF32 {
    typedef float2 elem_t;
    __device__ static __forceinline__ float2 get(elem_t e) { return e; }
    __device__ static __forceinline__ elem_t put(float2 v) { return v; }
};
// fp32 elements, and row factors of at most one product (SmallTwiddles): the windows with 1024-point columns, whose row
// transforms are four times as long as beside the 4096-point columns of the mixer's plan.
struct ScrF32Fine : ScrF32 {};
struct ScrBf16 {
    typedef uint32_t elem_t;
    __device__ static __forceinline__ float2 get(elem_t e) { return IoBf16::unpack(e); }
    __device__ static __forceinline__ elem_t put(float2 v) { return IoBf16::pack(v); }
};

// Head-affine placement (aff = heads in the launch, a multiple of 8; 0 = off).  Workgroup ids are dealt round-robin
// to the 8 XCDs, each with its own L2.  Here the per_head workgroups of head 8 * slot + xcd all get ids congruent to
// xcd mod 8, so a head's scratch is written and read through one L2, and the three kernels walk the slots in
// alternating order (row transforms up, column kernel down, inverse row transforms up), so that each starts with
// what its predecessor wrote last.  Pays when a few heads' scratch fits one 4 MB L2 (L <= 8192).
__device__ __forceinline__ void head_affine(int id, int per_head, int aff, bool reverse, int *bhl, int *within) {
    const int xcd = id & 7, idx = id >> 3;
    int slot = idx / per_head;
    *within = idx - slot * per_head;
    if (reverse) slot = aff / 8 - 1 - slot;
    *bhl = 8 * slot + xcd;
}

// exp(-j 2 pi t1 k2 / L) for k2 = 1 .. N2-1.  Only the powers of two are read from the table (five loads instead of
// 31 scattered ones at N2 = 32: the gathers were most of the kernel's cache-line requests).  With k2 = 4a + b the
// others are hi[a] * lo[b], products of at most five table values in all, i.e. within 4 rounding errors of the table
// value; only hi and lo stay in registers, the product is formed where it is used.
// FINE: hi and lo all come from the table (ten loads at N2 = 32), which takes the factors' error from 4.5e-8 to 3.3e-8.
template <int N2, bool FINE = false>
struct SmallTwiddles {
    float2 lo[4], hi[8];
    __device__ __forceinline__ SmallTwiddles(const float2 *__restrict__ twL, int t1) {
        if (FINE) {
#pragma unroll
            for (int b = 0; b < 4; ++b) lo[b] = (b && b < N2) ? *lane_pointer(twL, 8u * (t1 * b)) : make_float2(1.f, 0.f);
#pragma unroll
            for (int a = 0; a < 8; ++a) hi[a] = (a && 4 * a < N2) ? *lane_pointer(twL, 8u * (t1 * 4 * a)) : make_float2(1.f, 0.f);
            return;
        }
        float2 p[5];
#pragma unroll
        for (int e = 0; e < 5; ++e) p[e] = ((1 << e) < N2) ? *lane_pointer(twL, 8u * (t1 << e)) : make_float2(1.f, 0.f);
        lo[0] = make_float2(1.f, 0.f);
        lo[1] = p[0];
        lo[2] = p[1];
        lo[3] = cmul(p[1], p[0]);
        hi[0] = make_float2(1.f, 0.f);
        hi[1] = p[2];
        hi[2] = p[3];
        hi[3] = cmul(p[3], p[2]);
        hi[4] = p[4];
        hi[5] = cmul(p[4], p[2]);
        hi[6] = cmul(p[4], p[3]);
        hi[7] = cmul(p[4], hi[3]);
    }
    // Makes the factors opaque to the compiler: in a loop it would otherwise form all the products once and keep them in
    // registers.
    __device__ __forceinline__ void pin() {
#pragma unroll
        for (int a = 1; a < 8; ++a)
            if (4 * a < N2) asm volatile("" : "+v"(hi[a].x), "+v"(hi[a].y));
    }
    __device__ __forceinline__ float2 operator()(int k2) const {     // k2 a compile-time constant after unrolling
        const int a = k2 >> 2, b = k2 & 3;
        if (a == 0) return lo[b];
        if (b == 0) return hi[a];
        return cmul(hi[a], lo[b]);
    }
};

}  // namespace spectre
