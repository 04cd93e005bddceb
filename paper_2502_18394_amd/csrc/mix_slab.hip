// Short-sequence path of the SPECTRE mixing layer (Sec. 3.2 steps 2-4, Eq. 3 and Eq. 4):
// one workgroup owns the whole [L, d = 64] slab of one head of one sequence in LDS.
//
// Serves every L <= 2048 whose prime factors are in {2, 3, 5, 7} - in particular the
// 14 x 14 = 196 patch grid of the ViT workload and the powers of two up to 2048.
// Channel pairs are transformed as complex sequences (see mix_pow2.hip).
// Lengths of compile-time radices take k_mix_ct, any other k_mix_slab.
// The transform is an in-place mixed-radix decimation-in-frequency FFT: after the last
// forward pass position p holds bin k = reverse(p) (mixed-radix digit reversal), the gate
// is applied in that order from a per-workgroup table, and the inverse passes undo the
// forward ones in reverse, so nothing is ever reordered.
#include "mix_slab.h"

#include <stdlib.h>

#include <vector>

#include "fft_regs.h"
#include "internal.h"

namespace spectre {

template <int R, bool INV>
__device__ __forceinline__ void dft_any(float2 (&x)[R]) {
    small_dft<R, INV>(x);
}

// One in-place pass over all 32 columns of the slab.  n = current sub-transform length,
// S = n / R its stride; roots[m] = exp(-j 2 pi m / L).  Forward: butterfly then twiddle (and
// the gate, when GATE, which makes this the last forward pass).  Inverse: conjugate twiddle then
// inverse butterfly.
// UNIT: n == R, every twiddle is 1 and is skipped.
template <int R, bool INV, bool GATE, bool UNIT, int PP>
__device__ __forceinline__ void slab_pass(float2 *__restrict__ slab, const float2 *__restrict__ roots,
                                          const float2 *__restrict__ gpos, int L, int n, int tid, int nthreads) {
    constexpr int kShift = (PP == 32) ? 5 : (PP == 16) ? 4 : (PP == 8) ? 3 : 2;
    static_assert(PP == 32 || PP == 16 || PP == 8 || PP == 4, "pairs per workgroup");
    const int S = n / R, tstep = L / n;
    const int nb = (L / R) * PP;
    // bi / S by a multiply and shift: exact while bi * S < 2^20 (bi < L/R <= 1024, S <= L/R)
    const unsigned inv_s = ((1u << 20) + (unsigned)S - 1) / (unsigned)S;
    for (int w = tid; w < nb; w += nthreads) {
        const int col = w & (PP - 1), bi = w >> kShift;
        const int blk = (int)(((unsigned)bi * inv_s) >> 20), i = bi - blk * S;
        const int base = blk * n + i;
        float2 x[R];
#pragma unroll
        for (int j = 0; j < R; ++j) x[j] = slab[(base + S * j) * PP + col];
        if (INV && !UNIT) {
#pragma unroll
            for (int u = 1; u < R; ++u) x[u] = cmulc(x[u], roots[i * u * tstep]);
        }
        dft_any<R, INV>(x);
        if (!INV) {
            if (!UNIT) {
#pragma unroll
                for (int u = 1; u < R; ++u) x[u] = cmul(x[u], roots[i * u * tstep]);
            }
            if (GATE) {
#pragma unroll
                for (int u = 0; u < R; ++u) x[u] = cmul(x[u], gpos[base + S * u]);
            }
        }
#pragma unroll
        for (int j = 0; j < R; ++j) slab[(base + S * j) * PP + col] = x[j];
    }
}

template <bool INV, bool GATE, bool UNIT, int PP>
__device__ __forceinline__ void slab_pass_dispatch(int R, float2 *slab, const float2 *roots, const float2 *gpos,
                                                   int L, int n, int tid, int nthreads) {
    switch (R) {
        case 2: slab_pass<2, INV, GATE, UNIT, PP>(slab, roots, gpos, L, n, tid, nthreads); break;
        case 3: slab_pass<3, INV, GATE, UNIT, PP>(slab, roots, gpos, L, n, tid, nthreads); break;
        case 4: slab_pass<4, INV, GATE, UNIT, PP>(slab, roots, gpos, L, n, tid, nthreads); break;
        case 5: slab_pass<5, INV, GATE, UNIT, PP>(slab, roots, gpos, L, n, tid, nthreads); break;
        case 6: slab_pass<6, INV, GATE, UNIT, PP>(slab, roots, gpos, L, n, tid, nthreads); break;
        case 7: slab_pass<7, INV, GATE, UNIT, PP>(slab, roots, gpos, L, n, tid, nthreads); break;
        case 8: slab_pass<8, INV, GATE, UNIT, PP>(slab, roots, gpos, L, n, tid, nthreads); break;
        case 10: slab_pass<10, INV, GATE, UNIT, PP>(slab, roots, gpos, L, n, tid, nthreads); break;
        case 12: slab_pass<12, INV, GATE, UNIT, PP>(slab, roots, gpos, L, n, tid, nthreads); break;
        case 14: slab_pass<14, INV, GATE, UNIT, PP>(slab, roots, gpos, L, n, tid, nthreads); break;
        case 16: slab_pass<16, INV, GATE, UNIT, PP>(slab, roots, gpos, L, n, tid, nthreads); break;
        default: break;
    }
}

struct SlabRadices {
    int count;
    int r[10];
};

// grid = B*H*(32/PP) workgroups of 256 lanes, PP channel pairs each: a whole head, half a head when rows
// are fp32 (still full 128-byte row segments, half the LDS, twice the workgroups per CU), or as little as
// 4 pairs when there are few heads (then the call is one launch over every compute unit instead of four
// dependent ones) or the sequence is long (the slab must fit in LDS).
// LDS: slab [L][PP] float2, roots [L], gpos [L].
template <typename IO, int PP, int NT = 256>
__global__ __launch_bounds__(NT) void k_mix_slab(const typename IO::pair_t *__restrict__ v,
                                                 const float2 *__restrict__ g,
                                                 typename IO::pair_t *__restrict__ out,
                                                 const float2 *__restrict__ roots_g,
                                                 const int *__restrict__ bin_of_pos, int L, int H,
                                                 SlabRadices rad, int rows) {
    extern __shared__ float2 lds_slab[];
    float2 *slab = lds_slab;
    float2 *roots = slab + (size_t)L * PP;
    float2 *gpos = roots + L;
    constexpr int kParts = 32 / PP, kRows = NT / PP;       // workgroups per head; rows covered per sweep
    static_assert(NT % PP == 0 && NT % 64 == 0, "whole rows per sweep, whole waves");
    const int tid = threadIdx.x;
    const int bh = blockIdx.x / kParts, part = blockIdx.x % kParts, b = bh / H, h = bh % H;
    const int F = L / 2 + 1;

    // rows l = tid/PP + kRows i.  Sixteen loads are put in flight before any is consumed (all 196 rows of
    // the ViT grid at once for fp32 half heads); the first batch flies while the gate table below is built.
    const int lp_in = tid & (PP - 1), row_in = tid / PP;
    // the tensors hold `rows` <= L rows per sequence; the transform sees them followed by zeros and only the first
    // `rows` rows of the result are kept (zero-padded linear convolution)
    const typename IO::pair_t *src = v + (((size_t)b * rows) * H + h) * 32 + part * PP + lp_in;
    const size_t rs = (size_t)H * 32;
    constexpr int kBatch = 16;
    typename IO::pair_t val[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
        const int l = row_in + kRows * i;
        val[i] = (l < rows) ? src[(size_t)l * rs] : IO::zero();
    }

    // roots of unity and the gate in position order (bin_of_pos[p] = the bin that position p holds after
    // the last forward pass); full-length Hermitian extension, 1/L folded in.  The two dependent loads
    // (bin, then gate) are issued for all of a lane's positions at once: L <= 2048 = 8 * 256.
    {
        constexpr int kPos = (kSlabMaxL + NT - 1) / NT;
        int kbin[kPos];
        float2 gv[kPos], rv[kPos];
#pragma unroll
        for (int i = 0; i < kPos; ++i) {
            const int p = tid + NT * i;
            kbin[i] = (p < L) ? bin_of_pos[p] : 0;
            rv[i] = (p < L) ? roots_g[p] : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int i = 0; i < kPos; ++i) {
            const int k = kbin[i];
            gv[i] = (tid + NT * i < L) ? g[(size_t)bh * F + (2 * k <= L ? k : L - k)] : make_float2(0.f, 0.f);
        }
        const float sc = 1.0f / (float)L;
#pragma unroll
        for (int i = 0; i < kPos; ++i) {
            const int p = tid + NT * i, k = kbin[i];
            if (p < L) {
                float2 val = gv[i];
                if (2 * k > L) val.y = -val.y;
                if (k == 0 || 2 * k == L) val.y = 0.f;
                roots[p] = rv[i];
                gpos[p] = make_float2(val.x * sc, val.y * sc);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
        const int l = row_in + kRows * i;
        if (l < L) slab[l * PP + lp_in] = IO::unpack(val[i]);
    }
    for (int l0 = row_in + kBatch * kRows; l0 < L; l0 += kBatch * kRows) {
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int l = l0 + kRows * i;
            val[i] = (l < rows) ? src[(size_t)l * rs] : IO::zero();
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int l = l0 + kRows * i;
            if (l < L) slab[l * PP + lp_in] = IO::unpack(val[i]);
        }
    }
    __syncthreads();
    int n = L;
    for (int q = 0; q < rad.count; ++q) {
        if (q == rad.count - 1) slab_pass_dispatch<false, true, true, PP>(rad.r[q], slab, roots, gpos, L, n, tid, NT);
        else slab_pass_dispatch<false, false, false, PP>(rad.r[q], slab, roots, gpos, L, n, tid, NT);
        n /= rad.r[q];
        __syncthreads();
    }
    for (int q = rad.count - 1; q >= 0; --q) {
        n *= rad.r[q];
        if (q == rad.count - 1) slab_pass_dispatch<true, false, true, PP>(rad.r[q], slab, roots, gpos, L, n, tid, NT);
        else slab_pass_dispatch<true, false, false, PP>(rad.r[q], slab, roots, gpos, L, n, tid, NT);
        __syncthreads();
    }
    {
        typename IO::pair_t *dst = out + (((size_t)b * rows) * H + h) * 32 + part * PP + lp_in;
        for (int l = row_in; l < rows; l += kRows) dst[(size_t)l * rs] = IO::pack(slab[l * PP + lp_in]);
    }
}

// ------------------------------------------------------------------------------------------
// Lengths L = R0 R1 (R2) whose radices are compile-time constants: the same transform with the row accesses inside its
// outermost pass and the two innermost passes, forward and inverse, in one.  Rows go from memory into the registers of the
// lane that transforms them and back, and a point crosses LDS two (three) times each way where the general kernel above
// moves it once more on both sides of every pass.
//   pass 0      : lane (i, pair), i < L / R0: rows i + (L / R0) j, j < R0 -> R0-point transform, times W_L^(i u)
//   (pass 1     : the same inside every block of R1 R2 positions)
//   inner pass  : the blocks of R = R1 (R2) positions: transform, gate, inverse transform, in registers
//   back        : mirror images
// Position p of the slab lies at p + p / R, so that lanes with neighbouring blocks meet different banks (not needed where a
// row of pairs spans them all).  After the forward passes value u of block blk (blk = u0, or u0 R1 + u1) holds bin
// u0 + R0 (u1 + R1 u).
// What bounds it is memory at the shortest lengths and the vector units (butterflies and LDS accesses) above.  Against the
// general structure with compile-time lengths, us: B=256 H=12 L=196 bf16 48.5 -> 40.8 (fp32, at 5.1 TB/s, 63.8 -> 61.6); 2048 heads of
// bf16 rows at 256 47 -> 33, at 512 152 -> 92; 64 heads of fp32 at 1024 25 -> 13; 32 heads at 2048 30 -> 13; kernel alone for
// one head of fp32 rows at 1024 10.1 -> 7.9, for 32 of bf16 at 512 9.4 -> 6.7.
// DIRECT (few workgroups, where the chain of latencies counts and registers do not): every lane loads its factors and its
// gate entries itself, beside its rows; otherwise both are tables in LDS, built while the rows are under way.
template <int R0, int R1, int R2>
struct SlabPlan {
    static constexpr int L = R0 * R1 * R2, R = R2 > 1 ? R2 : R1, blocks = L / R;
    static constexpr int S0 = L / R0, S1 = R2;
    __device__ static constexpr int bin(int blk, int u) {
        return R2 > 1 ? blk / R1 + R0 * (blk % R1 + R1 * u) : blk + R0 * u;
    }
    static constexpr size_t lds(int PP, bool direct) {
        return ((size_t)(L + (PP < 16 ? blocks : 0)) * PP + (direct ? 0 : 2 * (size_t)L)) * sizeof(float2);
    }
};

// STREAM: the rows pass the caches by.
// HALF: the tensors hold `rows` <= L / 2 rows per sequence; the transform sees zeros behind them and only the first `rows` rows
// of the result are kept (zero-padded linear convolution).  Otherwise rows = L.
// Global addresses are one uniform base per row, table or head and one offset of the lane.  As 64-bit products per lane
// and row, with a test each, they were a fifth of the vector unit's time (a 64-bit multiply-add takes four slots), and the tests put
// a branch around every load.  us, before / now: 768 heads of bf16 rows at 512 47 / 38, at 576 55 / 48, at 1024 115 / 101, of fp32 rows at
// 784 95 / 82; B=256 H=12 L=196 fp32 62.0 / 56.5, bf16 41.2 / 36.0; the padded 197 of 768 heads 44.5 / 41.1 with its gate; one head of 1024 fp32 7.1 / 6.6.
// WIDE: 64 bits for the lane's offset, where hundreds of thousands of heads make S0 rows 2^32 bytes (at 32 heads 1 to 4 % slower).
template <typename IO, int PP, int NT, int R0, int R1, int R2, bool DIRECT, bool STREAM, bool HALF, bool WIDE>
__global__ __launch_bounds__(NT) void k_mix_ct(const typename IO::pair_t *v, const float2 *g,
                                               typename IO::pair_t *out, const float2 *roots_g,
                                               int H, int bh0, int BH, int rows, int affine) {
    typedef SlabPlan<R0, R1, R2> Plan;
    constexpr int L = Plan::L, R = Plan::R, F = L / 2 + 1, S0 = Plan::S0, PAD = PP < 16 ? 1 : 0, kParts = 32 / PP;
    constexpr int kSlab = (L + PAD * Plan::blocks) * PP;
    constexpr int kInner = (Plan::blocks * PP + NT - 1) / NT;        // blocks of the inner pass per lane
    static_assert(S0 * PP <= NT && NT % 64 == 0, "one transform of the outermost pass per lane");
    extern __shared__ float2 lds_ct[];
    float2 *slab = lds_ct, *roots = slab + kSlab, *gpos = roots + L;
    const int tid = threadIdx.x, col = tid % PP, i0 = tid / PP;
    int bh = bh0 + blockIdx.x / kParts, part = blockIdx.x % kParts;
    if (affine) {                                                    // the parts of a head on one XCD: ids 8 apart
        const int idx = blockIdx.x >> 3;
        part = idx % kParts;
        bh = bh0 + (idx / kParts) * 8 + (blockIdx.x & 7);
        if (bh >= BH) return;                                        // whole workgroup: heads are padded to 8
    }
    const int b = bh / H, h = bh % H;
    auto at = [&](int p) { return slab + (p + PAD * (p / R)) * PP + col; };
    const bool live = S0 * PP == NT || i0 < S0;
    typedef typename IO::pair_t pair_t;
    constexpr int kIn = HALF ? (R0 + 1) / 2 : R0;                    // the lane's rows i0 + S0 j that exist
    const int n_rows = HALF ? rows : L;
    const size_t base = ((size_t)b * n_rows * H + h) * 32 + part * PP;
    typedef typename std::conditional<WIDE, size_t, unsigned>::type at_t;
    const at_t lane_at = ((at_t)(S0 * PP == NT ? i0 : min(i0, S0 - 1)) * (at_t)(H * 32) + (at_t)col) * (at_t)sizeof(pair_t);
    // loads return in order: the tables' entries first, so that the tables are built while the rows are under way, and all of
    // them before the first is waited for (with __restrict__ pointers the compiler moves the rows' behind the tables' writes)
    const float2 *gh = g + (size_t)bh * F;
    constexpr int kPos = DIRECT ? 1 : (L + NT - 1) / NT;
    float2 rv[kPos], gv[kPos];
    if constexpr (!DIRECT) {
#pragma unroll
        for (int i = 0; i < kPos; ++i) {
            const int p = min(tid + NT * i, L - 1), k = Plan::bin(p / R, p % R);
            rv[i] = *lane_pointer(roots_g, 8u * p);
            gv[i] = *lane_pointer(gh, 8u * (2 * k <= L ? k : L - k));
        }
    }
    pair_t raw[kIn];
#pragma unroll
    for (int j = 0; j < kIn; ++j) {                                  // in HALF, the sweep's first row for lanes beyond the last one, then zero
        const int first = HALF ? min(S0 * j, n_rows - 1) : S0 * j;
        const pair_t *src = v + base + (size_t)first * (H * 32);
        src = lane_pointer(src, !HALF || i0 + S0 * j < n_rows ? lane_at : (at_t)col * (at_t)sizeof(pair_t));
        raw[j] = STREAM ? IO::load_stream(src) : *src;
    }
    // Above 1024 points the lanes of the form for few heads load so many factors of their own that those may go in between (us, held back /
    // free / before the scalar addresses: one head of bf16 rows at 1792 8.93 / 8.79 / 8.66, 16 of fp32 10.84 / 10.70 / 10.50, 32 at 1280
    // 11.49 / 11.31 / 11.22, one 8.83 / 8.67 / 8.81; but 32 at 784 8.22 / 8.41 / 7.97).
    if constexpr (!DIRECT || L <= 1024) __builtin_amdgcn_sched_barrier(0);
    constexpr float scale = 1.0f / (float)L;
    auto gate_fix = [&](float2 val, int k) {                         // Hermitian extension; real at DC and Nyquist
        // on the bits: selections of what a load returns become branches around it
        const uint32_t keep = (k == 0 || 2 * k == L) ? 0u : ~0u, sign = 2 * k > L ? 0x80000000u : 0u;
        return make_float2(val.x * scale, __uint_as_float((__float_as_uint(val.y) & keep) ^ sign) * scale);
    };
    float2 tw[DIRECT ? R0 : 1], G[DIRECT ? kInner * R : 1];
    if constexpr (DIRECT) {
#pragma unroll
        for (int u = 1; u < R0; ++u) tw[u] = *lane_pointer(roots_g, live ? 8u * i0 * u : 0u);
#pragma unroll
        for (int q = 0; q < kInner; ++q) {
            const int blk = min((tid + NT * q) / PP, Plan::blocks - 1);
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int k = Plan::bin(blk, u);
                G[q * R + u] = *lane_pointer(gh, 8u * (2 * k <= L ? k : L - k));
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < kPos; ++i) {
            const int p = min(tid + NT * i, L - 1);
            roots[p] = rv[i];
            gpos[p] = gate_fix(gv[i], Plan::bin(p / R, p % R));
        }
        __syncthreads();
    }
    auto factor0 = [&](int u) { return DIRECT ? tw[DIRECT ? u : 0] : roots[i0 * u]; };
    if (live) {
        float2 x[R0];
#pragma unroll
        for (int j = 0; j < R0; ++j) {
            x[j] = make_float2(0.f, 0.f);
            if (j < kIn && (!HALF || i0 + S0 * j < n_rows)) x[j] = IO::unpack(raw[j < kIn ? j : 0]);
        }
        small_dft<R0, false>(x);
#pragma unroll
        for (int u = 0; u < R0; ++u) *at(i0 + S0 * u) = u == 0 ? x[0] : cmul(x[u], factor0(u));
    }
    __syncthreads();
    // pass 1 of three: lane (i, pair) of block blk, i < R2
    constexpr int kMid = R2 > 1 ? (R0 * R2 * PP + NT - 1) / NT : 0;
    float2 tm[kMid ? R1 : 1];
    if constexpr (R2 > 1) {
        static_assert(NT % PP == 0 && NT / PP % R2 == 0, "a lane keeps its i over the blocks");
        const int i1 = i0 % R2;
#pragma unroll
        for (int u = 1; u < R1; ++u) tm[u] = DIRECT ? *lane_pointer(roots_g, 8u * i1 * u * R0) : roots[i1 * u * R0];
#pragma unroll
        for (int q = 0; q < kMid; ++q) {
            const int blk = i0 / R2 + NT / PP / R2 * q, p = blk * R1 * R2 + i1;
            if (R0 * R2 * PP % NT != 0 && blk >= R0) break;
            float2 x[R1];
#pragma unroll
            for (int j = 0; j < R1; ++j) x[j] = *at(p + R2 * j);
            small_dft<R1, false>(x);
#pragma unroll
            for (int u = 0; u < R1; ++u) *at(p + R2 * u) = u == 0 ? x[0] : cmul(x[u], tm[u]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < kInner; ++q) {
        const int blk = (tid + NT * q) / PP;
        if (Plan::blocks * PP % NT == 0 || blk < Plan::blocks) {
            float2 x[R];
#pragma unroll
            for (int j = 0; j < R; ++j) x[j] = *at(blk * R + j);
            small_dft<R, false>(x);
#pragma unroll
            for (int u = 0; u < R; ++u)
                x[u] = cmul(x[u], DIRECT ? gate_fix(G[DIRECT ? q * R + u : 0], Plan::bin(blk, u)) : gpos[blk * R + u]);
            small_dft<R, true>(x);
#pragma unroll
            for (int j = 0; j < R; ++j) *at(blk * R + j) = x[j];
        }
    }
    __syncthreads();
    if constexpr (R2 > 1) {
        const int i1 = i0 % R2;
#pragma unroll
        for (int q = 0; q < kMid; ++q) {
            const int blk = i0 / R2 + NT / PP / R2 * q, p = blk * R1 * R2 + i1;
            if (R0 * R2 * PP % NT != 0 && blk >= R0) break;
            float2 x[R1];
#pragma unroll
            for (int u = 0; u < R1; ++u) x[u] = u == 0 ? *at(p) : cmulc(*at(p + R2 * u), tm[u]);
            small_dft<R1, true>(x);
#pragma unroll
            for (int j = 0; j < R1; ++j) *at(p + R2 * j) = x[j];
        }
        __syncthreads();
    }
    if (live) {
        float2 x[R0];
#pragma unroll
        for (int u = 0; u < R0; ++u) x[u] = u == 0 ? *at(i0) : cmulc(*at(i0 + S0 * u), factor0(u));
        small_dft<R0, true>(x);
#pragma unroll
        for (int j = 0; j < kIn; ++j) {
            pair_t *dst = lane_pointer(out + base + (size_t)(S0 * j) * (H * 32), lane_at);
            if (!HALF || i0 + S0 * j < n_rows) {
                if (STREAM) IO::store_stream(dst, IO::pack(x[j]));
                else *dst = IO::pack(x[j]);
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
bool slab_supported(int L) {
    if (L < 2 || L > kSlabMaxL) return false;
    int n = L;
    for (int p : {2, 3, 5, 7})
        while (n % p == 0) n /= p;
    return n == 1;
}

// Fewest passes with radices from {16, 14, 12, 10, 8, 7, 6, 5, 4, 3, 2} (each a power of two times at most one
// of 3, 5, 7, which the in-register transform handles without twiddles); larger radices first.
static int slab_best_count(int n, int *memo) {
    if (n == 1) return 0;
    if (memo[n] != 0) return memo[n];
    int best = 1 << 20;
    for (int r : {16, 14, 12, 10, 8, 7, 6, 5, 4, 3, 2})
        if (n % r == 0) {
            const int c = 1 + slab_best_count(n / r, memo);
            if (c < best) best = c;
        }
    return memo[n] = best;
}

static SlabRadices slab_radices(int L) {
    SlabRadices r;
    r.count = 0;
    std::vector<int> memo((size_t)L + 1, 0);
    int n = L;
    while (n > 1 && r.count < 10) {
        const int want = slab_best_count(n, memo.data());
        if (want >= (1 << 20)) break;                      // not smooth: callers check slab_supported first
        for (int c : {16, 14, 12, 10, 8, 7, 6, 5, 4, 3, 2})
            if (n % c == 0 && 1 + slab_best_count(n / c, memo.data()) == want) {
                r.r[r.count++] = c;
                n /= c;
                break;
            }
    }
    return r;
}

// Position p = sum_q u_q S_q (S_q = stride of pass q) holds bin k = sum_q u_q (R_1 ... R_(q-1)) after the
// forward passes: mixed-radix digit reversal.
void slab_bin_order(int L, int *bin_of_pos) {
    const SlabRadices rad = slab_radices(L);
    for (int p = 0; p < L; ++p) {
        int rem = p, n = L, k = 0, w = 1;
        for (int q = 0; q < rad.count; ++q) {
            const int S = n / rad.r[q];
            const int u = rem / S;
            rem -= u * S;
            k += u * w;
            w *= rad.r[q];
            n = S;
        }
        bin_of_pos[p] = k;
    }
}

template <typename IO, int PP>
static hipError_t mix_slab_t(const void *v, const float2 *g, void *out, const float2 *roots, const int *bin_of_pos,
                             int B, int L, int H, int rows, hipStream_t st) {
    const size_t lds = ((size_t)L * PP + 2 * (size_t)L) * sizeof(float2);
    auto kern = k_mix_slab<IO, PP>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    kern<<<dim3(B * H * (32 / PP)), dim3(256), lds, st>>>(static_cast<const typename IO::pair_t *>(v), g,
                                                          static_cast<typename IO::pair_t *>(out), roots, bin_of_pos, L, H,
                                                          slab_radices(L), rows);
    return hipGetLastError();
}

template <typename IO, int PP, int NT, int R0, int R1, int R2, bool DIRECT, bool STREAM, bool HALF, bool WIDE>
static hipError_t mix_ct_t(const void *v, const float2 *g, void *out, const float2 *roots, int B, int H, int rows,
                           hipStream_t st) {
    constexpr size_t lds = SlabPlan<R0, R1, R2>::lds(PP, DIRECT);
    auto kern = k_mix_ct<IO, PP, NT, R0, R1, R2, DIRECT, STREAM, HALF, WIDE>;
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    const int BH = B * H, affine = PP < 32, most = slab_launch_heads(32 / PP, NT);
    for (int bh0 = 0, n; bh0 < BH; bh0 += n) {
        n = BH - bh0 < most ? BH - bh0 : most;
        const int grid = (affine ? (n + 7) / 8 * 8 : n) * (32 / PP);
        kern<<<dim3(grid), dim3(NT), lds, st>>>(static_cast<const typename IO::pair_t *>(v), g,
                                                static_cast<typename IO::pair_t *>(out), roots, H, bh0, BH, rows, affine);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Pairs per workgroup: as many as leave room for three workgroups per compute unit (slab L*PP + two tables of L
// complex numbers <= 52 KB; measured at B*H = 3072: L = 512 and the padded 197 are 5-24 % faster with 8 pairs than
// with 16, L = 256 bf16 30 % faster with 16 than with 32), no more than keeps every compute unit busy
// (B*H*32/PP >= 256 workgroups), at most a whole head (half a head for fp32 rows).
int slab_pairs_per_workgroup(int io, int BH, int L) {
    int pp = io ? 32 : 16;
    while (pp > 4 && (size_t)L * (pp + 2) * sizeof(float2) > (size_t)52 * 1024) pp /= 2;   // three workgroups per CU
    while (pp > 4 && (long long)BH * (32 / pp) < 256) pp /= 2;
    return pp;
}

// The lengths with compile-time radices, false for any other: the patch grids n x n with n = 12, 14, 16, 20, 24, 28 and 32, and
// the lengths of up to 2048 points that have a four-step plan or serve as data length of the padded convolution (mix_chirp.hip).
// Most have two forms.
//   few heads : four pairs per workgroup (1024, 1536 and 1792: two), every lane with its own loads of factors and gate, while the
//               launch has at most a wave per SIMD: until then a call costs what one workgroup does, and above it the
//               narrow pieces of rows and the repeated loads do.  Half a wave per SIMD for the two-pass lengths (80 heads, bf16: 144
//               points 4.3 / 4.1 us, 196 5.7 / 5.4; 64 heads 4.0 / 4.0 and 4.9 / 5.1).
//   otherwise : the tables in LDS, at the pairs per workgroup that are fastest for many heads.
// Kernel alone over rotating buffers, bf16 rows, us, few form / other form:
//   heads       1             8            32            64           128           768       few up to
//    196    3.9 /  4.6    4.0 /  4.8    4.2 /  4.8    4.9 /  5.1    6.6 /  5.7    25.2 / 15.1     64
//    256    3.6 /  4.8    3.7 /  5.0    4.1 /  5.1    5.3 /  5.7    6.7 /  6.2    29.1 / 17.4     64
//    448    4.1 /  4.5    4.2 /  4.6    5.1 /  5.4    6.8 /  6.0   10.4 /  8.8    54.2 / 36.9     32
//    896    6.4 /  7.3    6.6 /  8.0    8.4 /  8.9   10.9 / 10.2   21.6 / 16.5     132 / 82.2     32
//   1024    6.3 /  7.3    6.6 /  7.8   10.2 /  9.4   18.1 / 12.9   32.3 / 22.1     215 /  138     16
//   1280    8.9 /  9.3    9.1 /  9.5   11.6 / 11.7   18.4 / 18.1   33.8 / 31.6     203 /  175     32
//   1536    8.4 / 10.0    8.5 / 10.2   13.4 / 12.9   28.5 / 20.5   52.2 / 35.8     359 /  213     16
// Lengths without a form for few, and the splits of the other form: three short passes on more lanes beat two passes of radix 28 and 32,
// which leave two waves per SIMD (24 x 24 excepted), and eight pairs per workgroup beat four while a compute unit still holds two or
// more.  Chosen with per-lane addresses.  With scalar ones, bf16 rows over rotating buffers, us at one / 32 / 768 heads:
//    512 as  8 x 8 x 8 on eight pairs 4.7 / 5.7 / 40.6; on four 4.4 / 5.5 / 54.6, as form for few 4.1 / 5.2 / 62.9; 32 x 16 7.3 / 8.3 / 50.9
//    768 as 12 x 8 x 8 on eight (form for few 6.0 / 7.6) - / - / 67.6; 24 x 32 on four 7.3 / 8.9 / 96.5, on eight 7.4 / 8.9 / 69.4
//    896 as 14 x 8 x 8 on eight (6.5 / 8.3) - / - / 80.5; on four 7.0 / 8.6 / 113; 28 x 32 on four 8.0 / 9.9 / 123
//   1024 as 16 x 8 x 8 on four (6.4 / 9.3) - / - / 136; on eight 7.5 / 9.3 / 126; 16 x 16 x 4 6.9 / 9.0 / 130; 32 x 32 8.6 / 10.6 / 149
//   1280 as 20 x 8 x 8 on four (9.3 / 11.5) - / - / 172; 16 x 16 x 5 8.7 / 10.7 / 256; 10 x 16 x 8 7.7 / 9.6 / 214
//    576 as 24 x 24 on eight (5.3 / 6.6) - / - / 51.6; 12 x 6 x 8 5.7 / 6.9 / 54.4
//    640 as 20 x 32 on eight 6.7 / 8.2 / 53.4; as form for few on four 6.5 / 7.9 / 90.1; 10 x 8 x 8 6.1 / 7.3 / 58.3
//    400 as 20 x 20 on eight 6.1 / 7.0 / 36.2; on sixteen 5.8 / 6.6 / 30.3, as form for few on four 5.3 / 6.3 / 55.1; 10 x 8 x 5 5.5 / 6.4 / 40.4
//    320 as 20 x 16 on sixteen 6.1 / 6.8 / 23.8; as form for few on four 5.6 / 6.4 / 44.9; 5 x 8 x 8 as form for few 3.7 / 4.5 / 40.4
//   2048 as 16 x 16 x 8 on four 10.4 / 15.4 / 324; as form for few on two 10.3 / 22.8 / 324
// So 512, 640 and 1280 would now gain by another form for few heads and 400 by sixteen pairs, which is not taken yet; three passes of 320 and
// 400 have 3 and 5 % more error than two.
template <typename IO>
static bool mix_ct(int L, const void *v, const float2 *g, void *out, const float2 *roots, int B, int H, int rows,
                   hipStream_t st, hipError_t *e) {
    constexpr bool bf = IO::kBytes == 2;
    constexpr int kSimds = 1024;
    const long long heads = (long long)B * H;
    // Rows that will not be found in the memory-side cache again pass it by, where a workgroup's piece of a row is whole
    // 128-byte lines (fp32, H = 12, us: L = 196, B = 256 67.7 -> 62.1, 128 35.4 -> 34.0, but 64 16.5 -> 17.6; 256 at B = 256 86 -> 80,
    // bf16 53 -> 49).  fp32 rows of 196 go by whole heads from there on (half / whole heads, B = 64 16.5 / 17.6, 256 64.3 / 62.1,
    // 1300 315 / 296).
    const bool large = 64 * heads * rows * (long long)sizeof(typename IO::pair_t) > 100000000;
    const bool stream = large && ((reinterpret_cast<uintptr_t>(v) | reinterpret_cast<uintptr_t>(out)) & 127) == 0;
    if (!slab_ct_rows(L, rows)) return false;
#define SPECTRE_CT_RUN(PP, NT, R0, R1, R2, DIRECT, STREAM, HALF)                                                        \
    {                                                                                                                   \
        if constexpr (!DIRECT) {                                                                                        \
            if ((long long)(R1 * R2) * H * 32 * (long long)sizeof(typename IO::pair_t) >= (1LL << 32)) {                \
                *e = mix_ct_t<IO, PP, NT, R0, R1, R2, DIRECT, STREAM, HALF, true>(v, g, out, roots, B, H, rows, st);    \
                return true;                                                                                            \
            }                                                                                                           \
        }                                                                                                               \
        *e = mix_ct_t<IO, PP, NT, R0, R1, R2, DIRECT, STREAM, HALF, false>(v, g, out, roots, B, H, rows, st);           \
        return true;                                                                                                    \
    }
#define SPECTRE_CT(PP, NT, R0, R1, R2, DIRECT, STREAM)                                                                  \
    {                                                                                                                   \
        if (rows != L) {                                                                                                \
            if constexpr (chirp_uses(R0 * R1 * R2)) SPECTRE_CT_RUN(PP, NT, R0, R1, R2, DIRECT, STREAM, true)            \
            return false;                                                                                               \
        }                                                                                                               \
        SPECTRE_CT_RUN(PP, NT, R0, R1, R2, DIRECT, STREAM, false)                                                       \
    }
#define SPECTRE_CT_FEW(PP, NT, R0, R1, R2) \
    if (heads * (32 / PP) * (NT / 64) <= (R2 > 1 ? kSimds : kSimds / 2)) SPECTRE_CT(PP, NT, R0, R1, R2, true, false)
#define SPECTRE_CT_LINES(PP, NT, R0, R1, R2)                                                                            \
    {                                                                                                                   \
        static_assert(PP * sizeof(typename IO::pair_t) % 128 == 0, "whole lines");                                      \
        if (stream) SPECTRE_CT(PP, NT, R0, R1, R2, false, true)                                                         \
        SPECTRE_CT(PP, NT, R0, R1, R2, false, false)                                                                    \
    }
    switch (L) {
        case 144:
            SPECTRE_CT_FEW(4, 64, 12, 12, 1)
            if constexpr (bf) SPECTRE_CT_LINES(32, 384, 12, 12, 1)
            else SPECTRE_CT_LINES(16, 192, 12, 12, 1)
        case 196:
            SPECTRE_CT_FEW(4, 64, 14, 14, 1)
            if (!bf && !large) SPECTRE_CT(16, 256, 14, 14, 1, false, false)
            SPECTRE_CT_LINES(32, 448, 14, 14, 1)
        case 256:
            SPECTRE_CT_FEW(4, 128, 8, 8, 4)
            if constexpr (bf) SPECTRE_CT_LINES(32, 512, 16, 16, 1)
            else SPECTRE_CT_LINES(16, 512, 8, 8, 4)
        case 320: SPECTRE_CT(16, 256, 20, 16, 1, false, false)
        case 400: SPECTRE_CT(8, 192, 20, 20, 1, false, false)
        case 448: SPECTRE_CT_FEW(4, 256, 7, 8, 8) SPECTRE_CT(8, 512, 7, 8, 8, false, false)
        case 512: SPECTRE_CT(8, 512, 8, 8, 8, false, false)
        case 576: SPECTRE_CT_FEW(4, 192, 12, 12, 4) SPECTRE_CT(8, 192, 24, 24, 1, false, false)
        case 640: SPECTRE_CT(8, 256, 20, 32, 1, false, false)
        case 768: SPECTRE_CT_FEW(4, 256, 12, 8, 8) SPECTRE_CT(8, 512, 12, 8, 8, false, false)
        case 784: SPECTRE_CT_FEW(4, 256, 14, 7, 8) SPECTRE_CT(8, 448, 14, 7, 8, false, false)
        case 896: SPECTRE_CT_FEW(4, 256, 14, 8, 8) SPECTRE_CT(8, 512, 14, 8, 8, false, false)
        case 1024: SPECTRE_CT_FEW(2, 256, 8, 16, 8) SPECTRE_CT(4, 256, 16, 8, 8, false, false)
        case 1280: SPECTRE_CT_FEW(4, 256, 20, 8, 8) SPECTRE_CT(4, 256, 20, 8, 8, false, false)
        case 1536: SPECTRE_CT_FEW(2, 256, 12, 16, 8) SPECTRE_CT(4, 256, 24, 8, 8, false, false)
        case 1792: SPECTRE_CT_FEW(2, 256, 14, 16, 8) SPECTRE_CT(4, 512, 14, 16, 8, false, false)
        case 2048: SPECTRE_CT(4, 512, 16, 16, 8, false, false)
        default: return false;
    }
#undef SPECTRE_CT_RUN
#undef SPECTRE_CT
#undef SPECTRE_CT_FEW
#undef SPECTRE_CT_LINES
}

hipError_t launch_mix_slab(int io, const void *v, const float2 *g, void *out, const float2 *roots,
                           const int *bin_of_pos, int B, int L, int H, hipStream_t st, int rows) {
    if (rows <= 0) rows = L;
    if (rows > L) return hipErrorInvalidValue;
    const int pp = slab_pairs_per_workgroup(io, B * H, L);
    if ((size_t)L * (pp + 2) * sizeof(float2) > (size_t)160 * 1024) return hipErrorInvalidValue;
    if (option(SPECTRE_OPT_SLAB_COMPILE_TIME) != 0) {
        hipError_t e = hipSuccess;
        const bool done = io ? mix_ct<IoBf16>(L, v, g, out, roots, B, H, rows, st, &e)
                             : mix_ct<IoF32>(L, v, g, out, roots, B, H, rows, st, &e);
        if (done) return e;
    }
    switch (pp) {
#define SPECTRE_SLAB_CASE(PPV)                                                                    \
    case PPV:                                                                                    \
        return io ? mix_slab_t<IoBf16, PPV>(v, g, out, roots, bin_of_pos, B, L, H, rows, st)     \
                  : mix_slab_t<IoF32, PPV>(v, g, out, roots, bin_of_pos, B, L, H, rows, st);
        SPECTRE_SLAB_CASE(4)
        SPECTRE_SLAB_CASE(8)
        SPECTRE_SLAB_CASE(16)
        SPECTRE_SLAB_CASE(32)
#undef SPECTRE_SLAB_CASE
        default: return hipErrorInvalidValue;
    }
}

// Loads this translation unit's code object (the runtime loads them on first use): called by spectre_prepare so
// that no compute call is the first to touch it.
hipError_t load_kernels_mix_slab() {
    hipFuncAttributes a;
    return hipFuncGetAttributes(&a, reinterpret_cast<const void *>((k_mix_slab<IoF32, 4>)));
}

}  // namespace spectre
