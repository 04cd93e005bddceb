// Four-step transform path of the SPECTRE mixing layer (Sec. 3.2 steps 2-4,
// Eq. 3 and Eq. 4) for gfx950: L = N1 * N2 with N1 = 256 or 4096 and N2 <= 32 of the
// form {1, 3, 5, 7} * 2^a.
//
// Two adjacent channels of a head are transformed together as one complex
// sequence z = v_even + j v_odd.  Because the gate is extended to all L bins by
// Hermitian symmetry (App. B, Thm. B.1), multiplying the complex spectrum of z
// by it and transforming back leaves the two real results in the real and
// imaginary parts, so no split/merge pass is needed and a bf16 channel pair is
// one 32-bit load.
//
// L = N1 * N2, time index t = t1 + N1*t2, frequency index k = k2 + N2*k1:
//   small_fwd : A[t1,k2]  = W_L^(t1 k2) * sum_t2 z[t1 + N1 t2] W_N2^(t2 k2)      (one lane per (t1, pair))
//   big       : Z[k2+N2 k1] = sum_t1 A[t1,k2] W_N1^(t1 k1);  Y = G * Z;  B[t1,k2] = sum_k1 Y W_N1^(-t1 k1)
//   small_inv : out[t1 + N1 t2] = sum_k2 conj(W_L^(t1 k2)) B[t1,k2] W_N2^(-t2 k2)
// with W_n = exp(-j 2 pi / n) and the 1/L of the inverse folded into G.
#include "mix_pow2.h"

#include <type_traits>

#include "fft_regs.h"
#include "internal.h"
#include "scratch_elem.h"

namespace spectre {

// Shape of the row kernels' tile: TT = 16 adjacent t1 (128-byte runs in the scratch) times kPairs channel pairs, one
// 128-byte segment of every row: a whole bf16 head row, or one half of an fp32 head row (its two halves go to two
// workgroups, so that rows with 8-byte pairs keep whole 128-byte lines on both sides of the kernel).
// kStride: LDS row stride (in pair_t units) of the [t2][t1_local][pair] staging tile, chosen so that a wave reading
// along t1_local with 16 lanes per pair index hits every bank equally.
template <typename IO> struct RowTile;
template <> struct RowTile<IoBf16> { static constexpr int kPairs = 32, kStride = 36; };
template <> struct RowTile<IoF32> { static constexpr int kPairs = 16, kStride = 18; };
template <typename IO> struct TileStride { static constexpr int value = RowTile<IO>::kStride; };

// Where it gains, the addresses of the row kernels are a scalar base per row or block and one 32-bit offset of the lane
// (lane_pointer): 64-bit products per lane and row are a quarter of these kernels' vector time.
//
// small_fwd: grid (N1/TT * 32/PW, nbh); block PW*TT threads, PW = RowTile<IO>::kPairs.  Reads the N2*TT rows
// {t1_0 + r + N1*t2} of one head (PW pairs each, one 128-byte segment per row),
// stages them in LDS, then lane (pair p, t1_local) runs the N2-point DFT over t2.
// ring != nullptr (pre-fill of an empty Prefix-FFT cache): every row read is also copied, as fp32, to row l of head bh
// of the value ring buffer ring [B*H][N1 * N2][32 pairs] - the rows then cross HBM once for both purposes.
// PART: fewer rows than the transform, a ring, or a size at which it is the faster (small_fwd_t).  Addresses stay per lane there: as scalar
// ones the row loads and the stores to ring and scratch come in denser bursts, which memory moves more slowly (20011 tokens, B = 8 H =
// 32 N = 32768, 2760 -> 2815 us; mixer of 2 x 8 heads at 5000 105 -> 106).
template <int N2, int TT, typename IO, typename SC, bool PART>
__global__ __launch_bounds__(RowTile<IO>::kPairs * TT) void k_small_fwd(const typename IO::pair_t *__restrict__ v,
                                                       typename SC::elem_t *__restrict__ scr,
                                                       const float2 *__restrict__ twL, int rows, int H,
                                                       int N1, int bh0, int aff, float2 *__restrict__ ring) {
    typedef typename IO::pair_t pair_t;
    constexpr int S = TileStride<IO>::value, PW = RowTile<IO>::kPairs, NPART = 32 / PW;
    extern __shared__ unsigned char smem_raw[];
    pair_t *lds = reinterpret_cast<pair_t *>(smem_raw);
    const int tid = threadIdx.x;
    int tile = blockIdx.x, bhl = blockIdx.y;
    if (aff) head_affine(blockIdx.x, N1 / TT * NPART, aff, false, &bhl, &tile);
    const int t1_0 = (tile / NPART) * TT, p0 = (tile % NPART) * PW;
    const int bh = bh0 + bhl, b = bh / H, h = bh % H;
    {
        const int lp = tid % PW, r = tid / PW;
        pair_t val[N2];
        if (!PART) {
            const unsigned lane_at = (unsigned)(r * H * 32 + lp) * (unsigned)sizeof(pair_t);   // r < 16
#pragma unroll
            for (int t2 = 0; t2 < N2; ++t2)
                val[t2] = IO::load_stream(lane_pointer(v + (((size_t)b * rows + t1_0 + N1 * t2) * H + h) * 32 + p0, lane_at));
        } else {                                                     // zeros behind the last row
#pragma unroll
            for (int t2 = 0; t2 < N2; ++t2) {
                const int l = t1_0 + r + N1 * t2;
                val[t2] = (l < rows) ? IO::load_stream(v + (((size_t)b * rows + l) * H + h) * 32 + p0 + lp) : IO::zero();
            }
        }
#pragma unroll
        for (int t2 = 0; t2 < N2; ++t2) lds[(t2 * TT + r) * S + lp] = val[t2];
        if (PART && ring) {
#pragma unroll
            for (int t2 = 0; t2 < N2; ++t2) {
                const int l = t1_0 + r + N1 * t2;
                if (l < rows) stream_store(ring + ((size_t)bh * N1 * N2 + l) * 32 + p0 + lp, IO::unpack(val[t2]));
            }
        }
    }
    __syncthreads();
    const int tl = tid % TT, p = tid / TT, t1 = t1_0 + tl;
    float2 x[N2];
#pragma unroll
    for (int t2 = 0; t2 < N2; ++t2) x[t2] = IO::unpack(lds[(t2 * TT + tl) * S + p]);
    small_dft<N2, false>(x);
    typename SC::elem_t *dst = scr + (((size_t)bhl * N2) * 32 + p0) * N1 + t1_0, *own = dst + (size_t)p * N1 + tl;
    const unsigned scr_at = (unsigned)(p * N1 + tl) * (unsigned)sizeof(typename SC::elem_t);
    const SmallTwiddles<N2, std::is_same<SC, ScrF32Fine>::value> tw(twL, t1);
#pragma unroll
    for (int k2 = 0; k2 < N2; ++k2) {
        const float2 y = (k2 == 0) ? x[0] : cmul(x[k2], tw(k2));
        if (PART) own[(size_t)k2 * 32 * N1] = SC::put(y);
        else *lane_pointer(dst + (size_t)k2 * 32 * N1, scr_at) = SC::put(y);
    }
}

// small_fwd with the token projection in front (Sec. 3.2 step 1, Eq. 2, feeding step 2): the workgroup reads rows of
// the layer input X instead of V, multiplies every row by its head's 64 x 64 value matrix on the matrix cores and
// rounds the products to bfloat16 into the same LDS tile the plain kernel fills from memory - the bits the separate
// projection kernel would have stored as V (same instruction, same order of the hi/lo weight terms), which then
// never exist in HBM.  bf16 rows, TT = 16.  wpack: the weights as the B operand (k_pack_w), held in registers.
// A wave takes 32 tile rows at a time (two adjacent t2 of the 16 t1): lane l supplies row l % 32 and the channels
// 16 ks + 8 (l / 32) .. + 7 of k-step ks as one 16-byte LDS read; accumulator register v of lane l is row
// 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32 of a 32-column block, so a channel pair sits in two adjacent lanes:
// even lanes pack the pairs of columns 0..31, odd lanes those of columns 32..63, each fetching the neighbour's half
// with a quad permutation.  The rows a wave overwrites are the ones it has just read, and no other wave touches them.
typedef float floatx16_t __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

template <int N2, typename SC>
__global__ __launch_bounds__(512) void k_small_fwd_proj(const uint32_t *__restrict__ x, const uint4 *__restrict__ wpack,
                                                        int Hw, float2 *__restrict__ scr,
                                                        const float2 *__restrict__ twL, int rows, int H, int N1,
                                                        int bh0, int aff) {
    constexpr int TT = 16, S = TileStride<IoBf16>::value, NROW = N2 * TT, NGRP = (NROW + 31) / 32;
    extern __shared__ unsigned char smem_raw[];
    uint32_t *lds = reinterpret_cast<uint32_t *>(smem_raw);
    const int tid = threadIdx.x;
    int tile = blockIdx.x, bhl = blockIdx.y;
    if (aff) head_affine(blockIdx.x, N1 / TT, aff, false, &bhl, &tile);
    const int t1_0 = tile * TT;
    const int bh = bh0 + bhl, b = bh / H, h = bh % H;
    {
        const int lp = tid & 31, r = tid >> 5;
        uint32_t val[N2];
        const unsigned lane_at = 4u * (r * H * 32 + lp);                 // r < 16
        auto row = [&](int t2) { return x + (((size_t)b * rows + t1_0 + N1 * t2) * H + h) * 32; };
        if (t1_0 + TT + N1 * (N2 - 1) <= rows) {
#pragma unroll
            for (int t2 = 0; t2 < N2; ++t2) val[t2] = IoBf16::load_stream(lane_pointer(row(t2), lane_at));
        } else {
#pragma unroll
            for (int t2 = 0; t2 < N2; ++t2) {
                val[t2] = 0u;
                if (t1_0 + r + N1 * t2 < rows) val[t2] = IoBf16::load_stream(lane_pointer(row(t2), lane_at));
            }
        }
#pragma unroll
        for (int t2 = 0; t2 < N2; ++t2) lds[(t2 * TT + r) * S + lp] = val[t2];
    }
    const int lane = tid & 63, wave = tid >> 6, i = lane & 31, half = lane >> 5;
    uint4 whi[8], wlo[8];                              // [ks * 2 + column block]
    {
        const uint4 *wp = wpack + (size_t)((Hw == 1) ? 0 : h) * 1024 + lane;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            whi[e] = wp[e * 64];
            wlo[e] = wp[512 + e * 64];
        }
    }
    __syncthreads();
    for (int g = wave; g < NGRP; g += 8) {
        const int ri = 32 * g + i;
        uint4 a[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            a[ks] = (ri < NROW) ? *reinterpret_cast<const uint4 *>(lds + ri * S + 8 * ks + 4 * half) : make_uint4(0, 0, 0, 0);
        floatx16_t acc0 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}, acc1 = acc0;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const bf16x8_t av = __builtin_bit_cast(bf16x8_t, a[ks]);
            acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, __builtin_bit_cast(bf16x8_t, wlo[2 * ks]), acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, __builtin_bit_cast(bf16x8_t, wlo[2 * ks + 1]), acc1, 0, 0, 0);
            acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, __builtin_bit_cast(bf16x8_t, whi[2 * ks]), acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, __builtin_bit_cast(bf16x8_t, whi[2 * ks + 1]), acc1, 0, 0, 0);
        }
        const bool odd = i & 1;
        const int pcol = odd ? 16 + (i >> 1) : (i >> 1);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = 32 * g + 8 * (v / 4) + 4 * half + (v % 4);
            const float n0 = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(acc0[v]), 0xB1, 0xF, 0xF, false));
            const float n1 = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(acc1[v]), 0xB1, 0xF, 0xF, false));
            const float2 pr = odd ? make_float2(n1, acc1[v]) : make_float2(acc0[v], n0);
            if (row < NROW) lds[row * S + pcol] = IoBf16::pack(pr);
        }
    }
    __syncthreads();
    const int tl = tid % TT, p = tid / TT, t1 = t1_0 + tl;
    float2 xv[N2];
#pragma unroll
    for (int t2 = 0; t2 < N2; ++t2) xv[t2] = IoBf16::unpack(lds[(t2 * TT + tl) * S + p]);
    small_dft<N2, false>(xv);
    float2 *dst = scr + (size_t)bhl * N2 * 32 * N1 + t1_0;
    const unsigned scr_at = 8u * (p * N1 + tl);
    const SmallTwiddles<N2, std::is_same<SC, ScrF32Fine>::value> tw(twL, t1);
#pragma unroll
    for (int k2 = 0; k2 < N2; ++k2) {
        const float2 y = (k2 == 0) ? xv[0] : cmul(xv[k2], tw(k2));
        *lane_pointer(dst + (size_t)k2 * 32 * N1, scr_at) = y;
    }
}

// small_inv: mirror image.  Rows l of the inverse transform with row0 <= l < row0+out_rows
// are written to row l-row0 of out [B, out_rows, H, d].  With ring_w > 0 the rows are instead
// gathered from a ring buffer that occupies rows ring0 .. ring0+ring_w-1 and whose newest entry
// sits at ring0+newest: the out_rows newest entries are written oldest first.
// bsum != nullptr (mixer followed by the wavelet refinement): the workgroup also emits the sums of the TT adjacent rows
// it writes for every t2, taken over the values as stored (after rounding to the I/O type), to
// bsum [bh][L / TT][32 pairs]; block l / TT covers rows l .. l + TT - 1.  Added in row order.
template <int N2, int TT, typename IO, typename SC>
__global__ __launch_bounds__(RowTile<IO>::kPairs * TT) void k_small_inv(const typename SC::elem_t *__restrict__ scr,
                                                       typename IO::pair_t *__restrict__ out,
                                                       const float2 *__restrict__ twL, int row0,
                                                       int out_rows, int H, int N1, int bh0, int ring0,
                                                       int ring_w, int newest, int aff, float2 *__restrict__ bsum) {
    typedef typename IO::pair_t pair_t;
    constexpr int S = TileStride<IO>::value, PW = RowTile<IO>::kPairs, NPART = 32 / PW;
    extern __shared__ unsigned char smem_raw[];
    pair_t *lds = reinterpret_cast<pair_t *>(smem_raw);
    const int tid = threadIdx.x;
    int tile = blockIdx.x, bhl = blockIdx.y;
    if (aff) head_affine(blockIdx.x, N1 / TT * NPART, aff, false, &bhl, &tile);
    const int t1_0 = (tile / NPART) * TT, p0 = (tile % NPART) * PW;
    const int bh = bh0 + bhl, b = bh / H, h = bh % H;
    {
        const int tl = tid % TT, p = tid / TT, t1 = t1_0 + tl;
        const typename SC::elem_t *src = scr + (((size_t)bhl * N2) * 32 + p0) * N1 + t1_0, *own = src + (size_t)p * N1 + tl;
        const unsigned scr_at = (unsigned)(p * N1 + tl) * (unsigned)sizeof(typename SC::elem_t);
        // scalar addresses for 28 fp32 rows only (us, per lane / scalar: readout of 40 heads of 7168 slots 55.2 / 52.7, mixer of 20 heads at 7168
        // 49.1 / 48.0, 100 207.6 / 204.9, 2 at 114688 75.7 / 74.9, 9 at 28672 79.0 / 79.1; bf16 rows, readout of 40 47.7 / 48.7; 24 fp32 rows, window of 18
        // heads of 6144 slots 27.5 / 28.2, mixer of 64 at 24576 418 / 422)
        constexpr bool kScalar = std::is_same<IO, IoF32>::value && N2 == 28;
        typename SC::elem_t raw[N2];
#pragma unroll
        for (int k2 = 0; k2 < N2; ++k2) raw[k2] = kScalar ? *lane_pointer(src + (size_t)k2 * 32 * N1, scr_at) : own[(size_t)k2 * 32 * N1];
        float2 y[N2];
#pragma unroll
        for (int k2 = 0; k2 < N2; ++k2) y[k2] = SC::get(raw[k2]);
        const SmallTwiddles<N2, std::is_same<SC, ScrF32Fine>::value> tw(twL, t1);
#pragma unroll
        for (int k2 = 1; k2 < N2; ++k2) y[k2] = cmulc(y[k2], tw(k2));
        small_dft<N2, true>(y);
#pragma unroll
        for (int t2 = 0; t2 < N2; ++t2) lds[(t2 * TT + tl) * S + p] = IO::pack(y[t2]);
    }
    __syncthreads();
    const int lp = tid % PW, r = tid / PW;
#pragma unroll
    for (int t2 = 0; t2 < N2; ++t2) {
        const int l = t1_0 + r + N1 * t2;
        int orow = l - row0;
        if (ring_w > 0) {
            int age = newest - (l - ring0);            // 0 = newest entry of the ring
            if (age < 0) age += ring_w;
            orow = (l >= ring0) ? out_rows - 1 - age : -1;
        }
        if (orow >= 0 && orow < out_rows)
            IO::store_stream(out + (((size_t)b * out_rows + orow) * H + h) * 32 + p0 + lp, lds[(t2 * TT + r) * S + lp]);
    }
    if (bsum) {                                        // lane (lp, r) sums the TT rows of t2 = r, r + TT, ...
        for (int t2 = r; t2 < N2; t2 += TT) {
            float2 acc = make_float2(0.f, 0.f);
#pragma unroll
            for (int i = 0; i < TT; ++i) acc = acc + IO::unpack(lds[(t2 * TT + i) * S + lp]);
            bsum[((size_t)bh * (N1 / TT) * N2 + (t1_0 / TT + (N1 / TT) * t2)) * 32 + p0 + lp] = acc;
        }
    }
}

// ------------------------------------------------------------------------------------------
// big: N1 = 16^P points per column, 16 per lane, P radix-16 passes each way with an LDS
// exchange between passes.  Forward passes are decimation in frequency (natural order in,
// base-16 digit-reversed order out), inverse passes undo them in reverse, so the gate is
// applied in digit-reversed order (the expanded gate is stored that way) and no reordering
// pass exists.  Pass q (0-based) has stride S = 16^(P-1-q): lane tau owns positions
// (tau / S) * 16 S + tau % S + S * j, j = 0..15.  LDS positions are padded by one element per
// 16 (p -> p + p/16); for S >= 16 that keeps a lane's 16 positions an arithmetic sequence.
//
// Only the exchange between passes 0 and 1 of a 4096-point column crosses waves; every other
// exchange stays inside a group of 16 lanes that own the same 256-position block, and needs no
// workgroup barrier because the LDS operations of one wave complete in issue order.  The forward
// and the inverse cross-wave exchange share one buffer (35 KB per workgroup, which leaves room on a
// compute unit for a row-transform workgroup of a neighbouring head group running on the other
// stream).  Between the two, lanes only touch the 256-position block they own, so the only extra
// barrier is at the end of a column: the next column's forward write lands on positions that
// slower waves may still be reading for the inverse exchange.
template <int P, int Q>
__device__ __forceinline__ int pad_base(int tau) {
    constexpr int S = 1 << (4 * (P - 1 - Q));
    if (S == 1) return 17 * tau;
    const int p = (tau / S) * (16 * S) + (tau % S);
    return p + (p >> 4);
}
template <int P, int Q>
__device__ constexpr int pad_stride() {
    constexpr int S = 1 << (4 * (P - 1 - Q));
    return S == 1 ? 1 : S + S / 16;
}

// write at pass QFROM's positions, read at pass QTO's.  CROSS: other waves take part.
template <int P, int QFROM, int QTO, bool CROSS>
__device__ __forceinline__ void exchange(float2 (&x)[16], float2 *buf, int tau) {
    float2 *w = buf + pad_base<P, QFROM>(tau);
    const float2 *r = buf + pad_base<P, QTO>(tau);
#pragma unroll
    for (int j = 0; j < 16; ++j) w[j * pad_stride<P, QFROM>()] = x[j];
    if (CROSS) __syncthreads();
    else __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = r[j * pad_stride<P, QTO>()];
    if (!CROSS) __builtin_amdgcn_wave_barrier();
}

// The same exchange inside a group of 16 lanes without LDS: a 16 x 16 transpose (register j of lane a <-> register
// a of lane j) as four steps, one per index bit m, each swapping the elements whose register bit and lane bit
// differ with the partner lane a ^ m, by DPP moves (rows of 16 lanes are the DPP rows of a wave).  For m = 4, 8 the
// lanes that receive are whole banks of four lanes, so two masked moves per value do the step; for m = 1, 2 the
// partner's value is fetched with a quad permutation and selected per lane.  Pure data movement: results are
// bit-identical to the LDS exchange.
template <int M>
__device__ __forceinline__ void transpose16_step(float (&v)[16], int a) {
#pragma unroll
    for (int j0 = 0; j0 < 16; ++j0) {
        if (j0 & M) continue;
        const int j1 = j0 | M;
        const int lo = __float_as_int(v[j0]), hi = __float_as_int(v[j1]);
        int nlo, nhi;
        if constexpr (M == 8) {          // lanes 8..15 take the partner's hi into lo; lanes 0..7 the partner's lo into hi
            nlo = __builtin_amdgcn_update_dpp(lo, hi, 0x118, 0xF, 0xC, false);   // row_shr:8, banks 2,3
            nhi = __builtin_amdgcn_update_dpp(hi, lo, 0x108, 0xF, 0x3, false);   // row_shl:8, banks 0,1
        } else if constexpr (M == 4) {
            nlo = __builtin_amdgcn_update_dpp(lo, hi, 0x114, 0xF, 0xA, false);   // row_shr:4, banks 1,3
            nhi = __builtin_amdgcn_update_dpp(hi, lo, 0x104, 0xF, 0x5, false);   // row_shl:4, banks 0,2
        } else {
            constexpr int ctrl = (M == 1) ? 0xB1 : 0x4E;                          // quad_perm [1,0,3,2] / [2,3,0,1]
            const int phi = __builtin_amdgcn_update_dpp(0, hi, ctrl, 0xF, 0xF, false);
            const int plo = __builtin_amdgcn_update_dpp(0, lo, ctrl, 0xF, 0xF, false);
            nlo = (a & M) ? phi : lo;
            nhi = (a & M) ? hi : plo;
        }
        v[j0] = __int_as_float(nlo);
        v[j1] = __int_as_float(nhi);
    }
}
__device__ __forceinline__ void transpose16(float2 (&x)[16], int tau) {
    const int a = tau & 15;
    float re[16], im[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) { re[j] = x[j].x; im[j] = x[j].y; }
    transpose16_step<8>(re, a); transpose16_step<8>(im, a);
    transpose16_step<4>(re, a); transpose16_step<4>(im, a);
    transpose16_step<2>(re, a); transpose16_step<2>(im, a);
    transpose16_step<1>(re, a); transpose16_step<1>(im, a);
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = make_float2(re[j], im[j]);
}

// SHFL: the exchanges that stay inside 16 lanes go through transpose16 instead of LDS.
template <int P, int MODE, typename SC, bool SHFL = false>
__global__ __launch_bounds__(256) void k_big(typename SC::elem_t *__restrict__ scr, const float2 *__restrict__ gp,
                                             const float2 *__restrict__ twN1, int N2, int ppw, int bh0,
                                             int nplanes_xcd, int g_step, int aff, int through) {
    static_assert(P == 2 || P == 3, "N1 is 256 or 4096");
    constexpr int N1 = 1 << (4 * P), TPC = N1 / 16, CPI = 256 / TPC, COLW = N1 + N1 / 16;
    constexpr bool kCross = (P == 3);                // does the pass 0 <-> 1 exchange span waves?
    extern __shared__ float2 lds_big[];
    const int tid = threadIdx.x, tau = tid % TPC, ci = tid / TPC;
    // Workgroups are dealt round-robin to the 8 XCDs (each with its own L2).  The 32/ppw workgroups
    // that share one (head, k2) plane of the expanded gate are given ids 8 apart, so they run on
    // the same XCD and the plane is fetched into one L2 instead of eight.
    const int groups = 32 / ppw;
    int blk = blockIdx.x;
    if (nplanes_xcd > 0) {
        const int xcd = blk & 7, idx = blk >> 3;
        blk = ((idx / groups) * 8 + xcd) * groups + idx % groups;
    }
    int pg = blk % groups;
    blk /= groups;
    int k2 = blk % N2, bhl = blk / N2;
    if (aff) {                                       // all planes of a head on one XCD, heads walked downwards
        int within;
        head_affine(blockIdx.x, N2 * groups, aff, true, &bhl, &within);
        pg = within % groups;
        k2 = within / groups;
    }
    float2 *buf_f = lds_big + ci * COLW;             // forward exchanges
    float2 *buf_i = buf_f;                           // inverse cross-wave exchange: same buffer

    float2 tw[P - 1][15];
#pragma unroll
    for (int q = 0; q < P - 1; ++q) {
        const int S = 1 << (4 * (P - 1 - q));
        const int i = tau % S, step = N1 / (16 * S);
#pragma unroll
        for (int u = 1; u < 16; ++u) tw[q][u - 1] = twN1[i * u * step];
    }
    float2 G[16];
    if (MODE == 0) {
        const float2 *gsrc = gp + ((size_t)(bh0 + bhl * g_step) * N2 + k2) * N1;   // g_step 0: one gate for all
#pragma unroll
        for (int j = 0; j < 16; ++j) G[j] = gsrc[j * TPC + tau];
    }

    typedef typename SC::elem_t elem_t;
    elem_t *col = scr + (((size_t)bhl * N2 + k2) * 32 + pg * ppw + ci) * N1;
    // entry j * TPC + tau of a column <-> register j of lane tau, on the way in and on the way out, in every mode
    // (so every access of a wave is a contiguous 512-byte run); see big_position() for the bin such an entry holds
    elem_t nx[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) nx[j] = col[tau + TPC * j];
    // through: see through_store; for launches that have memory to themselves
    auto store_column = [&](elem_t *to, const float2 (&x)[16]) {
        if (through) {
#pragma unroll
            for (int j = 0; j < 16; ++j) through_store(to + tau + TPC * j, SC::put(x[j]));
        } else {
#pragma unroll
            for (int j = 0; j < 16; ++j) to[tau + TPC * j] = SC::put(x[j]);
        }
    };
    for (int c = ci; c < ppw; c += CPI) {
        float2 x[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) x[j] = SC::get(nx[j]);
        if (c + CPI < ppw) {                          // next column's loads fly during this one's passes
            const elem_t *ncol = col + (size_t)CPI * N1;
#pragma unroll
            for (int j = 0; j < 16; ++j) nx[j] = ncol[tau + TPC * j];
        }
        if (MODE != 2) {
            dft<16, false>(x);
#pragma unroll
            for (int u = 1; u < 16; ++u) x[u] = cmul(x[u], tw[0][u - 1]);
            if constexpr (SHFL && !kCross) transpose16(x, tau);
            else exchange<P, 0, 1, kCross>(x, buf_f, tau);
            dft<16, false>(x);
            if constexpr (P == 3) {
#pragma unroll
                for (int u = 1; u < 16; ++u) x[u] = cmul(x[u], tw[1][u - 1]);
                if constexpr (SHFL) transpose16(x, tau);
                else exchange<P, 1, 2, false>(x, buf_f, tau);
                dft<16, false>(x);
            }
        }
        if (MODE == 0) {
#pragma unroll
            for (int j = 0; j < 16; ++j) x[j] = cmul(x[j], G[j]);
        }
        if (MODE == 1) {
            store_column(col, x);
            if (kCross) __syncthreads();              // buf_f is rewritten by the next column
        } else {
            dft<16, true>(x);
            if constexpr (P == 3) {
                if constexpr (SHFL) transpose16(x, tau);
                else exchange<P, 2, 1, false>(x, buf_f, tau);
#pragma unroll
                for (int u = 1; u < 16; ++u) x[u] = cmulc(x[u], tw[1][u - 1]);
                dft<16, true>(x);
            }
            if constexpr (SHFL && !kCross) transpose16(x, tau);
            else exchange<P, 1, 0, kCross>(x, buf_i, tau);
#pragma unroll
            for (int u = 1; u < 16; ++u) x[u] = cmulc(x[u], tw[0][u - 1]);
            dft<16, true>(x);
            store_column(col, x);
            if (kCross) __syncthreads();              // the next column's forward write reuses the buffer
        }
        col += (size_t)CPI * N1;
    }
}

// ------------------------------------------------------------------------------------------
// fused: L = 4096.  A column of this length (32 KB as complex fp32) fits in LDS, so the three kernels above and the
// gate expansion collapse into one kernel and the tensor crosses HBM once each way.  A workgroup of 512 lanes owns
// four adjacent channel pairs of one head (16 or 32 contiguous bytes of every row), 4 x 34 KB of LDS; calls of few heads two pairs, so that more compute units share the arithmetic.
//   pass 0 : lane tau reads the pieces of rows tau + 512 j, j < 8, and transforms the four columns' eight values in registers;
//   core   : 16 lanes own a block of 512 positions of one column, 32 points each: passes of radix 32 and 16, gate and
//            inverse passes without a workgroup barrier (LDS operations of a wave complete in order); after them value u2 of
//            row u1 of block u0 is bin u0 + 8 u1 + 256 u2, and the gate is read there directly, Hermitian extension and the
//            1/L of the inverse transform included;
//   pass 0 again, inverse, from LDS to the rows.
// What bounds it is that its three phases, memory, arithmetic, memory, do not overlap in the one workgroup a compute unit
// holds: with the rows staged in LDS on both sides of three radix-16 passes, two columns at a time, 32 heads of bf16 rows took
// 29.5 us (38 from cold caches) and 512 heads 543, now 27 (34) and 466; fp32 rows, 128 heads 116 -> 107; one head 22 -> 16.5.
// The workgroups of a head (eight, or sixteen of two pairs) share its rows; their ids are 8 apart, so they run on the same XCD and a row is
// fetched into one L2.  (The same construction for L = 8192, two columns per pair, leaves room for only two pairs
// per workgroup, i.e. 8-byte pieces of every row, and measured slower than the three kernels.)
// CL adjacent pairs of a row at the alignment of an element, 16 bytes at most.
template <typename IO, int CL>
struct FusedPiece {
    typedef uint32_t vec_t __attribute__((ext_vector_type(CL * IO::kBytes / 2), aligned(4)));
    vec_t w;
    __device__ __forceinline__ float2 get(int c) const {
        if constexpr (IO::kBytes == 2) return IoBf16::unpack(w[c]);
        else return make_float2(__uint_as_float(w[2 * c]), __uint_as_float(w[2 * c + 1]));
    }
    __device__ __forceinline__ void set(int c, float2 v) {
        if constexpr (IO::kBytes == 2) {
            w[c] = IoBf16::pack(v);
        } else {
            w[2 * c] = __float_as_uint(v.x);
            w[2 * c + 1] = __float_as_uint(v.y);
        }
    }
};

// PP pairs per workgroup of 128 PP lanes; a lane owns CL of them, of 4 / CL taus (a lane of its own for the 32 bytes of four
// pairs of fp32 rows asks for twice the lines: 32 heads 31 -> 35 us).
template <typename IO, int PP, int CL>
__global__ __launch_bounds__(128 * PP, 2) void k_fused(const typename IO::pair_t *__restrict__ v,
                                                       const float2 *__restrict__ g,
                                                       typename IO::pair_t *__restrict__ out,
                                                       const float2 *__restrict__ twL, int H, int BH) {
    typedef FusedPiece<IO, CL> piece_t;
    constexpr int L = 4096, F = L / 2 + 1, COLW = L + L / 16, BLKW = 512 + 512 / 16, WPH = 32 / PP;
    constexpr int NS = PP / CL, NA = 4 / CL, TS = 128 * CL;          // lanes of a row, taus of a lane and their distance
    extern __shared__ float2 lds_fused[];
    const int tid = threadIdx.x;
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int bh = (idx / WPH) * 8 + xcd, part = idx % WPH;
    if (bh >= BH) return;                           // whole workgroup: the grid is padded to 8 heads
    const int b = bh / H, h = bh % H;
    const int t0 = tid / NS, c0 = tid % NS * CL;
    const size_t rs = (size_t)H * 32, off = (((size_t)b * L + t0) * H + h) * 32 + part * PP + c0;
    piece_t row[8 * NA];                             // row t0 + TS m: value j = m / NA of tau = t0 + TS (m % NA)
#pragma unroll
    for (int m = 0; m < 8 * NA; ++m) row[m].w = *reinterpret_cast<const typename piece_t::vec_t *>(v + off + (size_t)(TS * m) * rs);
    const int i = tid & 15, c = (tid >> 4) % PP, u0 = (tid >> 4) / PP;   // core: lane of the block u0 of column c
    float2 tw0[NA][8], tw1[32];
#pragma unroll
    for (int a = 0; a < NA; ++a) {
#pragma unroll
        for (int u = 1; u < 8; ++u) tw0[a][u] = twL[(t0 + TS * a) * u];   // W_4096^(tau u)
    }
#pragma unroll
    for (int u = 1; u < 32; ++u) tw1[u] = twL[8 * i * u];            // W_512^(i u)
    float2 *own = lds_fused + c0 * COLW + t0 + (t0 >> 4);            // position p of a column at p + p / 16
#pragma unroll
    for (int a = 0; a < NA; ++a) {
#pragma unroll
        for (int cc = 0; cc < CL; ++cc) {
            float2 x[8], *w = own + cc * COLW + a * (TS + TS / 16);
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = row[NA * j + a].get(cc);
            dft<8, false>(x);
#pragma unroll
            for (int u = 0; u < 8; ++u) w[u * BLKW] = u == 0 ? x[0] : cmul(x[u], tw0[a][u]);
        }
    }
    const float2 *gh = g + (size_t)bh * F;
    const float scale = 1.0f / (float)L;
    float2 G[16];
    auto load_gate = [&](int u1) {
#pragma unroll
        for (int u2 = 0; u2 < 16; ++u2) {
            const int k = u0 + 8 * u1 + 256 * u2;
            G[u2] = gh[2 * k <= L ? k : L - k];
        }
    };
    load_gate(i);
    __syncthreads();
    float2 *blk = lds_fused + c * COLW + u0 * BLKW;
    {
        float2 x[32];
#pragma unroll
        for (int j = 0; j < 32; ++j) x[j] = blk[i + 17 * j];
        dft<32, false>(x);
#pragma unroll
        for (int u = 0; u < 32; ++u) blk[i + 17 * u] = u == 0 ? x[0] : cmul(x[u], tw1[u]);
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int u1 = i + 16 * q;
        float2 *w = blk + 17 * u1, y[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) y[j] = w[j];
        dft<16, false>(y);
#pragma unroll
        for (int u2 = 0; u2 < 16; ++u2) {
            const int k = u0 + 8 * u1 + 256 * u2;
            float2 gv = make_float2(G[u2].x * scale, G[u2].y * scale);
            if (2 * k > L) gv.y = -gv.y;
            if (k == 0 || 2 * k == L) gv.y = 0.0f;
            y[u2] = cmul(y[u2], gv);
        }
        if (q == 0) load_gate(i + 16);
        dft<16, true>(y);
#pragma unroll
        for (int j = 0; j < 16; ++j) w[j] = y[j];
    }
    __builtin_amdgcn_wave_barrier();
    {
        float2 x[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) x[u] = u == 0 ? blk[i] : cmulc(blk[i + 17 * u], tw1[u]);
        dft<32, true>(x);
#pragma unroll
        for (int j = 0; j < 32; ++j) blk[i + 17 * j] = x[j];
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < NA; ++a) {
#pragma unroll
        for (int cc = 0; cc < CL; ++cc) {
            float2 x[8], *w = own + cc * COLW + a * (TS + TS / 16);
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = u == 0 ? w[0] : cmulc(w[u * BLKW], tw0[a][u]);
            dft<8, true>(x);
#pragma unroll
            for (int j = 0; j < 8; ++j) row[NA * j + a].set(cc, x[j]);
        }
    }
#pragma unroll
    for (int m = 0; m < 8 * NA; ++m) *reinterpret_cast<typename piece_t::vec_t *>(out + off + (size_t)(TS * m) * rs) = row[m].w;
}

// ------------------------------------------------------------------------------------------
// gate_expand: g [BH][L/2+1] -> gp [BH][N2][N1] with gp[bh][k2][r] = ext(g)[k2 + N2 * big_position(r)] / L: entry
// r = j * N1/16 + tau of plane k2 is the bin that register j of lane tau of the big kernel holds after the forward
// passes, and ext = Hermitian extension with real DC and Nyquist bins.  Consecutive bins run over k2 first, so a
// workgroup loads runs of N2 consecutive bins and turns them in LDS into runs of consecutive entries of each plane.
//
// N1 = 256 and 1024, where entry r of a plane is bin k1 = r: a workgroup takes 32 consecutive k1 of one
// head, i.e. 32 N2 consecutive bins, and writes 256-byte runs into each of the N2 planes.  N1 / 32 workgroups per head:
// one workgroup per head kept 32 compute units busy for 8 us with a chain of dependent loads and stores (a ninth
// of the whole call at L = 8192).
__global__ __launch_bounds__(256) void k_gate_expand256(const float2 *__restrict__ g, float2 *__restrict__ gp, int L,
                                                        int N1, int N2) {
    __shared__ float2 tile[32 * 33];
    const int tid = threadIdx.x, bh = blockIdx.y, F = L / 2 + 1, S = N2 + 1;
    const int k1_0 = blockIdx.x * 32, k0 = k1_0 * N2;
    const float scale = 1.0f / (float)L;
    const float2 *gh = g + (size_t)bh * F;
    for (int m = tid; m < 32 * N2; m += 256) {
        const int k = k0 + m;
        float2 val = gh[2 * k <= L ? k : L - k];
        if (2 * k > L) val.y = -val.y;
        if (k == 0 || 2 * k == L) val.y = 0.0f;
        tile[(m / N2) * S + m % N2] = make_float2(val.x * scale, val.y * scale);
    }
    __syncthreads();
    float2 *dst = gp + (size_t)bh * L + k1_0;
    for (int i = tid; i < 32 * N2; i += 256) {
        const int q = i & 31, k2 = i >> 5;
        dst[(size_t)k2 * N1 + q] = tile[q * S + k2];
    }
}

// N1 = 4096, one workgroup per (head, j, b): entries 256 j + 16 b + a, a = 0..15, of every plane are the bins
// k1 = 256 j + 16 a + b, i.e. 16 chunks of N2 consecutive bins, 16 N2 bins apart.  8192 small workgroups at 32 heads
// (two loads and two stores per lane); 512 workgroups that each walked 8192 bins in four dependent rounds took 18 us
// alone, and the expansion sits in front of the first column kernel of a call.
__global__ __launch_bounds__(256) void k_gate_expand4096(const float2 *__restrict__ g, float2 *__restrict__ gp, int L,
                                                         int N2) {
    __shared__ float2 tile[16 * 33];
    const int tid = threadIdx.x, bh = blockIdx.y, F = L / 2 + 1, S = N2 + 1;
    const int j = blockIdx.x >> 4, b = blockIdx.x & 15;
    const float scale = 1.0f / (float)L;
    const float2 *gh = g + (size_t)bh * F;
    for (int m = tid; m < 16 * N2; m += 256) {
        const int a = m / N2, k2 = m % N2;
        const int k = k2 + N2 * (256 * j + 16 * a + b);
        float2 val = gh[2 * k <= L ? k : L - k];
        if (2 * k > L) val.y = -val.y;
        if (k == 0 || 2 * k == L) val.y = 0.0f;
        tile[a * S + k2] = make_float2(val.x * scale, val.y * scale);
    }
    __syncthreads();
    float2 *dst = gp + (size_t)bh * L + 256 * j + 16 * b;
    for (int i = tid; i < 16 * N2; i += 256) {
        const int a = i & 15, k2 = i >> 4;
        dst[(size_t)k2 * 4096 + a] = tile[a * S + k2];
    }
}

// ------------------------------------------------------------------------------------------
bool pow2_split(int L, int *N1, int *N2, int *P) {
    if (L < 256 || L > 131072) return false;
    const bool by256 = (L % 256 == 0) && small_dft_supported(L / 256);
    const bool by4096 = (L % 4096 == 0) && small_dft_supported(L / 4096);
    // the in-register small transform is the cheaper place for stages, so N2 is made as large as 32 allows
    if (by256) { *N1 = 256; *P = 2; }
    else if (by4096) { *N1 = 4096; *P = 3; }
    else return false;
    *N2 = L / *N1;
    return true;
}

template <typename K>
static hipError_t allow_lds(K kernel, size_t bytes) {
    if (bytes <= 48 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <int N2, int TT, typename IO, typename SC>
static hipError_t small_fwd_t(const Pow2Plan &pl, const void *v, void *scr_v, int rows, int H, int bh0,
                              int nbh, hipStream_t st, int aff, float2 *ring, bool just_written, bool two_streams) {
    const size_t lds = (size_t)N2 * TT * TileStride<IO>::value * sizeof(typename IO::pair_t);
    // Scalar addresses for whole transforms, alone, of up to 16 MB and from 56 MB of fp32 rows or 128 MB of bf16 rows on, by the bytes of their
    // scratch.  Between, the denser bursts of loads and stores lose more often than they gain.  Mixer, us, per lane / scalar, fp32 rows: 8
    // heads at 5120 (10 MB) 19.4 / 18.6, 24 (31 MB) 38.3 / 42.3, 48 (63 MB) 76.1 / 74.5; 6 at 20480 (31 MB) 39.7 / 43.5; 2 at 49152 (25 MB)
    // 46.1 / 48.5; bf16 rows: 32 at 7168 (59 MB) 54.6 / 57.6, 48 (88 MB) 77.1 / 81.9, 64 (117 MB) 2 %, 96 (176 MB) -1 %, 32 at 6144 (50 MB) 47.3 / 49.8.  Windows of a cache (fp32 ring) alike: 8 to 16 MB -2 to
    // -3 %, 20 to 50 MB up to +5 %, 100 to 200 MB -1 to -5 %.  Rows that the projection has just written gain nothing above 16 MB and lose
    // there too (layer of fp32 rows, 32 heads at 16384 249 / 254, 2 x 20 at 12288 214 / 218, 20 at 32768 321 / 324).  Beside another launch
    // scalar ones gain at every size (launches of 64 to 100 MB, 32 heads of bf16 rows at 49152 360 / 351, 64 697 / 683, 256 at 12288 656 / 637, at
    // 131072 945 / 938; layer of 20 heads of fp32 rows at 65536 605 / 585, 77 at 24576 709 / 696).
    const size_t bytes = (size_t)nbh * pl.N1 * N2 * 32 * sizeof(typename SC::elem_t);
    const size_t from = (size_t)(std::is_same<IO, IoF32>::value ? 56 : 128) << 20;
    // 24 and 28 fp32 rows take scalar ones at every size (per lane, those keep 4 waves per SIMD instead of 6 or 7; 20 rows 5, 32 rows 3).  Mixer, 5
    // heads at 24576 (31 MB) 45.3 / 43.7, 20 at 6144 (31 MB) 44.8 / 43.2, 5 at 28672 (37 MB) 52.9 / 51.4, one at 98304 46.3 / 45.6; windows, 24
    // heads of 6144 39.1 / 37.0, 20 of 7168 39.2 / 37.5; layer, 8 heads at 24576 100.5 / 98.1, 32 354 / 345, 20 at 28672 277 / 266.  Between 16 and
    // 56 MB 32 rows lose (windows of 6 heads of 32768 50.1 / 52.0), and so do bf16 rows (24 heads at 6144 40.1 / 41.7).
    constexpr bool kEverySize = std::is_same<IO, IoF32>::value && (N2 == 24 || N2 == 28);
    const bool scalar = kEverySize || bytes <= ((size_t)16 << 20) || two_streams || (bytes >= from && !just_written);
    const bool part = ring || rows < pl.N1 * N2;
    auto kern = part || !scalar ? k_small_fwd<N2, TT, IO, SC, true> : k_small_fwd<N2, TT, IO, SC, false>;
    typename SC::elem_t *scr = static_cast<typename SC::elem_t *>(scr_v);
    hipError_t e = allow_lds(kern, lds);
    if (e != hipSuccess) return e;
    constexpr int PW = RowTile<IO>::kPairs;
    const int tiles = pl.N1 / TT * (32 / PW);
    const dim3 grid = aff ? dim3(tiles * nbh) : dim3(tiles, nbh);
    kern<<<grid, dim3(PW * TT), lds, st>>>(
        static_cast<const typename IO::pair_t *>(v), scr, pl.twL, rows, H, pl.N1, bh0, aff, ring);
    return hipGetLastError();
}

template <int N2, int TT, typename IO, typename SC>
static hipError_t small_inv_t(const Pow2Plan &pl, const void *scr_v, void *out, int row0, int out_rows,
                              int H, int bh0, int nbh, hipStream_t st, int ring0, int ring_w, int newest, int aff,
                              float2 *bsum) {
    const size_t lds = (size_t)N2 * TT * TileStride<IO>::value * sizeof(typename IO::pair_t);
    auto kern = k_small_inv<N2, TT, IO, SC>;
    const typename SC::elem_t *scr = static_cast<const typename SC::elem_t *>(scr_v);
    hipError_t e = allow_lds(kern, lds);
    if (e != hipSuccess) return e;
    constexpr int PW = RowTile<IO>::kPairs;
    const int tiles = pl.N1 / TT * (32 / PW);
    const dim3 grid = aff ? dim3(tiles * nbh) : dim3(tiles, nbh);
    kern<<<grid, dim3(PW * TT), lds, st>>>(
        scr, static_cast<typename IO::pair_t *>(out), pl.twL, row0, out_rows, H, pl.N1, bh0, ring0, ring_w, newest, aff,
        bsum);
    return hipGetLastError();
}

#define SPECTRE_N2_CASE(FN, N, ...) \
    case N: return io ? (scr16 ? FN<N, 16, IoBf16, ScrBf16>(__VA_ARGS__) : FN<N, 16, IoBf16, ScrF32>(__VA_ARGS__)) \
                      : FN<N, 16, IoF32, ScrF32>(__VA_ARGS__);
#define SPECTRE_DISPATCH_N2(FN, ...)                                         \
    switch (pl.N2) {                                                         \
        SPECTRE_N2_CASE(FN, 1, __VA_ARGS__) SPECTRE_N2_CASE(FN, 2, __VA_ARGS__) SPECTRE_N2_CASE(FN, 3, __VA_ARGS__)    \
        SPECTRE_N2_CASE(FN, 4, __VA_ARGS__) SPECTRE_N2_CASE(FN, 5, __VA_ARGS__) SPECTRE_N2_CASE(FN, 6, __VA_ARGS__)    \
        SPECTRE_N2_CASE(FN, 7, __VA_ARGS__) SPECTRE_N2_CASE(FN, 8, __VA_ARGS__) SPECTRE_N2_CASE(FN, 10, __VA_ARGS__)   \
        SPECTRE_N2_CASE(FN, 12, __VA_ARGS__) SPECTRE_N2_CASE(FN, 14, __VA_ARGS__) SPECTRE_N2_CASE(FN, 16, __VA_ARGS__) \
        SPECTRE_N2_CASE(FN, 20, __VA_ARGS__) SPECTRE_N2_CASE(FN, 24, __VA_ARGS__) SPECTRE_N2_CASE(FN, 28, __VA_ARGS__) \
        SPECTRE_N2_CASE(FN, 32, __VA_ARGS__)                                 \
        default: return hipErrorInvalidValue;                                \
    }

// 1024-point columns (N = 12288 .. 32768).
#define SPECTRE_FINE_CASE(FN, N, ...) \
    case N: return io ? FN<N, 16, IoBf16, ScrF32Fine>(__VA_ARGS__) : FN<N, 16, IoF32, ScrF32Fine>(__VA_ARGS__);
#define SPECTRE_DISPATCH_FINE(FN, ...)                                       \
    switch (pl.N2) {                                                         \
        SPECTRE_FINE_CASE(FN, 12, __VA_ARGS__) SPECTRE_FINE_CASE(FN, 16, __VA_ARGS__) SPECTRE_FINE_CASE(FN, 20, __VA_ARGS__) \
        SPECTRE_FINE_CASE(FN, 24, __VA_ARGS__) SPECTRE_FINE_CASE(FN, 28, __VA_ARGS__) SPECTRE_FINE_CASE(FN, 32, __VA_ARGS__) \
        default: return hipErrorInvalidValue;                                \
    }

hipError_t launch_small_fwd(const Pow2Plan &pl, int io, const void *v, float2 *scratch, int rows, int H,
                            int bh0, int nbh, hipStream_t st, bool scr16, bool affine, float2 *ring, bool just_written,
                            bool two_streams) {
    if (scr16 && !io) return hipErrorInvalidValue;
    if (affine && nbh % 8 != 0) return hipErrorInvalidValue;
    const int aff = affine ? nbh : 0;
    if (pl.N1 == 1024 && !scr16) SPECTRE_DISPATCH_FINE(small_fwd_t, pl, v, scratch, rows, H, bh0, nbh, st, aff, ring, just_written, two_streams)
    SPECTRE_DISPATCH_N2(small_fwd_t, pl, v, scratch, rows, H, bh0, nbh, st, aff, ring, just_written, two_streams)
}

template <int N2, typename SC>
static hipError_t small_fwd_proj_t(const Pow2Plan &pl, const void *x, const void *wpack, int Hw, float2 *scr, int rows, int H,
                                   int bh0, int nbh, hipStream_t st, int aff) {
    const size_t lds = (size_t)N2 * 16 * TileStride<IoBf16>::value * sizeof(uint32_t);
    auto kern = k_small_fwd_proj<N2, SC>;
    hipError_t e = allow_lds(kern, lds);
    if (e != hipSuccess) return e;
    const dim3 grid = aff ? dim3(pl.N1 / 16 * nbh) : dim3(pl.N1 / 16, nbh);
    kern<<<grid, dim3(512), lds, st>>>(static_cast<const uint32_t *>(x), static_cast<const uint4 *>(wpack), Hw,
                                       scr, pl.twL, rows, H, pl.N1, bh0, aff);
    return hipGetLastError();
}

// bf16 rows.  N2 >= 7: shorter lengths of a plan run in LDS.
hipError_t launch_small_fwd_proj(const Pow2Plan &pl, const void *x, const void *wpack, int Hw, float2 *scratch, int rows,
                                 int H, int bh0, int nbh, hipStream_t st, bool affine) {
    if (affine && nbh % 8 != 0) return hipErrorInvalidValue;
    const int aff = affine ? nbh : 0;
    const bool fine = pl.N1 == 1024;
#define SPECTRE_PROJ(N, SC) return small_fwd_proj_t<N, SC>(pl, x, wpack, Hw, scratch, rows, H, bh0, nbh, st, aff);
#define SPECTRE_PROJ_CASE(N) case N: SPECTRE_PROJ(N, ScrF32)
#define SPECTRE_PROJ_CASE_FINE(N) case N: if (fine) SPECTRE_PROJ(N, ScrF32Fine) SPECTRE_PROJ(N, ScrF32)
    switch (pl.N2) {
        SPECTRE_PROJ_CASE(7) SPECTRE_PROJ_CASE(8) SPECTRE_PROJ_CASE(10) SPECTRE_PROJ_CASE_FINE(12) SPECTRE_PROJ_CASE(14)
        SPECTRE_PROJ_CASE_FINE(16) SPECTRE_PROJ_CASE_FINE(20) SPECTRE_PROJ_CASE_FINE(24) SPECTRE_PROJ_CASE_FINE(28)
        SPECTRE_PROJ_CASE_FINE(32)
        default: return hipErrorInvalidValue;
    }
#undef SPECTRE_PROJ_CASE_FINE
#undef SPECTRE_PROJ_CASE
#undef SPECTRE_PROJ
}

int small_tile_rows(int io) { (void)io; return 16; }

hipError_t launch_small_inv(const Pow2Plan &pl, int io, const float2 *scratch, void *out, int row0,
                            int out_rows, int H, int bh0, int nbh, hipStream_t st, int ring0, int ring_w,
                            int newest, bool scr16, bool affine, float2 *bsum) {
    if (scr16 && !io) return hipErrorInvalidValue;
    if (affine && nbh % 8 != 0) return hipErrorInvalidValue;
    if (bsum && (row0 != 0 || out_rows != pl.L || ring_w > 0)) return hipErrorInvalidValue;   // whole transforms only
    const int aff = affine ? nbh : 0;
    if (pl.N1 == 1024 && !scr16)
        SPECTRE_DISPATCH_FINE(small_inv_t, pl, scratch, out, row0, out_rows, H, bh0, nbh, st, ring0, ring_w, newest, aff, bsum)
    SPECTRE_DISPATCH_N2(small_inv_t, pl, scratch, out, row0, out_rows, H, bh0, nbh, st, ring0, ring_w, newest, aff,
                        bsum)
}

template <int P, int MODE, typename SC = ScrF32, bool SHFL = false>
static hipError_t big_t(const Pow2Plan &pl, float2 *scr_v, const float2 *gp, int bh0, int nbh, bool shared_gate,
                        hipStream_t st, bool through, int aff = 0, bool wide = false) {
    constexpr int N1 = 1 << (4 * P), TPC = N1 / 16, CPI = 256 / TPC, COLW = N1 + N1 / 16;
    const size_t lds = (size_t)CPI * COLW * sizeof(float2);
    // pairs per workgroup; a multiple of CPI dividing 32.  `wide` (a call whose head groups alternate between two
    // streams): 8 columns per workgroup, so that a group's column kernel is fewer workgroups than the chip has room for
    // and the other stream's row kernels run beside it from its first to its last workgroup (-1.5 % at L = 131072; on
    // one stream the longer workgroups cost 2 %)
    const int ppw = (P == 2) ? 16 : (wide ? 8 : 4);
    auto kern = k_big<P, MODE, SC, SHFL>;
    typename SC::elem_t *scr = reinterpret_cast<typename SC::elem_t *>(scr_v);
    hipError_t e = allow_lds(kern, lds);
    if (e != hipSuccess) return e;
    const unsigned grid = (unsigned)nbh * pl.N2 * (32 / ppw);
    const int planes = nbh * pl.N2;                    // remapping needs the plane count to split 8 ways
    kern<<<dim3(grid), dim3(256), lds, st>>>(scr, gp, pl.twN1, pl.N2, ppw, bh0, planes % 8 == 0 ? planes : 0,
                                             shared_gate ? 0 : 1, aff, through);
    return hipGetLastError();
}

hipError_t launch_big(const Pow2Plan &pl, float2 *scratch, const float2 *gp, int bh0, int nbh, int mode,
                      hipStream_t st, bool shared_gate, bool scr16, bool affine, bool two_streams) {
    // through_store where the launch has memory to itself (mixer, us, plain / through: one head of fp32 rows at 16384 32.6 / 30.8, 6 at 6144
    // 27.4 / 24.1, one of bf16 rows at 65536 44.5 / 39.3, 20 of fp32 rows at 6144 46.5 / 45.0, 40 at 16384 186.8 / 184.6; on two streams 512
    // heads of bf16 rows at 3072 347 / 350, 128 at 20480 579 / 587), except columns that the next kernel finds in the L2s: placed by head,
    // 24 to 32 MB (fp32 rows, 32 heads at 3072 31.0 / 32.5, at 3584 35.6 / 37.3, 24 at 5120 40.7 / 42.3; 16 at 5120, 20 MB, 28.3 / 27.6, 32 at
    // 6144, 48 MB, 60.9 / 59.9), of 4096 points 20 to 26 MB (bf16 rows, 2 heads at 49152 41.9 / 43.5, one at 98304 44.4 / 45.8; 2 at 57344, 28
    // MB, 45.2 / 44.5; one at 65536, 16 MB, as above).
    const size_t mb = ((size_t)nbh * pl.N1 * pl.N2 * 32 * (scr16 ? sizeof(uint32_t) : sizeof(float2))) >> 20;
    const bool found = affine ? mb >= 24 && mb <= 32 : pl.P == 3 && mb >= 20 && mb <= 26;
    const bool through = !two_streams && !found;
    const bool shfl = option(SPECTRE_OPT_LANE_SHUFFLES) != 0 && mode == 0 && !scr16;
    if (affine) {                                      // the mixer's forward-gate-inverse pass, fp32 scratch
        if (mode != 0 || scr16 || nbh % 8 != 0) return hipErrorInvalidValue;
        if (pl.P == 2) return shfl ? big_t<2, 0, ScrF32, true>(pl, scratch, gp, bh0, nbh, shared_gate, st, through, nbh)
                                   : big_t<2, 0>(pl, scratch, gp, bh0, nbh, shared_gate, st, through, nbh);
        if (pl.P == 3) return shfl ? big_t<3, 0, ScrF32, true>(pl, scratch, gp, bh0, nbh, shared_gate, st, through, nbh)
                                   : big_t<3, 0>(pl, scratch, gp, bh0, nbh, shared_gate, st, through, nbh);
        return hipErrorInvalidValue;
    }
    if (shfl) {
        if (pl.P == 2) return big_t<2, 0, ScrF32, true>(pl, scratch, gp, bh0, nbh, shared_gate, st, through);
        if (pl.P == 3) return big_t<3, 0, ScrF32, true>(pl, scratch, gp, bh0, nbh, shared_gate, st, through);
        return hipErrorInvalidValue;
    }
    if (scr16) {                                       // the mixer's forward-gate-inverse pass only
        if (mode != 0) return hipErrorInvalidValue;
        if (pl.P == 2) return big_t<2, 0, ScrBf16>(pl, scratch, gp, bh0, nbh, shared_gate, st, through);
        if (pl.P == 3) return big_t<3, 0, ScrBf16>(pl, scratch, gp, bh0, nbh, shared_gate, st, through);
        return hipErrorInvalidValue;
    }
    if (pl.P == 2) {
        if (mode == 0) return big_t<2, 0>(pl, scratch, gp, bh0, nbh, shared_gate, st, through);
        if (mode == 1) return big_t<2, 1>(pl, scratch, gp, bh0, nbh, shared_gate, st, through);
    } else if (pl.P == 3) {
        if (mode == 0) return big_t<3, 0>(pl, scratch, gp, bh0, nbh, shared_gate, st, through, 0, two_streams);
        if (mode == 1) return big_t<3, 1>(pl, scratch, gp, bh0, nbh, shared_gate, st, through);
        if (mode == 2) return big_t<3, 2>(pl, scratch, gp, bh0, nbh, shared_gate, st, through);
    }
    return hipErrorInvalidValue;
}

bool fused_supported(int L) { return L == 4096; }

template <typename IO, int PP, int CL>
static hipError_t fused_t(const void *v, const float2 *g, void *out, const float2 *twL, int H, int BH, hipStream_t st) {
    constexpr int COLW = 4096 + 4096 / 16;
    const size_t lds = (size_t)PP * COLW * sizeof(float2);
    auto kern = k_fused<IO, PP, CL>;
    hipError_t e = allow_lds(kern, lds);
    if (e != hipSuccess) return e;
    const long long grid = (long long)((BH + 7) / 8) * 8 * (32 / PP);   // heads padded to 8
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    kern<<<dim3((unsigned)grid), dim3(128 * PP), lds, st>>>(static_cast<const typename IO::pair_t *>(v), g,
                                                            static_cast<typename IO::pair_t *>(out), twL, H, BH);
    return hipGetLastError();
}

hipError_t launch_fused(int io, const void *v, const float2 *g, void *out, const float2 *tw4096, int L, int H, int BH,
                        hipStream_t st) {
    if (!fused_supported(L)) return hipErrorInvalidValue;
    // Two pairs per workgroup while four would leave half the compute units without one (bf16, 1, 8, 16, 20 heads with four /
    // two / one pairs 19.5 / 16.5 / 17.5, 20.6 / 17.3 / 18.1, 22.5 / 20.5 / 28.1, 24.2 / 29.3 / 38.5 us).
#define SPECTRE_FUSED(IO, PP, CL) return fused_t<IO, PP, CL>(v, g, out, tw4096, H, BH, st)
    if (BH <= 16) { if (io) SPECTRE_FUSED(IoBf16, 2, 2); SPECTRE_FUSED(IoF32, 2, 2); }
    if (io) SPECTRE_FUSED(IoBf16, 4, 4);
    SPECTRE_FUSED(IoF32, 4, 2);
#undef SPECTRE_FUSED
}

hipError_t launch_gate_expand(const Pow2Plan &pl, const float2 *g, float2 *gp, int BH, hipStream_t st) {
    if (pl.P != 2 && pl.P != 3 && !(pl.P == 0 && pl.N1 == 1024)) return hipErrorInvalidValue;
    for (int bh0 = 0; bh0 < BH; bh0 += 65535) {         // grid.y limit
        const int n = (BH - bh0 < 65535) ? BH - bh0 : 65535;
        const int F = pl.L / 2 + 1;
        if (pl.P != 3)
            k_gate_expand256<<<dim3(pl.N1 / 32, n), dim3(256), 0, st>>>(g + (size_t)bh0 * F, gp + (size_t)bh0 * pl.L, pl.L, pl.N1,
                                                                        pl.N2);
        else
            k_gate_expand4096<<<dim3(256, n), dim3(256), 0, st>>>(g + (size_t)bh0 * F, gp + (size_t)bh0 * pl.L, pl.L, pl.N2);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Loads this translation unit's code object (the runtime loads them on first use): called by spectre_prepare so
// that no compute call is the first to touch it.
hipError_t load_kernels_mix_pow2() {
    hipFuncAttributes a;
    return hipFuncGetAttributes(&a, reinterpret_cast<const void *>(k_gate_expand256));
}

}  // namespace spectre
