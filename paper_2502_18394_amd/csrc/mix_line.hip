// Whole columns on one compute unit: the mixing layer for bf16 rows at L = 8192 and 16384 (Sec. 3.2 steps 2-4).
//
// The four-step route exchanges a column twice through memory as fp32: 8 bytes per channel pair and position each way,
// 40 with the rows.  A column of these lengths fits in LDS as fp32 (70 and 139 KB), so here only the bf16 rows
// themselves are turned, 4 bytes each way:
//   k_line_turn<in>  : rows [L][pairs] -> lines, one per channel pair, in the order the column kernel's lanes read; its
//                      first workgroups lay the gate out in the order of the column kernel's registers
//   k_line           : a line at a time: forward transform, gate, inverse transform, in place
//   k_line_turn<out> : lines -> rows
// 24 bytes per pair and position; the column kernel is bound by its vector arithmetic (about 90 instructions per point).
// Measured: L = 8192 66 -> 61 us for 32 heads, 241 -> 189 us for 128; L = 16384 132 -> 113 us for 32 heads, 253 -> 206 us
// for 64.  As many heads go through together as the scratch holds (line_group_heads; groups of 32 for 128 heads at
// L = 8192: 216 us).  Rows of fp32 would move the same 48 bytes either way and are slower here (78 -> 86 us), so they stay
// on the four-step route, as do lengths with an odd factor, whose passes would leave lanes idle.
#include "mix_line.h"

#include "fft_regs.h"
#include "internal.h"
#include "scratch_elem.h"

namespace spectre {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
// Rows lie on the 4-byte boundary of a channel pair and are read and written in 16-byte pieces all the same, so that a
// head's result does not depend on where its tensor starts.
typedef unsigned int u32x4_pair_t __attribute__((ext_vector_type(4), aligned(4)));

// A line's element t = tau + NT j (NT = lanes of the column kernel) sits at (j / 4) 4 NT + 4 tau + j % 4: four
// consecutive values of a lane's j are one 16-byte word.
constexpr int kVW = 4, kTurnRows = 32 * kVW;

// All workgroups of head 8 s + x on XCD x (ids are dealt round-robin), so that its lines and its gate meet one L2.
__device__ __forceinline__ void line_unit(int id, int per_head, int *bhl, int *within) {
    const int xcd = id & 7, idx = id >> 3, slot = idx / per_head;
    *within = idx - slot * per_head;
    *bhl = 8 * slot + xcd;
}

// A workgroup turns 4 j x 32 tau rows of one head, 128 bytes each, through LDS: 512-byte runs on the side of the lines.
// grid: nexp gate blocks (IN only), then the tiles of 8 ceil(nbh / 8) heads.
// ONCE: the rows pass the caches by; rows off a 16-byte boundary share lines with their neighbours and do not (L = 16384, 128
// heads 528 instead of 600 us).  THROUGH: see line_t.
template <bool IN, bool ONCE, bool THROUGH>
__global__ __launch_bounds__(256) void k_line_turn(const uint32_t *__restrict__ rows_in, uint32_t *__restrict__ rows_out,
                                                   uint32_t *__restrict__ lines, int L, int NT, int H, int bh0, int nbh,
                                                   const float2 *__restrict__ g, float2 *__restrict__ gp, int R0, int R1,
                                                   int nexp) {
    constexpr int S = 33;
    __shared__ uint32_t tile[kTurnRows * S];
    const int tid = threadIdx.x;
    int id = blockIdx.x;
    if (IN) {
        if (id < nexp) {                       // gp[bh][r][tau]: bin of register r of lane tau in k_line's last pass
            const int per = L / 256, bhl = id / per, e = (id % per) * 256 + tid;
            const int r = e / NT, tau = e % NT, m = (tau & 15) + 16 * (r / 16);
            const int k = (tau >> 4) + R1 * (m / R1) + R0 * (m % R1) + R0 * R1 * (r % 16);
            const float2 val = g[(size_t)(bh0 + bhl) * (L / 2 + 1) + (2 * k <= L ? k : L - k)];
            const float scale = 1.0f / (float)L;
            // Hermitian extension; only the real parts count at DC and Nyquist
            const float im = (k == 0 || 2 * k == L) ? 0.0f : 2 * k > L ? -val.y : val.y;
            gp[(size_t)bhl * L + e] = make_float2(val.x * scale, im * scale);
            return;
        }
        id -= nexp;
    }
    int bhl, t;
    line_unit(id, L / kTurnRows, &bhl, &t);
    if (bhl >= nbh) return;                    // whole workgroup: heads are padded to 8
    const int tau0 = (t % (NT / 32)) * 32, j0 = (t / (NT / 32)) * kVW;
    const int bh = bh0 + bhl, b = bh / H, h = bh % H;
    uint32_t *head = lines + (size_t)bhl * 32 * L, *line = head + (size_t)j0 * NT + (size_t)tau0 * kVW;
    const int tl = tid & 31, p0 = tid >> 5;    // line side: tau0 + tl of pairs p0 + 8 i
    const int piece = tid & 7, r0 = tid >> 3;  // row side: 16 bytes (four pairs) of rows r0 + 32 i
    const size_t row0 = (((size_t)b * L + tau0 + r0 + (size_t)NT * j0) * H + h) * 32 + 4 * piece, rstep = (size_t)NT * H * 32;
    u32x4_t w[4];
    if (IN) {
        const u32x4_pair_t *src = reinterpret_cast<const u32x4_pair_t *>(rows_in + row0);
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = ONCE ? __builtin_nontemporal_load(src + i * (rstep / 4)) : src[i * (rstep / 4)];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int c = 0; c < 4; ++c) tile[(r0 + 32 * i) * S + 4 * piece + c] = w[i][c];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int c = 0; c < 4; ++c) w[i][c] = tile[(c * 32 + tl) * S + p0 + 8 * i];
            if (THROUGH) through_store16(head, 128u * L, 4u * ((p0 + 8 * i) * L + j0 * NT + (tau0 + tl) * kVW), w[i]);
            else *(reinterpret_cast<u32x4_t *>(line + (size_t)(p0 + 8 * i) * L) + tl) = w[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = *(reinterpret_cast<const u32x4_t *>(line + (size_t)(p0 + 8 * i) * L) + tl);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int c = 0; c < 4; ++c) tile[(c * 32 + tl) * S + p0 + 8 * i] = w[i][c];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int c = 0; c < 4; ++c) w[i][c] = tile[(r0 + 32 * i) * S + 4 * piece + c];
        }
        u32x4_pair_t *dst = reinterpret_cast<u32x4_pair_t *>(rows_out + row0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (ONCE) __builtin_nontemporal_store(w[i], dst + i * (rstep / 4));
            else dst[i * (rstep / 4)] = w[i];
        }
    }
}

// L = R0 NT points, NT = 16 R1 lanes, R0 points per lane; decimation in frequency as in k_big (mix_pow2.hip), radices R0,
// R1, 16.  Pass 0: lane tau owns positions tau + NT u.  Passes 1 and 2 stay inside the blocks of NT positions that a
// group of 16 lanes owns (blocks tau / 16 + R1 q), so only the exchange between passes 0 and 1 crosses waves.  After pass
// 2 the 16 values of position block blk, row s of 16 are the bins blk + R0 s + R0 R1 u.
// The launch is as wide as the chip and a workgroup takes its share of the XCD's lines, the next one's loads in flight during
// the passes.  Workgroups of one, two or four lines ended in a ragged round, and with the head and the number of lines as
// arguments 24 registers spilled at L = 16384: 32, 40, 64, 65, 100, 128 and 256 heads took 126, 190, 233, 285, 395, 510 and
// 947 us (the four-step route 132, 162, 253, 270, 380, 478 and 935), now 113, 137, 206, 218, 315, 408 and 794; L = 8192,
// 32, 100, 128 and 256 heads 61, 168, 187 and 402 us (66, 175, 241 and 464), now 61, 150, 189 and 374.
// The factors are reloaded (five values per layer, from L1) where they are used: kept in registers over the loop, with the
// products the compiler forms from them, they spilled.
template <int R0, int R1, bool THROUGH>
__global__ __launch_bounds__(16 * R1, 2) void k_line(uint32_t *__restrict__ lines, const float2 *__restrict__ gp,
                                                     const float2 *__restrict__ twL, int nbh) {
    constexpr int NT = 16 * R1, L = R0 * NT, Q1 = R0 / R1, Q2 = R0 / 16, S0 = NT + NT / 16;   // LDS position p + p / 16
    extern __shared__ float2 lds_line[];
    const int tau = threadIdx.x, i = tau & 15, grp = tau >> 4;
    const int xcd = blockIdx.x & 7;
    const LineShare mine = line_share(xcd, blockIdx.x >> 3, gridDim.x >> 3, nbh);
    const int n0 = mine.first, n1 = n0 + mine.count;
    if (n0 == n1) return;                                            // whole workgroup
    auto line_of = [&](int n) {
        return reinterpret_cast<u32x4_t *>(lines + ((size_t)(8 * (n >> 5) + xcd) * 32 + (n & 31)) * L) + tau;
    };
    u32x4_t raw[R0 / kVW];
#pragma unroll
    for (int e = 0; e < R0 / kVW; ++e) raw[e] = line_of(n0)[e * NT];
    float2 *b0 = lds_line + tau + (tau >> 4);
    float2 *b1 = lds_line + grp * S0 + i;
#pragma unroll 1
    for (int n = n0; n < n1; ++n) {
        const float2 *gsrc = gp + (size_t)(8 * (n >> 5) + xcd) * L + tau;
        const float2 *tl = twL;
        asm volatile("" : "+s"(tl));                                 // a new value to the compiler in every round
        float2 x[R0];
#pragma unroll
        for (int j = 0; j < R0; ++j) x[j] = IoBf16::unpack(raw[j / kVW][j % kVW]);
        if (n + 1 < n1) {
#pragma unroll
            for (int j = 0; j < R0 / kVW; ++j) raw[j] = line_of(n + 1)[j * NT];
        }
        {
            const SmallTwiddles<R0> tw(tl, tau);
            small_dft<R0, false>(x);
#pragma unroll
            for (int u = 0; u < R0; ++u) b0[u * S0] = u == 0 ? x[0] : cmul(x[u], tw(u));
        }
        float2 G[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) G[r] = gsrc[r * NT];
        {
            SmallTwiddles<R1> tw(tl, R0 * i);
            __syncthreads();
#pragma unroll 1
            for (int q = 0; q < Q1; ++q) {
                tw.pin();
                float2 *w = b1 + R1 * q * S0, y[R1];
#pragma unroll
                for (int j = 0; j < R1; ++j) y[j] = w[17 * j];
                small_dft<R1, false>(y);
#pragma unroll
                for (int u = 0; u < R1; ++u) w[17 * u] = u == 0 ? y[0] : cmul(y[u], tw(u));
            }
        }
        __builtin_amdgcn_wave_barrier();                             // LDS operations of a wave complete in order
#pragma unroll 1
        for (int q = 0; q < Q2; ++q) {
            const int m = i + 16 * q;
            float2 *w = lds_line + (grp + R1 * (m / R1)) * S0 + 17 * (m % R1), y[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) y[j] = w[j];
            dft<16, false>(y);
#pragma unroll
            for (int u = 0; u < 16; ++u) y[u] = cmul(y[u], G[u]);
            if (q + 1 < Q2) {
#pragma unroll
                for (int r = 0; r < 16; ++r) G[r] = gsrc[(16 * (q + 1) + r) * NT];
            }
            dft<16, true>(y);
#pragma unroll
            for (int j = 0; j < 16; ++j) w[j] = y[j];
        }
        __builtin_amdgcn_wave_barrier();
        asm volatile("" : "+s"(tl));
        {
            SmallTwiddles<R1> tw(tl, R0 * i);
#pragma unroll 1
            for (int q = 0; q < Q1; ++q) {
                tw.pin();
                float2 *w = b1 + R1 * q * S0, y[R1];
#pragma unroll
                for (int u = 0; u < R1; ++u) y[u] = u == 0 ? w[0] : cmulc(w[17 * u], tw(u));
                small_dft<R1, true>(y);
#pragma unroll
                for (int j = 0; j < R1; ++j) w[17 * j] = y[j];
            }
        }
        const SmallTwiddles<R0> tw(tl, tau);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < R0; ++u) x[u] = u == 0 ? b0[0] : cmulc(b0[u * S0], tw(u));
        small_dft<R0, true>(x);
#pragma unroll
        for (int j = 0; j < R0 / kVW; ++j) {
            u32x4_t o;
#pragma unroll
            for (int e = 0; e < kVW; ++e) o[e] = IoBf16::pack(x[kVW * j + e]);
            if (THROUGH) through_store16(lines + ((size_t)(8 * (n >> 5) + xcd) * 32 + (n & 31)) * L, 4u * L, 16u * (j * NT + tau), o);
            else line_of(n)[j * NT] = o;
        }
        if (n + 1 < n1) __syncthreads();                             // the next line's pass 0 writes what is read above
    }
}

// ------------------------------------------------------------------------------------------
bool line_supported(int L, int io) { return io == 1 && (L == 8192 || L == 16384); }

// THROUGH: the lines are written through the L2 both times (through_store) where they are more than the eight L2s hold, 32 MB; fewer
// lines stay there for the next kernel.  us, plain / through: L = 8192, 6 heads 19.6 / 20.2, 16 28.1 / 29.1, 24 (25 MB) 42.1 / 42.9, 32
// (34 MB) 55.4 / 53.5, 64 98 / 93; L = 16384, 6 heads 27.9 / 30.5, 8 29.8 / 31.7, 12 (25 MB) 44.5 / 44.9, 16 (34 MB) 58.5 / 56.9.
template <int R0, int R1, bool THROUGH>
static hipError_t line_t(const uint32_t *v, const float2 *g, uint32_t *out, float2 *gp, uint32_t *lines, const float2 *twL,
                         int H, int bh0, int nbh, hipStream_t st) {
    constexpr int NT = 16 * R1, L = R0 * NT;
    const int heads8 = (nbh + 7) / 8 * 8, tiles = L / kTurnRows * heads8, nexp = nbh * (L / 256);
    const auto turn_in = reinterpret_cast<uintptr_t>(v) & 15 ? k_line_turn<true, false, THROUGH> : k_line_turn<true, true, THROUGH>;
    turn_in<<<nexp + tiles, 256, 0, st>>>(v, nullptr, lines, L, NT, H, bh0, nbh, g, gp, R0, R1, nexp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t lds = (size_t)R0 * (NT + NT / 16) * sizeof(float2);
    auto kern = k_line<R0, R1, THROUGH>;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    kern<<<8 * line_workgroups(L, nbh), NT, lds, st>>>(lines, gp, twL, nbh);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const auto turn_out = reinterpret_cast<uintptr_t>(out) & 15 ? k_line_turn<false, false, false> : k_line_turn<false, true, false>;
    turn_out<<<tiles, 256, 0, st>>>(nullptr, out, lines, L, NT, H, bh0, nbh, nullptr, nullptr, R0, R1, 0);
    return hipGetLastError();
}

hipError_t launch_mix_line(const void *v, const float2 *g, void *out, float2 *gp, void *lines, const float2 *twL, int L,
                           int H, int bh0, int nbh, hipStream_t st) {
    const uint32_t *vp = static_cast<const uint32_t *>(v);
    uint32_t *op = static_cast<uint32_t *>(out), *lp = static_cast<uint32_t *>(lines);
    const bool through = (size_t)nbh * L * 32 * sizeof(uint32_t) >= kL2Bytes;
    if (L == 8192) return (through ? line_t<32, 16, true> : line_t<32, 16, false>)(vp, g, op, gp, lp, twL, H, bh0, nbh, st);
    if (L == 16384) return (through ? line_t<32, 32, true> : line_t<32, 32, false>)(vp, g, op, gp, lp, twL, H, bh0, nbh, st);
    return hipErrorInvalidValue;
}

// Loads this translation unit's code object (the runtime loads them on first use): called by spectre_prepare so
// that no compute call is the first to touch it.
hipError_t load_kernels_mix_line() {
    hipFuncAttributes a;
    return hipFuncGetAttributes(&a, reinterpret_cast<const void *>(&k_line_turn<true, true, true>));
}

}  // namespace spectre
