// Content-adaptive spectral gate (Sec. 3.2 step 3a, 3c; positional phase of Sec. 3.5;
// Algorithm 1's decode gate) for gfx950.
//
//   pool    : sum of the query rows over positions, accumulated in fp64 in a fixed order (short sequences: one kernel
//             for everything, k_gate_small)
//   prep    : x = inv_count * sum;  qbar = LayerNorm(x);  hid = GELU(qbar W1 + b1); inside `out` where that has few workgroups
//   out     : u = W2 hid + b2 on the matrix cores (fp32 MFMA, v_mfma_f32_4x4x1_16B_f32: 64
//             output reals x 4 rows per instruction), with bias and modReLU in the epilogue
//   phase   : the positional phase, when a position is given: in the epilogue of `out`, or a separate pass over g (k_gate_small, the
//             Toeplitz update, very many tiles)
#include "gate.h"

#include "common.h"
#include "fold16.h"

namespace spectre {

typedef float floatx16 __attribute__((ext_vector_type(16)));

// ------------------------------------------------------------------------------------------
// pool, stage 1: grid (ceil(pairs_per_row/256), nchunks, B).  Lane = one channel pair of the
// [H*d] row; the workgroup sums rows [chunk*R, min(L, chunk*R+R)) in order.
template <typename IO>
__global__ __launch_bounds__(256) void k_pool_partial(const typename IO::pair_t *__restrict__ q,
                                                      double2 *__restrict__ partial, int L, int ppr,
                                                      int R, int nchunks) {
    const int pi = blockIdx.x * 256 + threadIdx.x;
    if (pi >= ppr) return;
    const int chunk = blockIdx.y, b = blockIdx.z;
    const int l0 = chunk * R, l1 = min(L, l0 + R);
    const typename IO::pair_t *src = q + ((size_t)b * L + l0) * ppr + pi;
    double sx = 0.0, sy = 0.0;
    int l = l0;
    for (; l + 4 <= l1; l += 4) {
        float2 a0 = IO::unpack(src[0]), a1 = IO::unpack(src[(size_t)ppr]);
        float2 a2 = IO::unpack(src[2 * (size_t)ppr]), a3 = IO::unpack(src[3 * (size_t)ppr]);
        sx += (double)a0.x; sy += (double)a0.y;
        sx += (double)a1.x; sy += (double)a1.y;
        sx += (double)a2.x; sy += (double)a2.y;
        sx += (double)a3.x; sy += (double)a3.y;
        src += 4 * (size_t)ppr;
    }
    for (; l < l1; ++l) {
        float2 a = IO::unpack(src[0]);
        sx += (double)a.x; sy += (double)a.y;
        src += ppr;
    }
    partial[((size_t)b * nchunks + chunk) * ppr + pi] = make_double2(sx, sy);
}

// The same sums with 16-byte loads: a lane owns four adjacent bf16 pairs or two adjacent fp32 pairs, eight rows in
// flight (the order of additions per channel is the row order, as above).  Needs the pairs per row to be a multiple
// of that and a 16-byte aligned tensor.  ppv = row length in 16-byte pieces.
template <bool BF16>
__global__ __launch_bounds__(256) void k_pool_partial_x16(const uint4 *__restrict__ q, double *__restrict__ partial,
                                                          int L, int ppv, int R, int nchunks) {
    constexpr int NCH = BF16 ? 8 : 4;                 // channels per 16 bytes
    const int pi = blockIdx.x * 256 + threadIdx.x;
    if (pi >= ppv) return;
    const int chunk = blockIdx.y, b = blockIdx.z;
    const int l0 = chunk * R, l1 = min(L, l0 + R);
    const uint4 *src = q + ((size_t)b * L + l0) * ppv + pi;
    double s[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) s[i] = 0.0;
    auto add = [&](const uint4 w) {
        if (BF16) {
            const float2 a = IoBf16::unpack(w.x), c = IoBf16::unpack(w.y), e = IoBf16::unpack(w.z), f = IoBf16::unpack(w.w);
            s[0] += (double)a.x; s[1] += (double)a.y; s[2] += (double)c.x; s[3] += (double)c.y;
            s[4 % NCH] += (double)e.x; s[5 % NCH] += (double)e.y; s[6 % NCH] += (double)f.x; s[7 % NCH] += (double)f.y;
        } else {
            s[0] += (double)__uint_as_float(w.x); s[1] += (double)__uint_as_float(w.y);
            s[2] += (double)__uint_as_float(w.z); s[3] += (double)__uint_as_float(w.w);
        }
    };
    typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
    int l = l0;
    for (; l + 8 <= l1; l += 8) {
        uint4 w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(src + (size_t)i * ppv));
            w[i] = make_uint4(t.x, t.y, t.z, t.w);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) add(w[i]);
        src += 8 * (size_t)ppv;
    }
    for (; l < l1; ++l) {
        add(*src);
        src += ppv;
    }
    double *dst = partial + ((size_t)b * nchunks + chunk) * ((size_t)NCH * ppv) + (size_t)NCH * pi;
#pragma unroll
    for (int i = 0; i < NCH; i += 2) *reinterpret_cast<double2 *>(dst + i) = make_double2(s[i], s[i + 1]);
}

// The same for short sequences of rows of whole 128-byte lines: 512 lanes take COLS adjacent pieces of 512 / COLS rows at a
// time, so that a chunk of the partial sums stands for 64 to 256 rows where whole rows on so many compute units leave 16, and
// what adds the chunks up reads a sixteenth (32 heads of 8192 bf16 rows: 32 chunks for 512, and with the hidden layer inside
// the output layer's launch the gate takes 22 instead of 30 us).
template <bool BF16, int COLS>
__global__ __launch_bounds__(512) void k_pool_deep(const void *__restrict__ q, double *__restrict__ partial, int L, int ppv,
                                                   int R, int nchunks) {
    constexpr int NCH = BF16 ? 8 : 4, GRP = 512 / COLS, kU = 8;          // channels per 16 bytes, rows at a time, in flight
    typedef unsigned int u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));   // the same sums at any alignment
    __shared__ double red[8][COLS * NCH];
    const int tid = threadIdx.x, col = tid % COLS, grp = tid / COLS;
    const int chunk = blockIdx.y, b = blockIdx.z, l1 = min(L, (chunk + 1) * R);
    int l = chunk * R + grp;
    const u32x4_a4 *src = static_cast<const u32x4_a4 *>(q) + ((size_t)b * L + l) * ppv + (size_t)blockIdx.x * COLS + col;
    double s[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) s[i] = 0.0;
    for (; l < l1; l += GRP * kU) {
        u32x4_a4 w[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            w[u] = u32x4_a4{0, 0, 0, 0};
            if (l + GRP * u < l1) w[u] = __builtin_nontemporal_load(src + (size_t)(GRP * u) * ppv);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (BF16) {
                    const float2 v = IoBf16::unpack(w[u][i]);
                    s[(2 * i) % NCH] += (double)v.x;
                    s[(2 * i + 1) % NCH] += (double)v.y;
                } else {
                    s[i] += (double)__uint_as_float(w[u][i]);
                }
            }
        }
        src += (size_t)(GRP * kU) * ppv;
    }
#pragma unroll
    for (int off = COLS; off < 64; off <<= 1) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) s[c] += __shfl_xor(s[c], off);
    }
    if ((tid & 63) < COLS) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) red[tid >> 6][NCH * col + c] = s[c];
    }
    __syncthreads();
    if (tid < COLS * NCH) {
        double t = red[0][tid];
#pragma unroll
        for (int r = 1; r < 8; ++r) t += red[r][tid];
        partial[(((size_t)b * nchunks + chunk) * ppv + (size_t)blockIdx.x * COLS) * NCH + tid] = t;
    }
}

// pool, stage 2: sum_q[b][ch] = sum over chunks.  grid (row/32, B); 256 lanes = 32 channels x 8
// chunk groups; group r adds chunks r, r+8, ... in order, the 8 group sums are then added in order.
__global__ __launch_bounds__(256) void k_pool_final(const double *__restrict__ partial,
                                                    double *__restrict__ sum_q, int row, int nchunks, int accumulate) {
    __shared__ double red[8][32];
    const int lane = threadIdx.x & 31, grp = threadIdx.x >> 5;
    const int ch = blockIdx.x * 32 + lane, b = blockIdx.y;
    double s = 0.0;
    if (ch < row) {
        const double *src = partial + (size_t)b * nchunks * row + ch;
        int c = grp;
        for (; c + 56 < nchunks; c += 64) {       // eight loads in flight, added in the same order
            double t[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) t[i] = src[(size_t)(c + 8 * i) * row];
#pragma unroll
            for (int i = 0; i < 8; ++i) s += t[i];
        }
        for (; c < nchunks; c += 8) s += src[(size_t)c * row];
    }
    red[grp][lane] = s;
    __syncthreads();
    if (grp == 0 && ch < row) {
        double t = red[0][lane];
#pragma unroll
        for (int r = 1; r < 8; ++r) t += red[r][lane];
        sum_q[(size_t)b * row + ch] = accumulate ? sum_q[(size_t)b * row + ch] + t : t;
    }
}

// ------------------------------------------------------------------------------------------
// prep: one workgroup of NT = 512 lanes, or 256 where there are many, per (b, h), from the pooling pass's partial sums to the hidden layer: the chunks'
// sums (fp64, fixed order), optionally times W_q (the sums are then those of X: pooling commutes with the projection),
// LayerNorm with fp64 statistics, and the small d x d_g product on the vector units, its d terms split over lane groups
// (fixed split, partial sums added in group order).  sum_q != nullptr: the pooled query is also stored.
// One dependent launch where there were two (three with W_q): 5 us each at any size.
template <int NT>
__device__ __forceinline__ double block_sum(double x, double *red, int lane, int wave) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
    if (lane == 0) red[wave] = x;
    __syncthreads();
    const double s = (red[0] + red[1]) + (red[2] + red[3]);
    return NT == 256 ? s : s + ((red[4] + red[5]) + (red[6] + red[7]));
}

template <int NT>
__global__ __launch_bounds__(NT) void k_gate_prep(const double *__restrict__ partial, int nchunks,
                                                  const float *__restrict__ Wq, int Hw, double *__restrict__ sum_q,
                                                  double inv_count, GateDev P, float *__restrict__ hid, int H) {
    constexpr int NW = NT / 64, IPW = 64 / NW;                       // waves; inputs of a 64 x 64 product per wave
    __shared__ double2 acc[NT];
    __shared__ double xs[256], red[2 * NW];
    __shared__ float qbar[256], part[NT];
    const int bh = blockIdx.x, b = bh / H, h = bh % H, hp = (P.Hg == 1) ? 0 : h, d = P.d, dg = P.d_g;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the weights' latency passes behind the sums (the usual widths only; any other is read where it is used)
    const bool usual = d == 64 && dg == 64;
    float w1[IPW], wq[IPW], gam = 0.f, bet = 0.f, b1 = 0.f;
    if (usual) {
#pragma unroll
        for (int i = 0; i < IPW; ++i) w1[i] = P.W1[(size_t)hp * 4096 + (IPW * wave + i) * 64 + lane];
        gam = P.ln_gamma[hp * 64 + lane];
        bet = P.ln_beta[hp * 64 + lane];
        b1 = P.b1[hp * 64 + lane];
    }
    if (Wq) {
#pragma unroll
        for (int i = 0; i < IPW; ++i) wq[i] = Wq[(size_t)((Hw == 1) ? 0 : h) * 4096 + (IPW * wave + i) * 64 + lane];
    }
    const int np = d / 2, ng = NT / np, p = tid % np, grp = tid / np;
    double2 s = make_double2(0.0, 0.0);
    if (grp < ng) {
        const size_t row = (size_t)H * np;
        const f64x2_elem_t *src = reinterpret_cast<const f64x2_elem_t *>(partial) + (size_t)b * nchunks * row + (size_t)h * np + p;
        int c = grp;
        for (; c + 7 * ng < nchunks; c += 8 * ng) {      // eight loads in flight, added in chunk order
            f64x2_elem_t t[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) t[i] = src[(size_t)(c + i * ng) * row];
#pragma unroll
            for (int i = 0; i < 8; ++i) { s.x += t[i].x; s.y += t[i].y; }
        }
        for (; c < nchunks; c += ng) {
            const f64x2_elem_t t = src[(size_t)c * row];
            s.x += t.x;
            s.y += t.y;
        }
    }
    acc[tid] = s;
    __syncthreads();
    if (tid < np) {
        double2 t = acc[tid];
        for (int r = 1; r < ng && r < nchunks; ++r) { t.x += acc[r * np + tid].x; t.y += acc[r * np + tid].y; }
        xs[2 * tid] = t.x;
        xs[2 * tid + 1] = t.y;
    }
    __syncthreads();
    if (Wq) {                                            // d = 64: lane (j, seg) takes IPW of the 64 terms of output j
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < IPW; ++i) t += xs[IPW * wave + i] * (double)wq[i];
        double *a = reinterpret_cast<double *>(acc);
        a[tid] = t;
        __syncthreads();
        if (tid < 64) {
            double q = a[tid];
#pragma unroll
            for (int r = 1; r < NW; ++r) q += a[64 * r + tid];
            xs[tid] = q;
        }
        __syncthreads();
    }
    if (sum_q && tid < d) sum_q[(size_t)bh * d + tid] = xs[tid];
    if (usual) {                                         // every wave normalises for itself (lane = channel)
        const double x = inv_count * xs[lane];
        const double dev = x - wave_sum(x) / 64;
        const double rstd = 1.0 / sqrt(wave_sum(dev * dev) / 64 + (double)P.ln_eps);
        const float qv = (float)((double)gam * dev * rstd + (double)bet);
        float a = 0.f;
#pragma unroll
        for (int i = 0; i < IPW; ++i) a = fmaf(__shfl(qv, IPW * wave + i), w1[i], a);
        part[tid] = a;
        __syncthreads();
        if (tid < 64) {
            float t = b1;
#pragma unroll
            for (int q = 0; q < NW; ++q) t += part[64 * q + tid];
            hid[(size_t)bh * 64 + tid] = 0.5f * t * (1.0f + erff(t * 0.70710678118654752440f));
        }
        return;
    }
    const double x = (tid < d) ? inv_count * xs[tid] : 0.0;
    const double mean = block_sum<NT>(x, red, lane, wave) / d;
    const double dev = (tid < d) ? x - mean : 0.0;
    const double var = block_sum<NT>(dev * dev, red + NW, lane, wave) / d;
    const double rstd = 1.0 / sqrt(var + (double)P.ln_eps);
    if (tid < d) qbar[tid] = (float)((double)P.ln_gamma[hp * d + tid] * dev * rstd + (double)P.ln_beta[hp * d + tid]);
    __syncthreads();
    const int nseg = NT / (dg <= 64 ? 64 : dg <= 128 ? 128 : 256), cols = NT / nseg;
    const int jcol = tid % cols, seg = tid / cols;
    const int dseg = (d + nseg - 1) / nseg, i0 = seg * dseg, i1 = (i0 + dseg < d) ? i0 + dseg : d;
    float a = 0.f;
    if (jcol < dg) {
        const float *w = P.W1 + (size_t)hp * d * dg + jcol;
#pragma unroll 8
        for (int i = i0; i < i1; ++i) a = fmaf(qbar[i], w[(size_t)i * dg], a);
    }
    part[tid] = a;
    __syncthreads();
    if (tid < dg) {
        float t = P.b1[hp * dg + tid];
        for (int q = 0; q < nseg; ++q) t += part[q * cols + tid];
        hid[(size_t)bh * dg + tid] = 0.5f * t * (1.0f + erff(t * 0.70710678118654752440f));
    }
}

// ------------------------------------------------------------------------------------------
// out: u = W2 hid + b2 on the matrix cores, then modReLU.  W2 is stored [Hg][2F][d_g] (the d_g
// weights of one output real are contiguous), so a tile of 64 consecutive output reals n is one
// contiguous 64*d_g*4-byte block; every wave walks over tiles with a grid stride and streams them.
//
// v_mfma_f32_4x4x1_16B_f32 multiplies 16 independent 4x1 by 1x4 blocks: lane l belongs to block
// l/4; it supplies A_b[i = l%4] and B_b[j = l%4] and receives D_b[i = v][j = l%4] in register v.
// Block b holds output reals n = n0 + 4b + i (so lane l supplies the weight of n = n0 + l for the
// current hidden index, and ends up with two whole complex bins), j is one of four rows (b, h) of
// the product.  Up to 8 row groups (32 rows) are accumulated per pass over W2.
// Row r means (b, h): r = b for per-head weights (head = blockIdx.y), r = b*H + h for shared.
typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int kTileStride = 66;   // floats per staged row: 64 + 2, conflict-free for 8-byte row reads
constexpr int kHalfStride = 34;   // same for the 32-wide half rows of the d_g = 64 fast path

template <bool VEC>
__device__ __forceinline__ float4 load4(const float *__restrict__ p, int j, int dg, bool ok) {
    if (VEC) return ok ? *reinterpret_cast<const float4 *>(p + j) : make_float4(0.f, 0.f, 0.f, 0.f);
    float4 v;
    v.x = (ok && j + 0 < dg) ? p[j + 0] : 0.f;
    v.y = (ok && j + 1 < dg) ? p[j + 1] : 0.f;
    v.z = (ok && j + 2 < dg) ? p[j + 2] : 0.f;
    v.w = (ok && j + 3 < dg) ? p[j + 3] : 0.f;
    return v;
}

// four hidden indices of one staged weight row against RG row groups of hidden activations
template <int RG>
__device__ __forceinline__ void gate_mfma4(floatx4 (&acc)[RG], const float *arow, const float *hrow, int dgs) {
    const float2 a01 = *reinterpret_cast<const float2 *>(arow);
    const float2 a23 = *reinterpret_cast<const float2 *>(arow + 2);
#pragma unroll
    for (int q = 0; q < RG; ++q) {
        const float4 bv = *reinterpret_cast<const float4 *>(hrow + 4 * q * dgs);
        acc[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(a01.x, bv.x, acc[q], 0, 0, 0);
        acc[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(a01.y, bv.y, acc[q], 0, 0, 0);
        acc[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(a23.x, bv.z, acc[q], 0, 0, 0);
        acc[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(a23.y, bv.w, acc[q], 0, 0, 0);
    }
}

// 64 consecutive rows of W2 (d_g = 64) as sixteen 16-byte loads per lane: loads 0..7 cover hidden
// indices 0..31 of rows 8s + lane/8, loads 8..15 indices 32..63 (a wave instruction reads 8 half rows
// of 128 B)
__device__ __forceinline__ void gate_load_tile(float4 (&a)[16], const float *__restrict__ w2h, int tile, int lr,
                                               int lc, int twoF) {
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        const int n = tile * 64 + 8 * (s & 7) + lr;
        a[s] = (n < twoF) ? stream_load(reinterpret_cast<const float4 *>(w2h + (size_t)n * 64 + 32 * (s >> 3) + lc))
                          : make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// exp(+j 2 pi ((k p) mod n)/n), the positional phase of bin k < n at position p < n: angle reduced in integers (the quotient is
// below 2^31, so its estimate in fp64 is off by one at most) and evaluated in fp64.
struct GatePhase {
    unsigned p, n;
    double inv_n;
};
__device__ __forceinline__ float2 gate_phase(unsigned k, GatePhase ph) {
    const unsigned q = (unsigned)((double)k * (double)ph.p * ph.inv_n);
    long long m = (long long)((unsigned long long)k * ph.p - (unsigned long long)q * ph.n);
    m += m < 0 ? (long long)ph.n : m >= (long long)ph.n ? -(long long)ph.n : 0;
    double s, c;
    sincospi(2.0 * (double)(int)m * ph.inv_n, &s, &c);
    return make_float2((float)c, (float)s);
}

// modReLU (Sec. 3.2 step 3c) of one bin and its store
__device__ __forceinline__ void gate_store_bin(float2 *dst, float re, float im, bool act_on, float mb) {
    if (act_on) {
        const float mag = sqrtf(re * re + im * im);
        const float act = fmaxf(mag + mb, 0.0f);
        const float sc = (mag > 0.0f) ? act / mag : 0.0f;
        re *= sc;
        im *= sc;
    }
    *dst = make_float2(re, im);
}

struct GatePrep {                // the hidden layer's operands where k_gate_out forms it itself
    const double *partial;       // [B][nchunks][H*64]
    int nchunks;
    double inv_count;
    const float *ln_gamma, *ln_beta, *W1, *b1;
    float ln_eps;
};

// Hidden layer of the M <= 4 rows of one weight set by one workgroup of 256 lanes (d = d_g = 64): pooled sums (fp64, fixed
// order), LayerNorm with fp64 statistics, first layer, GELU.  hs [4][dgs] receives the rows; buf is scratch of 17 KB.
__device__ __forceinline__ void gate_hidden_rows(float *hs, int dgs, double *buf, const GatePrep &pr, int H, int Hg, int hsel,
                                                 int M) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hp = (Hg == 1) ? 0 : hsel;
    double *s_sum = buf;                                             // [row][wave][channel]
    float *s_qb = reinterpret_cast<float *>(buf + 4 * 4 * 64);       // [row][channel]
    float *s_part = s_qb + 4 * 64;                                   // [row][input / 8][hidden unit]
    const float gam = pr.ln_gamma[hp * 64 + lane], bet = pr.ln_beta[hp * 64 + lane], b1 = pr.b1[hp * 64 + lane];
    const size_t row = (size_t)H * 64;
    auto sums_of = [&](int r) {
        const int b = (Hg == 1) ? r / H : r, h = (Hg == 1) ? r % H : hsel;
        return pr.partial + (size_t)b * pr.nchunks * row + (size_t)h * 64 + lane;
    };
    double x = 0.0;
    if (pr.nchunks == 1) {                                           // sums already: a wave takes its row
        if (wave < M) x = *sums_of(wave);
    } else {
#pragma unroll 1
        for (int r = 0; r < M; ++r) {
            const double *src = sums_of(r);
            double t = 0.0;
            int c = wave;
            for (; c + 28 < pr.nchunks; c += 32) {                   // eight loads in flight, added in chunk order
                double v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = src[(size_t)(c + 4 * i) * row];
#pragma unroll
                for (int i = 0; i < 8; ++i) t += v[i];
            }
            for (; c < pr.nchunks; c += 4) t += src[(size_t)c * row];
            s_sum[(r * 4 + wave) * 64 + lane] = t;
        }
        __syncthreads();
        if (wave < M) {
            const double *t = s_sum + wave * 256 + lane;
            x = (t[0] + t[64]) + (t[128] + t[192]);
        }
    }
    float w1[16];                                                    // 16 of the 64 inputs per wave, lane = hidden unit
#pragma unroll
    for (int i = 0; i < 16; ++i) w1[i] = pr.W1[(size_t)hp * 4096 + (16 * wave + i) * 64 + lane];
    if (wave < M) {
        x *= pr.inv_count;
        const double dev = x - wave_sum(x) / 64;
        const double rstd = 1.0 / sqrt(wave_sum(dev * dev) / 64 + (double)pr.ln_eps);
        s_qb[wave * 64 + lane] = (float)((double)gam * dev * rstd + (double)bet);
    }
    __syncthreads();
#pragma unroll 1
    for (int r = 0; r < M; ++r) {                                    // eight inputs at a time, as k_gate_prep<512> adds them
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            float a = 0.f;
#pragma unroll
            for (int i = 8 * e; i < 8 * e + 8; ++i) a = fmaf(s_qb[r * 64 + 16 * wave + i], w1[i], a);
            s_part[(r * 8 + 2 * wave + e) * 64 + lane] = a;
        }
    }
    __syncthreads();
    float t = 0.f;
    if (wave < M) {
        const float *pp = s_part + wave * 512 + lane;
        t = b1;
#pragma unroll
        for (int q = 0; q < 8; ++q) t += pp[64 * q];
        t = 0.5f * t * (1.0f + erff(t * 0.70710678118654752440f));
    }
    hs[wave * dgs + lane] = t;                                       // rows beyond M are zero
}

// TURN: the positional phase is applied as well.  The workgroup evaluates it once for every bin of its `rounds` tiles per wave,
// while its first weights are under way, and keeps it in LDS: inside the loop over the tiles, fp64 constants and temporaries cost
// a wave per SIMD or spills.  Gate of pooled sums with a position, us, as a pass of its own over g / evaluated in the loop / now, H=32:
// B=4 n=8192 21.3 / 21.5 / 17.1; B=8 29.9 / 33.0 / 22.2; B=64 n=1024 29.4 / 33.8 / 21.8.
// FEW, for up to four rows per weight set (one tile of them) on the fast path: kTail, the two rows of W2 behind the last whole tile
// ride with the last workgroup (gate_grid); kPrep, the hidden layer is formed here as well (gate_prep_inside), the two rows as `tail` says.
enum { kTail = 1, kPrep = 2 };
template <bool VEC, int RG, bool TURN, int FEW = 0>   // VEC: d_g % 4 == 0 and 16-byte aligned rows; RG: row groups of 4
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(RG <= 2 ? 4 : 2))) void k_gate_out(const float *__restrict__ hid, const float *__restrict__ W2,
                                                  const float *__restrict__ b2,
                                                  const float *__restrict__ mbias, float2 *__restrict__ g,
                                                  int B, int H, int Hg, int dg, int F, int r_base0,
                                                  int rounds, bool has_tail, GatePhase phase, GatePrep pr) {
    static_assert(!FEW || (VEC && RG == 1), "four rows on the fast path");
    extern __shared__ float hs[];
    const int r_base = r_base0 + 4 * RG * (int)blockIdx.z;   // blockIdx.z: tile of the rows (sequences)                    // [4*RG][dgs] hidden rows of this pass, zero padded
    const int dgp = (dg + 3) & ~3, dgs = dgp + 4;    // row stride padded against bank conflicts
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int twoF = 2 * F;
    const int hsel = blockIdx.y;                     // head of this block when weights are per head
    const int hp = (Hg == 1) ? 0 : hsel;
    const int M = (Hg == 1) ? B * H : B;
    const bool tail = FEW == kTail || (FEW == kPrep && has_tail);
    const int ntiles = tail ? twoF / 64 : (twoF + 63) / 64;
    const float *w2h = W2 + (size_t)hp * twoF * dg;
    // the fast path's first tile is requested before anything else (with more than two row groups the registers it would
    // hold meanwhile cost a wave per SIMD)
    constexpr bool kEarly = RG <= 2;
    const int lr = lane >> 3, lc = 4 * (lane & 7), tstep = gridDim.x * 4;
    int ftile = blockIdx.x * 4 + wave;
    float4 a[16];
    if (kEarly && VEC && dg == 64 && ftile < ntiles) gate_load_tile(a, w2h, ftile, lr, lc, twoF);
    if (FEW == kPrep) {
        gate_hidden_rows(hs, dgs, reinterpret_cast<double *>(hs + 4 * dgs), pr, H, Hg, hsel, M);
    } else {
        for (int idx = threadIdx.x; idx < 4 * RG * dgs; idx += 256) {
            const int rr = idx / dgs, j = idx % dgs, r = r_base + rr;
            float v = 0.f;
            if (r < M && j < dg) v = hid[(size_t)((Hg == 1) ? r : r * H + hsel) * dg + j];
            hs[idx] = v;
        }
    }
    const bool mine = FEW && tail && wave == 3 && blockIdx.x == gridDim.x - 1;
    float4 w_re = make_float4(0.f, 0.f, 0.f, 0.f), w_im = w_re;
    if (mine) {                                                      // lane = row of the hidden values and four of the 64 weights
        const float4 *src = reinterpret_cast<const float4 *>(w2h + (size_t)ntiles * 4096) + (lane & 15);
        w_re = src[0];
        w_im = src[16];
    }
    float2 *turn = reinterpret_cast<float2 *>(hs + 4 * RG * dgs + 4 * 64 * ((VEC && dg == 64) ? kHalfStride : kTileStride));
    if (TURN)
        for (int e = threadIdx.x; e < 128 * rounds; e += 256)        // [round][wave][bin of the tile]
            turn[e] = gate_phase(((unsigned)(blockIdx.x * 4 + ((e >> 5) & 3) + (e >> 7) * tstep)) * 32 + (e & 31), phase);
    const float2 turn_last = TURN && mine ? gate_phase(F - 1, phase) : make_float2(1.f, 0.f);
    __syncthreads();
    turn += wave * 32 + ((lane & ~3) >> 1);                          // this lane's two bins of a tile
    const int jrow = lane & 3;
    // per-wave staging tile [64 rows][kTileStride floats]: filled with fully coalesced 16-byte
    // loads (a wave instruction covers 4 whole rows of 64 weights), read back one row per lane
    float *tile_w = hs + 4 * RG * dgs + wave * (64 * ((VEC && dg == 64) ? kHalfStride : kTileStride));
    if (VEC && dg == 64) {
        // fast path (one 64-wide slab per tile), software pipelined: the next tile's weights and this
        // tile's bias terms are in flight while the matrix cores work on the staged tile
        if (!kEarly && ftile < ntiles) gate_load_tile(a, w2h, ftile, lr, lc, twoF);
        for (int tile = ftile; tile < ntiles; tile += tstep) {
            floatx4 acc[RG];
#pragma unroll
            for (int q = 0; q < RG; ++q) acc[q] = floatx4{0.f, 0.f, 0.f, 0.f};
            const float *arow = tile_w + lane * kHalfStride;
            const float *hrow = hs + jrow * dgs;
            // first half of the hidden indices through the staging tile
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                float2 *dst = reinterpret_cast<float2 *>(tile_w + (8 * s + lr) * kHalfStride + lc);
                dst[0] = make_float2(a[s].x, a[s].y);
                dst[1] = make_float2(a[s].z, a[s].w);
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int jj = 0; jj < 32; jj += 4) gate_mfma4<RG>(acc, arow + jj, hrow + jj, dgs);
            __builtin_amdgcn_wave_barrier();
            // second half; after its copy to LDS the registers are free for the next tile's loads
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                float2 *dst = reinterpret_cast<float2 *>(tile_w + (8 * s + lr) * kHalfStride + lc);
                dst[0] = make_float2(a[8 + s].x, a[8 + s].y);
                dst[1] = make_float2(a[8 + s].z, a[8 + s].w);
            }
            if (tile + tstep < ntiles) gate_load_tile(a, w2h, tile + tstep, lr, lc, twoF);
            const int n4 = tile * 64 + (lane & ~3);
            const bool e_ok = n4 < twoF;                      // twoF is even and n4 a multiple of 4
            const bool e_ok2 = n4 + 2 < twoF;
            float4 bias4 = make_float4(0.f, 0.f, 0.f, 0.f);
            float2 mb2 = make_float2(0.f, 0.f);
            if (e_ok) {
                const float *bp = b2 + (size_t)hp * twoF + n4;
                bias4.x = bp[0]; bias4.y = bp[1];
                if (e_ok2) { bias4.z = bp[2]; bias4.w = bp[3]; }
                if (mbias) {
                    const float *mp = mbias + (size_t)hp * F + (n4 >> 1);
                    mb2.x = mp[0];
                    if (e_ok2) mb2.y = mp[1];
                }
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int jj = 0; jj < 32; jj += 4) gate_mfma4<RG>(acc, arow + jj, hrow + 32 + jj, dgs);
            __builtin_amdgcn_wave_barrier();
            float4 ph = make_float4(1.f, 0.f, 1.f, 0.f);
            if (TURN) {
                ph = *reinterpret_cast<const float4 *>(turn);
                turn += 128;
            }
#pragma unroll
            for (int q = 0; q < RG; ++q) {
                const int r = r_base + 4 * q + jrow;
                if (r >= M || !e_ok) continue;
                const int bh = (Hg == 1) ? r : r * H + hsel;
                float2 v0, v1;
                gate_store_bin(&v0, acc[q][0] + bias4.x, acc[q][1] + bias4.y, mbias != nullptr, mb2.x);
                gate_store_bin(&v1, acc[q][2] + bias4.z, acc[q][3] + bias4.w, mbias != nullptr, mb2.y);
                if (TURN) {
                    v0 = cmul(v0, make_float2(ph.x, ph.y));
                    v1 = cmul(v1, make_float2(ph.z, ph.w));
                }
                g[(size_t)bh * F + (n4 >> 1)] = v0;
                if (e_ok2) g[(size_t)bh * F + (n4 >> 1) + 1] = v1;
            }
        }
        if (mine) {                            // the last bin, all four rows at once
            const float2 bias = make_float2(b2[(size_t)hp * twoF + twoF - 2], b2[(size_t)hp * twoF + twoF - 1]);
            const float mb = mbias ? mbias[(size_t)hp * F + F - 1] : 0.f;
            const int r = lane >> 4;
            const float4 hv = *reinterpret_cast<const float4 *>(hs + r * dgs + 4 * (lane & 15));
            float re = fmaf(w_re.x, hv.x, fmaf(w_re.y, hv.y, fmaf(w_re.z, hv.z, w_re.w * hv.w)));
            float im = fmaf(w_im.x, hv.x, fmaf(w_im.y, hv.y, fmaf(w_im.z, hv.z, w_im.w * hv.w)));
            re += partner16<8>(re);
            im += partner16<8>(im);
            re += partner16<4>(re);
            im += partner16<4>(im);
            re += partner16<2>(re);
            im += partner16<2>(im);
            re += partner16<1>(re);
            im += partner16<1>(im);
            if ((lane & 15) == 0 && r < M) {
                const int bh = (Hg == 1) ? r : r * H + hsel;
                float2 v;
                gate_store_bin(&v, re + bias.x, im + bias.y, mbias != nullptr, mb);
                g[(size_t)bh * F + F - 1] = TURN ? cmul(v, turn_last) : v;
            }
        }
        return;
    }
    for (int tile = blockIdx.x * 4 + wave; tile < ntiles; tile += gridDim.x * 4) {
        floatx4 acc[RG];
#pragma unroll
        for (int q = 0; q < RG; ++q) acc[q] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int j0 = 0; j0 < dgp; j0 += 64) {
            const int width = min(64, dgp - j0);          // hidden indices in this slab, multiple of 4
            const int lpr = width / 4;                     // lanes per row
            const int rows_per_instr = 64 / lpr;
            const int lr = lane / lpr, lc = 4 * (lane % lpr);
            for (int r0 = 0; r0 < 64; r0 += rows_per_instr) {
                const int row = r0 + lr, n = tile * 64 + row;
                if (row < 64) {
                    const float4 v = load4<VEC>(w2h + (size_t)(n < twoF ? n : 0) * dg, j0 + lc, dg, n < twoF);
                    float *dst = tile_w + row * kTileStride + lc;
                    dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
                }
            }
            // LDS operations of one wave complete in issue order, so the reads below see the writes
            // above; the wave barrier only stops the compiler from moving code across this point
            __builtin_amdgcn_wave_barrier();
            const float *arow = tile_w + lane * kTileStride;
            const float *hrow = hs + jrow * dgs + j0;
            for (int jj = 0; jj < width; jj += 4) gate_mfma4<RG>(acc, arow + jj, hrow + jj, dgs);
            __builtin_amdgcn_wave_barrier();
        }
        // epilogue: this lane holds reals n4 .. n4+3 (two bins) of row r for every row group
        const int n4 = tile * 64 + (lane & ~3);
        float2 ph[2] = {};
        if (TURN) {
            ph[0] = turn[0];
            ph[1] = turn[1];
            turn += 128;
        }
#pragma unroll
        for (int q = 0; q < RG; ++q) {
            const int r = r_base + 4 * q + jrow;
            if (r >= M) continue;
            const int bh = (Hg == 1) ? r : r * H + hsel;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int nn = n4 + 2 * half;
                if (nn >= twoF) continue;
                const int k = nn >> 1;
                float2 v;
                gate_store_bin(&v, acc[q][2 * half] + b2[(size_t)hp * twoF + nn], acc[q][2 * half + 1] + b2[(size_t)hp * twoF + nn + 1],
                               mbias != nullptr, mbias ? mbias[(size_t)hp * F + k] : 0.0f);
                g[(size_t)bh * F + k] = TURN ? cmul(v, ph[half]) : v;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// short sequences: everything in one launch.  A workgroup pools the rows of one (b, h) itself (fp64), normalises,
// evaluates the hidden layer, and emits tiles of 64 output reals, one per wave at a time; grid (parts, B*H), the parts of
// a head repeat the pooling from L2.
// What bounds it is the chain of latencies (rows, first layer, output layer): the first tile's weights are requested
// before the rows.  Against the pooling, prep and output launches: B=1 H=32 bf16 L=512 26.3 -> 20.2 us for a step of
// gate and mixer, B=256 H=12 fp32 L=196 120 -> 105 us.
// ONCE: one part per head, so nobody reads its rows again and they pass the caches by, which the heads' weights keep:
// B=256 H=12 fp32 L=196 106.0 -> 100.8 us (five waves per SIMD instead of four spill: 125.7).
// A lane's four weights of row 4 s + lane / 16 of a tile meet the hidden values, summed over the 16 lanes (fold16).
template <bool BF16, int NT, bool ONCE>
__global__ __launch_bounds__(NT, 4) void k_gate_small(const void *__restrict__ q, double inv_count, GateDev P,
                                                    const float *__restrict__ act_bias, float2 *__restrict__ g,
                                                    int L, int H, int F, int ntiles) {
    constexpr int NCH = BF16 ? 8 : 4, LPR = 64 / NCH, RPW = 64 / LPR;   // channels per lane, lanes per row, rows per wave
    constexpr int NW = NT / 64, IPW = 64 / NW;                              // waves; first-layer inputs per wave
    __shared__ double psum[NW][64];
    __shared__ float qb[NW][64], part[NW][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int bh = blockIdx.y, b = bh / H, h = bh % H, hp = (P.Hg == 1) ? 0 : h, twoF = 2 * F;
    // tile t = the 64 rows of W2 from tile_row(t) on: the last one is moved back to end with the matrix (2F >= 64), so that
    // every access is in range without a test per row; its overlap is computed twice, to the same bits
    const float4 *w2 = reinterpret_cast<const float4 *>(P.W2 + (size_t)hp * twoF * 64) + lane;
    auto tile_row = [&](int t) { return min(64 * t, twoF - 64); };
    int tile = __builtin_amdgcn_readfirstlane(blockIdx.x * NW + wave);
    float4 a[16];
    auto request = [&](int t) {
        const float4 *src = w2 + (size_t)tile_row(t) * 16;
#pragma unroll
        for (int s = 0; s < 16; ++s) a[s] = src[64 * s];
    };
    // the small operands first, so that their latency passes behind the rows
    const float gam = P.ln_gamma[hp * 64 + lane], bet = P.ln_beta[hp * 64 + lane], b1 = P.b1[hp * 64 + lane];
    float w1[IPW];
#pragma unroll
    for (int i = 0; i < IPW; ++i) w1[i] = P.W1[(size_t)hp * 4096 + (IPW * wave + i) * 64 + lane];

    const size_t rs = (size_t)H * LPR;                                  // 16-byte pieces per token row
    const int r0 = tid / LPR;
    // 16 bytes at any 4-byte boundary, so that the tensor's alignment does not change the order of the additions
    typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
    const u32x4_a4 *src = reinterpret_cast<const u32x4_a4 *>(q) + ((size_t)b * L + r0) * rs + (size_t)h * LPR + (lane % LPR);
    double sum[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) sum[c] = 0.0;
    constexpr int RPS = NW * RPW, kU = 8;                                // rows per sweep, sweeps in flight
    for (int l = r0; l < L; l += RPS * kU) {
        u32x4_a4 w[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            w[u] = u32x4_a4{0, 0, 0, 0};
            if (l + RPS * u < L) w[u] = ONCE ? __builtin_nontemporal_load(src + (size_t)RPS * u * rs) : src[(size_t)RPS * u * rs];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (BF16) {
                    const float2 v = IoBf16::unpack(w[u][i]);
                    sum[(2 * i) % NCH] += (double)v.x;
                    sum[(2 * i + 1) % NCH] += (double)v.y;
                } else {
                    sum[i] += (double)__uint_as_float(w[u][i]);
                }
            }
        }
        src += (size_t)RPS * kU * rs;
    }
#pragma unroll
    for (int off = LPR; off < 64; off <<= 1) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) sum[c] += __shfl_xor(sum[c], off);
    }
    if (tile < ntiles) request(tile);                            // in flight during the first layer
    if (lane < LPR) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) psum[wave][NCH * lane + c] = sum[c];
    }
    __syncthreads();
    {   // every wave repeats the LayerNorm for itself (lane = channel)
        double t = psum[0][lane];
#pragma unroll
        for (int r = 1; r < NW; ++r) t += psum[r][lane];
        const double x = inv_count * t;
        const double dev = x - wave_sum(x) / 64;
        const double rstd = 1.0 / sqrt(wave_sum(dev * dev) / 64 + (double)P.ln_eps);
        qb[wave][lane] = (float)((double)gam * dev * rstd + (double)bet);
    }
    __builtin_amdgcn_wave_barrier();
    {   // first layer: wave w takes inputs IPW w .. IPW w + IPW - 1, lane = hidden unit
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < IPW; ++i) t = fmaf(qb[wave][IPW * wave + i], w1[i], t);
        part[wave][lane] = t;
    }
    __syncthreads();
    {
        float t = b1;
#pragma unroll
        for (int r = 0; r < NW; ++r) t += part[r][lane];
        qb[wave][lane] = 0.5f * t * (1.0f + erff(t * 0.70710678118654752440f));
    }
    __builtin_amdgcn_wave_barrier();
    const float4 hv = *reinterpret_cast<const float4 *>(&qb[wave][4 * (lane & 15)]);
    for (int first = tile; tile < ntiles; tile += NW * gridDim.x) {
        if (tile != first) request(tile);
        float p[16];
#pragma unroll
        for (int s = 0; s < 16; ++s) p[s] = fmaf(a[s].x, hv.x, fmaf(a[s].y, hv.y, fmaf(a[s].z, hv.z, a[s].w * hv.w)));
        fold16<8>(p, lane);
        fold16<4>(p, lane);
        fold16<2>(p, lane);
        fold16<1>(p, lane);
        // lane holds real tile_row + 4 (lane % 16) + lane / 16: the imaginary part of an even one sits 16 lanes further
        const float other = __shfl_xor(p[0], 16);
        const int k = tile_row(tile) / 2 + 2 * (lane & 15) + (lane >> 5);
        if (!(lane & 16)) {
            const float2 bias = *reinterpret_cast<const float2 *>(P.b2 + ((size_t)hp * F + k) * 2);
            gate_store_bin(g + (size_t)bh * F + k, p[0] + bias.x, other + bias.y, act_bias != nullptr,
                           act_bias ? act_bias[(size_t)hp * F + k] : 0.0f);
        }
    }
}

// Toeplitz low-rank update (Sec. 3.2 step 3b) followed by modReLU (step 3c):
//   g_k = act( raw_k + sum_{m=-r..r} t_m raw_{k-m} ),  raw = 0 outside 0..F-1.   One lane per bin.
__global__ __launch_bounds__(256) void k_gate_toeplitz(const float2 *__restrict__ raw, const float2 *__restrict__ taps,
                                                       const float *__restrict__ mbias, float2 *__restrict__ g,
                                                       int H, int Hg, int F, int r, size_t total) {
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int k = (int)(idx % F);
    const size_t bh = idx / F;
    const int hp = (Hg == 1) ? 0 : (int)(bh % H);
    const float2 *t = taps + (size_t)hp * (2 * r + 1) + r;
    const float2 *row = raw + bh * F;
    float2 acc = row[k];
    for (int m = -r; m <= r; ++m) {
        const int src = k - m;
        if (src < 0 || src >= F) continue;
        const float2 pr = cmul(t[m], row[src]);
        acc.x += pr.x;
        acc.y += pr.y;
    }
    gate_store_bin(g + idx, acc.x, acc.y, mbias != nullptr, mbias ? mbias[(size_t)hp * F + k] : 0.0f);
}

// positional phase: g[bh][k] *= exp(+j 2 pi ((k p) mod n)/n), angle reduced in integers and
// evaluated in fp64.  One lane per gate entry; only launched when p != 0.
__global__ __launch_bounds__(256) void k_gate_phase(float2 *__restrict__ g, int F, GatePhase phase, size_t total) {
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    g[idx] = cmul(g[idx], gate_phase((unsigned)(idx % F), phase));
}

// ------------------------------------------------------------------------------------------
// Rows summed by one workgroup of the pooling pass: kPoolRows, halved (down to 16) while the pass would launch
// fewer than about two workgroups per compute unit (short sequences: 8192 rows of 32 heads are only 32 chunks of 256).
int pool_rows(int B, int L, int H, int d) {
    const long long wide = ((long long)H * d / 8 + 255) / 256;       // workgroups across a row with 16-byte lanes
    int rows = kPoolRows;
    while (rows > 16 && (long long)B * ((L + rows - 1) / rows) * wide < 512) rows /= 2;
    return rows;
}

// Pieces of a row per workgroup of k_pool_deep, 0 where the pass of whole rows takes the sums: rows that are no whole number
// of 128-byte lines; sequences long enough for 256 rows a chunk (32 heads of 131072 bf16 rows: step of gate and mixer 1237
// instead of 1226 us); and chunks of 128 whole rows of 2 or 4 KB, which fill half or all of that pass's workgroups (gate, us, whole rows /
// deep: 4 x 16 heads of 16384 bf16 42.9 / 45.2, fp32 60.8 / 64.5, 4 x 8 fp32 36.2 / 38.0, 4 x 32 bf16 74.3 / 77.3; rows of 1 KB, 4 x 8 bf16
// 31.6 / 27.1, of 1.5 KB, 4 x 12 bf16 38.0 / 34.4, of 8 KB, 8 x 32 of 8192 fp32 110.5 / 108.0; chunks of 64 rows -2 to +4 %).
static int pool_deep_cols(int io, int B, int L, int H, int d) {
    const int bytes = H * d * (io ? 2 : 4), ppv = bytes / 16, rows = pool_rows(B, L, H, d);
    if (bytes % 128 || rows == kPoolRows || (rows == kPoolRows / 2 && (bytes == 2048 || bytes == 4096))) return 0;
    return ppv % 32 == 0 ? 32 : ppv % 16 == 0 ? 16 : 8;
}
// Rows of one of its chunks: halved from 256 while there are less workgroups than compute units, and never fewer than the size
// of the partial sums is for.
static int pool_deep_rows(int io, int B, int L, int H, int d, int cols) {
    const long long wide = (long long)H * d * (io ? 2 : 4) / 16 / cols;
    const int least = pool_rows(B, L, H, d);
    int rows = kPoolRows;
    while (rows > 64 && rows > least && (long long)B * ((L + rows - 1) / rows) * wide < 256) rows /= 2;
    return rows;
}

size_t gate_partial_bytes(int B, int L, int H, int d) {
    const int rows = pool_rows(B, L, H, d);
    const int nchunks = (L + rows - 1) / rows;
    return (size_t)B * nchunks * H * d * sizeof(double);
}

int pool_chunks(int io, int B, int L, int H, int d) {
    const int cols = pool_deep_cols(io, B, L, H, d);
    const int rows = cols ? pool_deep_rows(io, B, L, H, d, cols) : pool_rows(B, L, H, d);
    return (L + rows - 1) / rows;
}

hipError_t launch_pool_partial(int io, const void *q, double *partial, int B, int L, int H, int d, hipStream_t st) {
    if (const int cols = pool_deep_cols(io, B, L, H, d)) {
        const int rows = pool_deep_rows(io, B, L, H, d, cols), nchunks = (L + rows - 1) / rows, ppv = H * d * (io ? 2 : 4) / 16;
        const dim3 grid(ppv / cols, nchunks, B);
#define SPECTRE_POOL_DEEP(C)                                                                \
    if (io) k_pool_deep<true, C><<<grid, 512, 0, st>>>(q, partial, L, ppv, rows, nchunks); \
    else k_pool_deep<false, C><<<grid, 512, 0, st>>>(q, partial, L, ppv, rows, nchunks)
        if (cols == 32) { SPECTRE_POOL_DEEP(32); } else if (cols == 16) { SPECTRE_POOL_DEEP(16); } else { SPECTRE_POOL_DEEP(8); }
#undef SPECTRE_POOL_DEEP
        return hipGetLastError();
    }
    const int ppr = H * d / 2;
    const int rows = pool_rows(B, L, H, d);
    const int nchunks = (L + rows - 1) / rows;
    dim3 grid((ppr + 255) / 256, nchunks, B);
    const bool aligned = (reinterpret_cast<uintptr_t>(q) & 15) == 0;
    if (io && ppr % 4 == 0 && aligned)
        k_pool_partial_x16<true><<<dim3((ppr / 4 + 255) / 256, nchunks, B), 256, 0, st>>>(
            static_cast<const uint4 *>(q), partial, L, ppr / 4, rows, nchunks);
    else if (!io && ppr % 2 == 0 && aligned)
        k_pool_partial_x16<false><<<dim3((ppr / 2 + 255) / 256, nchunks, B), 256, 0, st>>>(
            static_cast<const uint4 *>(q), partial, L, ppr / 2, rows, nchunks);
    else if (io)
        k_pool_partial<IoBf16><<<grid, 256, 0, st>>>(static_cast<const uint32_t *>(q),
                                                     reinterpret_cast<double2 *>(partial), L, ppr, rows, nchunks);
    else
        k_pool_partial<IoF32><<<grid, 256, 0, st>>>(static_cast<const float2 *>(q),
                                                    reinterpret_cast<double2 *>(partial), L, ppr, rows, nchunks);
    return hipGetLastError();
}

hipError_t launch_pool(int io, const void *q, double *partial, double *sum_q, int B, int L, int H, int d,
                       hipStream_t st) {
    const hipError_t e = launch_pool_partial(io, q, partial, B, L, H, d, st);
    if (e != hipSuccess) return e;
    k_pool_final<<<dim3((H * d + 31) / 32, B), 256, 0, st>>>(partial, sum_q, H * d, pool_chunks(io, B, L, H, d), 0);
    return hipGetLastError();
}

hipError_t launch_pool_final(const double *partial, double *sum, int B, int row, int nchunks, hipStream_t st,
                             bool accumulate) {
    k_pool_final<<<dim3((row + 31) / 32, B), 256, 0, st>>>(partial, sum, row, nchunks, accumulate ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_gate_prep(const double *partial, int nchunks, const float *Wq, int Hw, double *sum_q, double inv_count,
                            const GateDev &P, float *hid, int B, int H, hipStream_t st) {
    if (Wq && P.d != 64) return hipErrorInvalidValue;
    // four workgroups of 512 lanes fit a compute unit; with more heads than twice that many the number in flight counts for
    // more than the latency of one (from pooled sums, H=32 n=196: B=128 23 -> 18 us, B=256 38 -> 28)
    if (B * H >= 2048) k_gate_prep<256><<<B * H, 256, 0, st>>>(partial, nchunks, Wq, Hw, sum_q, inv_count, P, hid, H);
    else k_gate_prep<512><<<B * H, 512, 0, st>>>(partial, nchunks, Wq, Hw, sum_q, inv_count, P, hid, H);
    return hipGetLastError();
}

static GatePhase gate_phase_of(const GateDev &P, long long phase) {
    return {(unsigned)(phase % P.n_fft), (unsigned)P.n_fft, 1.0 / (double)P.n_fft};
}

// Toeplitz update and positional phase, the passes over g behind the output layer.
static hipError_t launch_gate_tail(const GateDev &P, const float2 *raw, int B, int H, long long phase, float2 *g,
                                   hipStream_t st) {
    const int F = P.n_fft / 2 + 1;
    const size_t total = (size_t)B * H * F;
    if (P.toeplitz) {
        k_gate_toeplitz<<<(unsigned)((total + 255) / 256), 256, 0, st>>>(raw, P.toeplitz, P.modrelu_bias, g, H, P.Hg, F,
                                                                         P.toeplitz_r, total);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (phase == 0) return hipSuccess;
    k_gate_phase<<<(unsigned)((total + 255) / 256), 256, 0, st>>>(g, F, gate_phase_of(P, phase), total);
    return hipGetLastError();
}

// partial != nullptr: the hidden layer from these partial sums, inside the same launch (gate_prep_inside); else hid.
static hipError_t gate_out(const float *hid, const double *partial, int nchunks, double inv_count, const GateDev &P, float2 *raw,
                           int B, int H, long long phase, float2 *g, hipStream_t st) {
    const int F = P.n_fft / 2 + 1;
    const int M = (P.Hg == 1) ? B * H : B, twoF = 2 * F;
    const GateGrid gr = gate_grid(P, B, H);
    const int rounds = gr.rounds;
    dim3 grid(gr.gx, gr.gy);
    const GatePrep pr = {partial, nchunks, inv_count, P.ln_gamma, P.ln_beta, P.W1, P.b1, P.ln_eps};
    const bool vec = gate_vec(P);
    const int dgp = (P.d_g + 3) & ~3;
    // with the Toeplitz update the MLP output goes to `raw` un-activated and a second pass finishes it
    const float *out_bias = P.toeplitz ? nullptr : P.modrelu_bias;
    float2 *out_g = P.toeplitz ? raw : g;
    // the phase of a wave's tiles takes 1 KB of LDS a round; beyond 16 rounds (hundreds of heads with long gates) it is a pass of its own
    const bool turn = phase != 0 && !P.toeplitz && rounds <= 16;
    {
        // every tile of the rows in one launch (grid.z); a single tile takes the narrowest kernel that fits
        // rows per tile: 32, fewer while the launch would have less than four workgroups per compute unit (B=256 H=12
        // L=196, 96 workgroups of 32 rows: 15 -> 7.4 us).  Every tile reads the weights again, so where those of one set
        // do not stay in an XCD's 4 MB of L2, two workgroups per compute unit are enough and 16 rows the least (from pooled
        // sums, 32 / 16 / 8 / 4 rows: n = 20480, 24 rows over 4 sets 20 / 17 / 17 / 21 us, 96 over one 19 / 16 / 17 / 22,
        // 256 over one 27 / 31 / 36 / 51; n = 8192, 96 over one 18 / 13 / 12 / 12).
        const bool large = (size_t)twoF * P.d_g * sizeof(float) > ((size_t)4 << 20);
        int per = 32;
        while (per > (large ? 16 : 4) && M > per / 2 &&
               (long long)grid.x * grid.y * ((M + per - 1) / per) < (large ? 512 : 1024)) per /= 2;
        const int ntile = (M + per - 1) / per;
        const int rows = (ntile > 1) ? per : M;
        const int rg = (rows + 3) / 4;            // 1..8 row groups per tile
        const size_t lds = ((size_t)4 * (rg <= 1 ? 1 : rg <= 2 ? 2 : rg <= 4 ? 4 : 8) * (dgp + 4) +
                            4 * 64 * ((vec && P.d_g == 64) ? kHalfStride : kTileStride)) * sizeof(float) +
                           (turn ? rounds * 128 * sizeof(float2) : 0);
        for (int z0 = 0; z0 < ntile; z0 += 65535) {
            const int nz = (ntile - z0 < 65535) ? ntile - z0 : 65535;
            const dim3 grid3(grid.x, grid.y, nz);
            const int r_base = per * z0;
#define SPECTRE_GATE_OUT(V, R, FEW)                                                                                             \
    if (turn) k_gate_out<V, R, true, FEW><<<grid3, 256, lds, st>>>(hid, P.W2, P.b2, out_bias, out_g, B, H, P.Hg, P.d_g, F,      \
                                                                   r_base, rounds, gr.tail, gate_phase_of(P, phase), pr);       \
    else k_gate_out<V, R, false, FEW><<<grid3, 256, lds, st>>>(hid, P.W2, P.b2, out_bias, out_g, B, H, P.Hg, P.d_g, F, r_base,  \
                                                               rounds, gr.tail, gate_phase_of(P, phase), pr)
            if (partial) { SPECTRE_GATE_OUT(true, 1, kPrep); }
            else if (gr.tail) { SPECTRE_GATE_OUT(true, 1, kTail); }
            else if (vec) {
                if (rg <= 1) { SPECTRE_GATE_OUT(true, 1, 0); } else if (rg <= 2) { SPECTRE_GATE_OUT(true, 2, 0); }
                else if (rg <= 4) { SPECTRE_GATE_OUT(true, 4, 0); } else { SPECTRE_GATE_OUT(true, 8, 0); }
            } else {
                if (rg <= 1) { SPECTRE_GATE_OUT(false, 1, 0); } else if (rg <= 2) { SPECTRE_GATE_OUT(false, 2, 0); }
                else if (rg <= 4) { SPECTRE_GATE_OUT(false, 4, 0); } else { SPECTRE_GATE_OUT(false, 8, 0); }
            }
#undef SPECTRE_GATE_OUT
            hipError_t e2 = hipGetLastError();
            if (e2 != hipSuccess) return e2;
        }
    }
    return launch_gate_tail(P, raw, B, H, turn ? 0 : phase, g, st);
}

hipError_t launch_gate_out(const float *hid, const GateDev &P, float2 *raw, int B, int H, long long phase, float2 *g,
                           hipStream_t st) {
    return gate_out(hid, nullptr, 0, 0.0, P, raw, B, H, phase, g, st);
}

// Short sequences: up to 256 KB of rows per head (B=1 H=32, step of gate and mixer: bf16 L=2048 46.0 -> 42.8 us, L=4096
// would be 50.4 -> 53.8), unless several sequences would each read a head's output weights of more than 320 KB again
// (B=8 H=32 L=1024, 263 KB: 82.1 -> 77.9 us; B=4 L=2048, 525 KB: 82.3 -> 88.4), or all of them together would read so much
// that way, at about 17 TB/s, that it costs more than the other route's 23 us and 3 ns a head.  Gate alone, bf16, this
// kernel and the three launches: H=32 B=64 L=900 65 and 66 us, B=64 L=1024 73 and 66, B=128 L=1024 144 and 116, B=256
// L=512 147 and 125, B=256 L=1240 337 and 270.
static bool gate_small(int io, const GateDev &P, int B, int L, int H) {
    const int F = P.n_fft / 2 + 1;
    const size_t rows = (size_t)L * 64 * (io ? 2 : 4), w2 = (size_t)2 * F * 64 * 4;
    const long long heads = (long long)B * H;
    if (P.d != 64 || P.d_g != 64 || F < 32 || rows > ((size_t)256 << 10)) return false;
    if ((reinterpret_cast<uintptr_t>(P.W2) & 15) || (reinterpret_cast<uintptr_t>(P.b2) & 7)) return false;
    if (heads > 65535) return false;
    return B == 1 || (w2 <= ((size_t)320 << 10) && heads * ((long long)w2 - 50000) <= 400000000);
}

hipError_t launch_gate(int io, const void *q, double *partial, double inv_count, const GateDev &P, float *hid, float2 *raw,
                       int B, int L, int H, long long phase, float2 *g, hipStream_t st) {
    if (gate_small(io, P, B, L, H)) {
        const int F = P.n_fft / 2 + 1, ntiles = (2 * F + 63) / 64;
        // Few heads: 16 waves each, so that a head's rows are in flight together; many: 4 waves, four workgroups on a
        // compute unit.  Parts of a head: one wave per tile, while that leaves the pooling repeated in less than two
        // workgroups per compute unit.
        const bool wide = B * H < 256;
        int parts = (ntiles + (wide ? 15 : 3)) / (wide ? 16 : 4);
        while (parts > 1 && (long long)parts * B * H > 512) parts = (parts + 1) / 2;
        const float *act = P.toeplitz ? nullptr : P.modrelu_bias;
        float2 *out = P.toeplitz ? raw : g;
        const dim3 grid(parts, B * H);
#define SPECTRE_GATE_SMALL(BF, NT, ONCE) \
    k_gate_small<BF, NT, ONCE><<<grid, NT, 0, st>>>(q, inv_count, P, act, out, L, H, F, ntiles)
#define SPECTRE_GATE_SMALL_IO(BF)                              \
    if (wide) SPECTRE_GATE_SMALL(BF, 1024, false);             \
    else if (parts == 1) SPECTRE_GATE_SMALL(BF, 256, true);    \
    else SPECTRE_GATE_SMALL(BF, 256, false)
        if (io) { SPECTRE_GATE_SMALL_IO(true); } else { SPECTRE_GATE_SMALL_IO(false); }
#undef SPECTRE_GATE_SMALL_IO
#undef SPECTRE_GATE_SMALL
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_gate_tail(P, raw, B, H, phase, g, st);
    }
    hipError_t e = launch_pool_partial(io, q, partial, B, L, H, P.d, st);
    if (e != hipSuccess) return e;
    const int nchunks = pool_chunks(io, B, L, H, P.d);
    if (gate_prep_inside(P, B, H, nchunks)) return gate_out(hid, partial, nchunks, inv_count, P, raw, B, H, phase, g, st);
    e = launch_gate_prep(partial, nchunks, nullptr, 1, nullptr, inv_count, P, hid, B, H, st);
    if (e != hipSuccess) return e;
    return launch_gate_out(hid, P, raw, B, H, phase, g, st);
}

hipError_t launch_gate_mlp(const double *sum_q, double inv_count, const GateDev &P, float *hid, float2 *raw,
                           int B, int H, long long phase, float2 *g, hipStream_t st) {
    if (gate_prep_inside(P, B, H, 1)) return gate_out(hid, sum_q, 1, inv_count, P, raw, B, H, phase, g, st);
    const hipError_t e = launch_gate_prep(sum_q, 1, nullptr, 1, nullptr, inv_count, P, hid, B, H, st);
    if (e != hipSuccess) return e;
    return launch_gate_out(hid, P, raw, B, H, phase, g, st);
}

// Loads this translation unit's code object (the runtime loads them on first use): called by spectre_prepare so
// that no compute call is the first to touch it.
hipError_t load_kernels_gate() {
    hipFuncAttributes a;
    return hipFuncGetAttributes(&a, reinterpret_cast<const void *>(k_pool_final));
}

}  // namespace spectre
