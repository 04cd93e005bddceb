// Columns of the cache's window transform and full-window readout, together with the step between the pair spectrum and
// the two channels' half spectra (N <= 32768; gfx950), and the mixer's columns of 1024 points.
//
//   k_cache_fwd : scratch columns [k2][pair][t1] -> N1-point transforms -> half-spectrum rows X[k][channel]
//   k_cache_inv : rows X, times the gate -> pair spectrum -> inverse N1-point transforms -> scratch columns
//   k_mix_cols  : scratch columns -> transforms, gate, inverse transforms, in place
//
// A bin k = k2 + N2 k1 and its Hermitian partner N - k lie in the planes k2 and N2 - k2, so a workgroup that holds both
// planes of a few channel pairs separates (or joins) the channels itself.  As kernels of their own the column transforms
// and that step moved 16 bytes each per pair and position beside those of the row transforms; here the spectrum crosses
// memory once less.  What bounds them is memory traffic, 16 bytes per pair and position: 25 heads of N = 32768 forward 134
// -> 72 us (5.8 TB/s), 102 heads of N = 8192 inverse 134 -> 77 us (5.6 TB/s).  With 64-byte pieces of the rows of X and whole
// columns in LDS the former took 105 us, with plain stores of X, which push the scratch out of the memory-side cache, 88.
// Whole calls: prompt of 20011 tokens, B = 8 H = 32 N = 32768, 3603 -> 2956 us; 57 tokens and the window's readout, B = 4
// H = 32 N = 8192, 427 -> 352 us.
//
// N1 = R * R points are two passes of R-point transforms in registers with one exchange inside R lanes of a wave.  R = 16
// for N = 256 N2.  Above, R = 32 (N = 1024 N2) instead of the 4096-point columns of the mixer's plan: those do not fit
// with their partners (8 pairs x 2 planes x 32 KB), and two in-register passes are shorter than three.
//
// The factors between the two passes come from a table of R x R values, copied into LDS behind the exchange buffers (2 or
// 8 KB).  As products of two to five values of the long table, which the row kernels use to save loads, they took the
// spectra of 16384 rows from 1.34e-7 to 1.42e-7 of 64 bits; with the table 1.33e-7, at the same speed (prompt of 20011
// tokens as above 2951 and 2939 us; read from memory where they are used 3015 us).
#include "fft_regs.h"
#include "internal.h"
#include "mix_pow2.h"
#include "prefix_dev.h"
#include "scratch_elem.h"

namespace spectre {

// One unit of work: two planes (k2 = u and N2 - u; for u = 0 the two planes that are their own partners, 0 and, if N2 is
// even, N2 / 2) of PW channel pairs of one head.  R adjacent lanes own a column, lane tau holds the entries k1 = tau + R v
// in register v, and the next R lanes own the same pair in the other plane: the partner of (lane, v) is then register
// R - 1 - v of a lane of the same 2 R, and no column has to stand in LDS as a whole.  LDS carries one component at a time
// of the exchange, and a half of the rows at a time on their way between lanes along k1 and lines along the pairs (whole
// 128-byte lines of X); two workgroups or more share a compute unit and fill each other's waits.
__host__ __device__ inline int cache_plane_pairs(int N2) { return (N2 + 1) / 2; }

template <int R, int PW>
struct CacheUnit {
    static constexpr int N1 = R * R, NT = 2 * PW * R, kRows = R * R / 2;   // kRows: rows of X in flight, of both planes
    static constexpr int kCol = N1 + N1 / R;                         // floats: entry e at e + e / R
    static constexpr int kRow = PW + 1;                              // float4
    static constexpr int kStep = NT / PW, kIter = kRows / kStep;
    static constexpr int kWork = 2 * PW * kCol > kRows * kRow * 4 ? 2 * PW * kCol / 4 : kRows * kRow;   // float4
    static constexpr size_t kLds = kWork * sizeof(float4) + N1 * sizeof(float2);
    static_assert(64 % (2 * R) == 0 && kRows % kStep == 0, "a wave holds whole pairs of columns");
    static_assert(N1 / 2 <= NT && 2 * PW * kCol % 4 == 0, "one lane copies two column factors, to a 16-byte boundary");
    int bhl, pg, u, planes, plane1;
    // The 32 / PW units that share the rows of X get ids 8 apart, hence one XCD.
    __device__ __forceinline__ bool init(int id, int N2, int nbh) {
        constexpr int G = 32 / PW;
        const int U = cache_plane_pairs(N2), xcd = id & 7, idx = id >> 3;
        pg = idx % G;
        const int unit = (idx / G) * 8 + xcd;
        bhl = unit / U;
        u = unit - bhl * U;
        plane1 = u ? N2 - u : N2 / 2;
        planes = (u || N2 % 2 == 0) ? 2 : 1;
        return bhl < nbh;
    }
    __device__ __forceinline__ int plane(int s) const { return s ? plane1 : u; }
    // Lane with the partners of this lane's entries, in registers R - 1 - v; for plane 0 itself that holds for tau > 0, and
    // the partner of entry R v is entry R (R - v).
    __device__ __forceinline__ int partner_lane(int lane) const {
        const int tau = lane % R, s = (lane / R) & 1, base = lane & ~(2 * R - 1);
        if (u) return base + 2 * R - 1 - (lane - base);
        return s ? base + 2 * R - 1 - tau : base + ((R - tau) & (R - 1));
    }
    // entry k1 of row rr of half h
    __device__ static __forceinline__ int row_entry(int rr, int h) { return rr % R + R * (h * (R / 4) + (rr / R) % (R / 4)); }
    __device__ static __forceinline__ int row_plane(int rr) { return rr / (R * R / 4); }
};

// x[u] at entry u R + tau -> entry tau R + i, one component at a time; LDS operations of a wave complete in order.
template <int R>
__device__ __forceinline__ void cache_exchange(float2 (&x)[R], float *buf, int tau, bool forward) {
    float *b0 = buf + tau, *b1 = buf + tau * (R + 1);
    const int s0 = forward ? R + 1 : 1, s1 = forward ? 1 : R + 1;
    float *w = forward ? b0 : b1, *r = forward ? b1 : b0;
#pragma unroll
    for (int i = 0; i < R; ++i) w[i * s0] = x[i].x;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < R; ++i) x[i].x = r[i * s1];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < R; ++i) w[i * s0] = x[i].y;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < R; ++i) x[i].y = r[i * s1];
}

__device__ __forceinline__ float2 shfl2(float2 v, int lane) { return make_float2(__shfl(v.x, lane), __shfl(v.y, lane)); }

template <int R, int PW>
__global__ __launch_bounds__(2 * PW * R, R == 32 ? 4 : 6) void k_cache_fwd(const float2 *__restrict__ scr,
                                                                           float4 *__restrict__ X,
                                                                           const float4 *__restrict__ tw, int N2,
                                                                           int bh0, int nbh) {
    typedef CacheUnit<R, PW> Unit;
    constexpr int N1 = Unit::N1, V = R / 4;
    extern __shared__ float4 lds_cc[];
    Unit un;
    if (!un.init(blockIdx.x, N2, nbh)) return;                       // whole workgroup: units are padded to 8
    const int tid = threadIdx.x, lane = tid & 63, F = N1 * N2 / 2 + 1;
    const int tau = tid % R, s = (tid / R) & 1, pw = tid / (2 * R);
    float4 factors = make_float4(0.f, 0.f, 0.f, 0.f);
    if (tid < N1 / 2) factors = tw[tid];
    float2 x[R];
    const float2 *col = scr + (((size_t)un.bhl * N2 + un.plane(s)) * 32 + un.pg * PW + pw) * N1 + tau;   // in range also
#pragma unroll                                                       // without a second plane: plane N2 / 2 twice
    for (int j = 0; j < R; ++j) x[j] = col[R * j];
    if (tid < N1 / 2) lds_cc[Unit::kWork + tid] = factors;
    dft<R, false>(x);
    __syncthreads();
    const float2 *w = reinterpret_cast<const float2 *>(lds_cc + Unit::kWork) + tau;
#pragma unroll
    for (int u = 1; u < R; ++u) x[u] = cmul(x[u], w[u * R]);         // W_N1^(tau u)
    cache_exchange<R>(x, reinterpret_cast<float *>(lds_cc) + (tid / R) * Unit::kCol, tau, true);
    dft<R, false>(x);                                                // register v: bin k1 = tau + R v
    const int src = un.partner_lane(lane);
    const bool own = un.u == 0 && s == 0 && tau == 0;
    float4 *Xh = X + (size_t)(un.bhl + bh0) * F * 32 + un.pg * PW;
    if (own) Xh[(size_t)(F - 1) * 32 + pw] = untangle_pair(x[R / 2], x[R / 2]);   // Nyquist: its own partner
    const int p = tid % PW, r0 = tid / PW;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        __syncthreads();                                             // the LDS of the exchange, of the half before
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int v = h * V + i;
            float2 n = shfl2(x[R - 1 - v], src);
            if (own) n = x[(R - v) % R];
            lds_cc[((s * V + i) * R + tau) * Unit::kRow + pw] = untangle_pair(x[v], n);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < Unit::kIter; ++i) {
            const int rr = r0 + Unit::kStep * i, sr = Unit::row_plane(rr);
            if (sr < un.planes)
                stream_store(Xh + (size_t)(un.plane(sr) + N2 * Unit::row_entry(rr, h)) * 32 + p, lds_cc[rr * Unit::kRow + p]);
        }
    }
}

// THROUGH: see through_store and cache_cols_t.
template <int R, int PW, bool THROUGH>
__global__ __launch_bounds__(2 * PW * R, R == 32 ? 4 : 6) void k_cache_inv(const float4 *__restrict__ X,
                                                                           const float2 *__restrict__ g,
                                                                           float2 *__restrict__ scr,
                                                                           const float4 *__restrict__ tw, int N2,
                                                                           int bh0, int nbh) {
    typedef CacheUnit<R, PW> Unit;
    constexpr int N1 = Unit::N1, V = R / 4;
    extern __shared__ float4 lds_cc[];
    Unit un;
    if (!un.init(blockIdx.x, N2, nbh)) return;                       // whole workgroup: units are padded to 8
    const int tid = threadIdx.x, lane = tid & 63, N = N1 * N2, F = N / 2 + 1;
    const int tau = tid % R, s = (tid / R) & 1, pw = tid / (2 * R);
    const float scale = 1.0f / (float)N;
    const float4 *Xh = X + (size_t)(un.bhl + bh0) * F * 32 + un.pg * PW;
    const float2 *gh = g + (size_t)(un.bhl + bh0) * F;
    const int src = un.partner_lane(lane);
    const bool own = un.u == 0 && s == 0 && tau == 0;
    const int p = tid % PW, r0 = tid / PW;
    if (tid < N1 / 2) lds_cc[Unit::kWork + tid] = tw[tid];
    float2 x[R];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        float4 row[Unit::kIter];
        float2 gk[Unit::kIter];
#pragma unroll
        for (int i = 0; i < Unit::kIter; ++i) {
            const int rr = r0 + Unit::kStep * i, k = un.plane(Unit::row_plane(rr)) + N2 * Unit::row_entry(rr, h);
            row[i] = stream_load(Xh + (size_t)k * 32 + p);                        // without a second plane: plane N2 / 2, unused
            gk[i] = gh[k];
        }
        if (h) __syncthreads();
#pragma unroll
        for (int i = 0; i < Unit::kIter; ++i) {
            const int rr = r0 + Unit::kStep * i;
            const bool dc = un.u == 0 && rr == 0 && h == 0;          // only the real parts count
            const TangledPair z = tangle_pair(row[i], gk[i], dc, scale);
            lds_cc[rr * Unit::kRow + p] = make_float4(z.k.x, z.k.y, z.n.x, z.n.y);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int v = h * V + i;
            const float4 z = lds_cc[((s * V + i) * R + tau) * Unit::kRow + pw];
            const float2 zn = make_float2(z.z, z.w);
            x[v] = make_float2(z.x, z.y);
            x[R - 1 - v] = shfl2(zn, src);
            if (v > 0 && own) x[R - v] = zn;
        }
    }
    if (own) x[R / 2] = tangle_pair(Xh[(size_t)(F - 1) * 32 + pw], gh[F - 1], true, scale).k;   // Nyquist
    __syncthreads();                                                 // the rows' LDS
    const float2 *w = reinterpret_cast<const float2 *>(lds_cc + Unit::kWork) + tau;
    dft<R, true>(x);
    cache_exchange<R>(x, reinterpret_cast<float *>(lds_cc) + (tid / R) * Unit::kCol, tau, false);
#pragma unroll
    for (int u = 1; u < R; ++u) x[u] = cmulc(x[u], w[u * R]);        // W_N1^(-tau u)
    dft<R, true>(x);
    if (s >= un.planes) return;
    float2 *col = scr + (((size_t)un.bhl * N2 + un.plane(s)) * 32 + un.pg * PW + pw) * N1 + tau;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (THROUGH) through_store(col + R * j, x[j]);
        else col[R * j] = x[j];
    }
}

// The mixer's columns of R * R points in place: forward, times the expanded gate gp [bh][k2][k1], inverse.  R adjacent lanes
// own a column, a workgroup PW pairs of one plane; the 32 / PW workgroups of a plane get ids 8 apart, so that its part of the
// gate meets one L2.  grid: 8 ceil(planes / 8) * 32 / PW.
// For L = 12288 ... 32768 instead of the 4096-point columns of k_big, whose three passes exchange twice across the waves of a
// workgroup: here two longer passes exchange inside 32 lanes, without a barrier.  What bounds it is memory traffic, 16 bytes
// per pair and position: 32 heads of L = 24576 94 -> 73 us (403 MB, 5.5 TB/s).
// THROUGH: see through_store and launch_mix_cols.
template <int R, int PW, bool THROUGH>
__global__ __launch_bounds__(PW * R, 3) void k_mix_cols(float2 *__restrict__ scr, const float2 *__restrict__ gp,
                                                        const float4 *__restrict__ tw, int N2, int bh0, int planes) {
    constexpr int N1 = R * R, NT = PW * R, kCol = N1 + N1 / R, G = 32 / PW;
    static_assert(PW * kCol % 4 == 0 && N1 / 2 % NT == 0, "the factors on a 16-byte boundary, whole sweeps of them");
    extern __shared__ float4 lds_cc[];
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int pg = idx % G, plane = (idx / G) * 8 + xcd;
    if (plane >= planes) return;                                     // whole workgroup: planes are padded to 8
    const int tid = threadIdx.x, tau = tid % R, pw = tid / R;
    float2 *col = scr + ((size_t)plane * 32 + pg * PW + pw) * N1 + tau;
    float2 x[R];
#pragma unroll
    for (int j = 0; j < R; ++j) x[j] = col[R * j];
    float4 *wl = lds_cc + PW * kCol / 4;
#pragma unroll
    for (int i = 0; i < N1 / 2 / NT; ++i) wl[tid + NT * i] = tw[tid + NT * i];
    dft<R, false>(x);
    __syncthreads();
    const float2 *w = reinterpret_cast<const float2 *>(wl) + tau;
    float *buf = reinterpret_cast<float *>(lds_cc) + pw * kCol;
#pragma unroll
    for (int u = 1; u < R; ++u) x[u] = cmul(x[u], w[u * R]);         // W_N1^(tau u)
    cache_exchange<R>(x, buf, tau, true);
    dft<R, false>(x);                                                // register v: bin k1 = tau + R v
    const float2 *gsrc = gp + ((size_t)bh0 * N2 + plane) * N1 + tau;
#pragma unroll
    for (int v = 0; v < R; ++v) x[v] = cmul(x[v], gsrc[R * v]);
    dft<R, true>(x);
    __builtin_amdgcn_wave_barrier();
    cache_exchange<R>(x, buf, tau, false);
#pragma unroll
    for (int u = 1; u < R; ++u) x[u] = cmulc(x[u], w[u * R]);
    dft<R, true>(x);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (THROUGH) through_store(col + R * j, x[j]);
        else col[R * j] = x[j];
    }
}

// ------------------------------------------------------------------------------------------
bool cache_cols_split(int N, int *N1, int *N2) {
    for (int n1 : {256, 1024}) {
        if (N % n1 == 0 && N / n1 <= 32 && small_dft_supported(N / n1)) {
            *N1 = n1;
            *N2 = N / n1;
            return true;
        }
    }
    return false;
}

template <int R, int PW>
static hipError_t cache_cols_t(bool inverse, const Pow2Plan &pl, float2 *scr, float2 *X, const float2 *g, int bh0, int nbh,
                               hipStream_t st) {
    typedef CacheUnit<R, PW> Unit;
    const size_t lds = Unit::kLds;
    const long long units = ((long long)nbh * cache_plane_pairs(pl.N2) + 7) / 8 * 8 * (32 / PW);
    if (units > 0x7fffffffLL) return hipErrorInvalidValue;
    // The inverse writes its columns through the L2, except those of 256 points of windows of 2560 slots and more, 18 MB to what the eight L2s
    // hold: there the readout's row transforms find them after plain stores.  Readout of a window, us, plain / through: 12 heads of N = 8192 (24
    // MB) 22.8 / 23.6, 18 of 6144 (27 MB) 26.7 / 27.8, 20 of 5120 (25 MB) 23.1 / 24.1, 32 of 4096 (32 MB) 27.7 / 28.0, 50 of 2560 (31 MB) 25.1 /
    // 25.5; but 9 of 8192 (18 MB) 22.1 / 22.3, 8 22.1 / 20.1; 17 (34 MB) 33.8 / 33.1, 26 of 5120 (32.5 MB) 31.9 / 29.6, 40 of 4096 (40 MB) 34.2 /
    // 32.7, 128 of 8192 174 / 171; 64 of 2048 (32 MB) 25.8 / 25.3, 40 (20 MB) 19.9 / 19.4, 150 of 512 (19 MB) 19.5 / 19.0.  Of 1024 points: 3 heads of
    // 24576 (18 MB) 27.8 / 25.6, 4 of 32768 (32 MB) 30.9 / 30.5, 6 (48 MB) 44.6 / 42.1.
    const size_t bytes = (size_t)nbh * pl.N1 * pl.N2 * 32 * sizeof(float2);
    const bool found = R == 16 && pl.N2 >= 10 && bytes >= ((size_t)18 << 20) && bytes <= kL2Bytes, through = !found;
    auto inv = through ? k_cache_inv<R, PW, true> : k_cache_inv<R, PW, false>;
    const void *kern = inverse ? reinterpret_cast<const void *>(inv)
                               : reinterpret_cast<const void *>(&k_cache_fwd<R, PW>);
    const hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    float4 *X4 = reinterpret_cast<float4 *>(X);
    const float4 *tw = reinterpret_cast<const float4 *>(pl.twN1);
    const unsigned grid = (unsigned)units;
    if (inverse) inv<<<grid, Unit::NT, lds, st>>>(X4, g, scr, tw, pl.N2, bh0, nbh);
    else k_cache_fwd<R, PW><<<grid, Unit::NT, lds, st>>>(scr, X4, tw, pl.N2, bh0, nbh);
    return hipGetLastError();
}

static hipError_t cache_cols(bool inverse, const Pow2Plan &pl, float2 *scr, float2 *X, const float2 *g, int bh0, int nbh,
                             hipStream_t st) {
    if (pl.N1 == 256) return cache_cols_t<16, 16>(inverse, pl, scr, X, g, bh0, nbh, st);
    if (pl.N1 == 1024) return cache_cols_t<32, 8>(inverse, pl, scr, X, g, bh0, nbh, st);
    return hipErrorInvalidValue;
}

hipError_t launch_cache_fwd(const Pow2Plan &pl, const float2 *scr, float2 *X, int bh0, int nbh, hipStream_t st) {
    return cache_cols(false, pl, const_cast<float2 *>(scr), X, nullptr, bh0, nbh, st);
}

hipError_t launch_cache_inv(const Pow2Plan &pl, const float2 *X, const float2 *g, float2 *scr, int bh0, int nbh,
                            hipStream_t st) {
    return cache_cols(true, pl, scr, const_cast<float2 *>(X), g, bh0, nbh, st);
}

hipError_t launch_mix_cols(const Pow2Plan &pl, float2 *scr, const float2 *gp, int bh0, int nbh, hipStream_t st, bool alone) {
    constexpr int R = 32, PW = 8;
    if (pl.N1 != R * R) return hipErrorInvalidValue;
    const size_t lds = (size_t)PW * (pl.N1 + R) * sizeof(float) + (size_t)pl.N1 * sizeof(float2);
    const int planes = nbh * pl.N2;
    // through_store for launches of up to 128 MB that have memory to themselves (mixer of bf16 rows, us, plain / through: one head at 24576 (6 MB)
    // 28.9 / 26.8, 8 at 28672 (59 MB) 3 %, 32 at 12288 (100 MB) 95.9 / 92.8, 40 (126 MB) 1 %; 48 to 128 heads at 12288 to 28672 -0.3 %, layer
    // of 24576 (201 MB) 318.8 / 324.2)
    const auto kern = alone && (size_t)planes * 32 * R * R * sizeof(float2) <= ((size_t)128 << 20) ? k_mix_cols<R, PW, true> : k_mix_cols<R, PW, false>;
    kern<<<(planes + 7) / 8 * 8 * (32 / PW), PW * R, lds, st>>>(scr, gp, reinterpret_cast<const float4 *>(pl.twN1), pl.N2, bh0, planes);
    return hipGetLastError();
}

// Loads this translation unit's code object (the runtime loads them on first use): called by spectre_prepare so
// that no compute call is the first to touch it.
hipError_t load_kernels_cache_cols() {
    hipFuncAttributes a;
    return hipFuncGetAttributes(&a, reinterpret_cast<const void *>(&k_cache_fwd<16, 16>));
}

}  // namespace spectre
