// Arbitrary-length mixing through the four-step kernels: chirp-z evaluation of the per-head
// convolution kernel and its embedding in a padded convolution of a four-step length.
#include "mix_chirp.h"

#include <cmath>
#include <complex>
#include <vector>

#include "fft_regs.h"
#include "mix_pow2.h"

namespace spectre {

int chirp_padded_length(int L) {
    if (L < 1 || L > 65536) return 0;
    const int need = 2 * L - 1;
    int best = 0;
    for (int N1 : {256, 4096})
        for (int N2 = 1; N2 <= 32; ++N2) {
            const int M = N1 * N2;
            int a, b, c;
            if (M >= need && (best == 0 || M < best) && pow2_split(M, &a, &b, &c)) best = M;
        }
    return best;
}

__global__ __launch_bounds__(256) void k_chirp_pre(const float2 *__restrict__ g, const float2 *__restrict__ w,
                                                   float2 *__restrict__ A, int BH, int L, int nph, size_t total) {
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int p = (int)(idx % 32);
    const size_t r = idx / 32;
    const int ph = (int)(r % nph), k = (int)(r / nph);
    const int bh = ph * 32 + p, F = L / 2 + 1;
    float2 val = make_float2(0.f, 0.f);
    if (bh < BH) {
        float2 ge;
        if (k == 0 || 2 * k == L) ge = make_float2(g[(size_t)bh * F + k].x, 0.f);
        else if (2 * k < L) ge = g[(size_t)bh * F + k];
        else ge = cconj(g[(size_t)bh * F + (L - k)]);
        val = cmul(ge, w[k]);
    }
    A[idx] = val;
}

__global__ __launch_bounds__(256) void k_chirp_post(const float2 *__restrict__ U, const float2 *__restrict__ w,
                                                    float2 *__restrict__ KK, int L, int M, int nph, size_t total) {
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const size_t lane = idx % ((size_t)nph * 32);
    const int i = (int)(idx / ((size_t)nph * 32));
    int m = -1;
    if (i < L) m = i;
    else if (i > M - L) m = i - (M - L);
    float kap = 0.f;
    if (m >= 0) {
        const float2 u = U[(size_t)m * nph * 32 + lane], wm = w[m];
        kap = (wm.x * u.x - wm.y * u.y) * (1.0f / (float)L);
    }
    KK[idx] = make_float2(kap, 0.f);
}

__global__ __launch_bounds__(256) void k_chirp_gate(const float2 *__restrict__ scr, float2 *__restrict__ gp, int BH,
                                                    int N1, int N2, int ph0, float scale, size_t total) {
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int r = (int)(idx % N1);
    const size_t q = idx / N1;
    const int k2 = (int)(q % N2);
    const size_t lh = q / N2;                         // head index within this group of pseudo-heads
    const int phl = (int)(lh / 32), p = (int)(lh % 32);
    const size_t bh = (size_t)ph0 * 32 + lh;
    if (bh >= (size_t)BH) return;
    const float2 z = scr[(((size_t)phl * N2 + k2) * 32 + p) * N1 + r];   // same entry order on both sides
    gp[(bh * N2 + k2) * N1 + r] = make_float2(z.x * scale, z.y * scale);
}

// Short padded lengths (M = 256 N2 <= 2048, where the data pass is one in-LDS launch): everything between the caller's
// gate and the gate of the data pass - chirp, two transforms around the filter, periodic extension, one more transform -
// in one launch, a head's column in LDS from start to end.  16 N2 lanes per head, 16 points per lane in every pass: the
// N2-point transforms of the row kernels, then the two radix-16 passes of the 256-point columns (register j of lane tau
// of column k2 holds bin k2 + N2 (16 j + tau), the order of the filter table).
// What bounds it is the latency of this chain of passes.  As eight launches of the kernels of longer lengths, each with
// a few microseconds of work, it took a third of the call: L = 197, 768 heads of fp32 rows, 71.4 -> 53.0 us.
template <int N2> constexpr int kChirpHeads = N2 < 4 ? 4 : 1;        // heads per workgroup: at least a wave of lanes

template <int N2>
struct ChirpColumn {
    static constexpr int M = 256 * N2, NL = 16 * N2, COLW = 272;     // entry e of a column at e + e / 16
    static constexpr int kLds = N2 * COLW * 8 + M / 2 * 4;           // bytes per head: the columns, then kappa (L <= M / 2)
    float2 *buf;
    int t, tau;
    float2 tw[15];                                                   // W_256^(tau u)
    __device__ __forceinline__ float2 *own() const { return buf + (t >> 4) * COLW; }
    // the lane's rows in batches of kBatch whose loads are all under way before the first is used: one row at a time, each waited
    // for memory on its own
    static constexpr int kTrips = (256 + NL - 1) / NL, kBatch = N2 == 1 ? 8 : N2 == 2 ? 4 : N2 == 3 ? 3 : N2 == 6 || N2 == 7 ? 1 : 2;
    template <typename L, typename F>
    __device__ __forceinline__ void rows_fwd(const float2 *twM, L load, F element) {
#pragma unroll 1
        for (int q0 = 0; q0 < kTrips; q0 += kBatch) {
            decltype(load(0)) raw[kBatch][N2];
            float2 tw_row[kBatch][N2];
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                const int t1 = min(t + NL * (q0 + q), 255);
#pragma unroll
                for (int j = 0; j < N2; ++j) raw[q][j] = load(t1 + 256 * j);
#pragma unroll
                for (int k2 = 1; k2 < N2; ++k2) tw_row[q][k2] = *lane_pointer(twM, 8u * (t1 * k2));
            }
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                const int t1 = t + NL * (q0 + q);
                float2 x[N2];
#pragma unroll
                for (int j = 0; j < N2; ++j) x[j] = element(min(t1, 255) + 256 * j, raw[q][j]);
                small_dft<N2, false>(x);
                if (256 % NL == 0 || t1 < 256) {
#pragma unroll
                    for (int k2 = 0; k2 < N2; ++k2) buf[k2 * COLW + t1 + (t1 >> 4)] = k2 == 0 ? x[0] : cmul(x[k2], tw_row[q][k2]);
                }
            }
        }
    }
    __device__ __forceinline__ void cols_fwd(float2 (&y)[16]) {
        float2 *c = own();
#pragma unroll
        for (int j = 0; j < 16; ++j) y[j] = c[tau + 17 * j];
        dft<16, false>(y);
#pragma unroll
        for (int u = 0; u < 16; ++u) c[tau + 17 * u] = u == 0 ? y[0] : cmul(y[u], tw[u - 1]);
        __builtin_amdgcn_wave_barrier();                             // 16 lanes of one wave; its LDS operations keep their order
#pragma unroll
        for (int j = 0; j < 16; ++j) y[j] = c[17 * tau + j];
        dft<16, false>(y);
    }
    __device__ __forceinline__ void cols_inv(float2 (&y)[16]) {
        float2 *c = own();
        dft<16, true>(y);
#pragma unroll
        for (int j = 0; j < 16; ++j) c[17 * tau + j] = y[j];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < 16; ++u) y[u] = u == 0 ? c[tau] : cmulc(c[tau + 17 * u], tw[u - 1]);
        dft<16, true>(y);
#pragma unroll
        for (int j = 0; j < 16; ++j) c[tau + 17 * j] = y[j];
    }
};

// gp [BH][D / 2 + 1] = the data pass's gate in plain bin order, unscaled (the in-LDS kernel divides by its length), D
// the length of that pass: M itself (R0 = 0) or R0 R1 < M, for which this last transform is two passes of its own with
// rootsD [D] = exp(-j 2 pi m / D).
template <int N2, int R0, int R1>
__global__ __launch_bounds__(16 * N2 * kChirpHeads<N2>) void k_chirp_lds(const float2 *__restrict__ g,
                                                                        const float2 *__restrict__ w,
                                                                        const float2 *__restrict__ filt,
                                                                        const float2 *__restrict__ twM,
                                                                        const float2 *__restrict__ rootsD,
                                                                        float2 *__restrict__ gp, int BH, int L) {
    typedef ChirpColumn<N2> Col;
    constexpr int M = Col::M, HW = kChirpHeads<N2>, D = R0 ? R0 * R1 : M;
    static_assert(R0 * (R1 + 1) <= N2 * Col::COLW, "the last transform's column fits where the others were");
    __shared__ __align__(16) unsigned char lds[HW * Col::kLds];
    const int hl = threadIdx.x / Col::NL, bh = blockIdx.x * HW + hl;
    const bool live = bh < BH;                                       // the others run along on head 0 and store nothing
    Col col;
    col.buf = reinterpret_cast<float2 *>(lds + hl * Col::kLds);
    col.t = threadIdx.x % Col::NL;
    col.tau = col.t & 15;
    float *kap = reinterpret_cast<float *>(col.buf + N2 * Col::COLW);
    const int t = col.t, tau = col.tau, k2 = t >> 4;
    const float2 *gh = g + (size_t)(live ? bh : 0) * (L / 2 + 1);
#pragma unroll
    for (int u = 1; u < 16; ++u) col.tw[u - 1] = twM[N2 * tau * u];
    float2 f[16], y[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) f[j] = filt[256 * k2 + 16 * j + tau];

    struct GateTimesChirp {
        float2 g, w;
    };
    col.rows_fwd(twM,
        [&](int k) {
            const int at = min(k, L - 1);
            return GateTimesChirp{gh[2 * at <= L ? at : L - at], *lane_pointer(w, 8u * at)};
        },
        [&](int k, GateTimesChirp v) {
            if (k >= L) return make_float2(0.f, 0.f);
            if (2 * k > L) v.g.y = -v.g.y;
            if (k == 0 || 2 * k == L) v.g.y = 0.f;
            return cmul(v.g, v.w);
        });
    __syncthreads();
    col.cols_fwd(y);
#pragma unroll
    for (int j = 0; j < 16; ++j) y[j] = cmul(y[j], f[j]);
    col.cols_inv(y);
    __syncthreads();
#pragma unroll 1
    for (int q0 = 0; q0 < Col::kTrips; q0 += Col::kBatch) {
        float2 tw_row[Col::kBatch][N2], wm[Col::kBatch][N2];
#pragma unroll
        for (int q = 0; q < Col::kBatch; ++q) {
            const int t1 = min(t + Col::NL * (q0 + q), 255);
#pragma unroll
            for (int j = 0; j < N2; ++j) {
                if (j) tw_row[q][j] = *lane_pointer(twM, 8u * (t1 * j));
                wm[q][j] = *lane_pointer(w, 8u * min(t1 + 256 * j, L - 1));
            }
        }
#pragma unroll
        for (int q = 0; q < Col::kBatch; ++q) {
            const int t1 = t + Col::NL * (q0 + q), at = min(t1, 255);
            float2 x[N2];
#pragma unroll
            for (int j = 0; j < N2; ++j) {
                const float2 b = col.buf[j * Col::COLW + at + (at >> 4)];
                x[j] = j == 0 ? b : cmulc(b, tw_row[q][j]);
            }
            small_dft<N2, true>(x);
#pragma unroll
            for (int j = 0; j < N2; ++j) {
                const int m = t1 + 256 * j;
                if (t1 < 256 && m < L) kap[m] = (wm[q][j].x * x[j].x - wm[q][j].y * x[j].y) * (1.0f / (float)L);
            }
        }
    }
    __syncthreads();
    auto extended = [&](int i) {
        return make_float2(i < L ? kap[i] : i > D - L ? kap[i - (D - L)] : 0.f, 0.f);
    };
    float2 *gh_out = gp + (size_t)bh * (D / 2 + 1);
    if constexpr (R0 != 0) {
        for (int i = t; i < R1; i += Col::NL) {                      // positions i + R1 j, padded by one per block of R1
            float2 x[R0];
#pragma unroll
            for (int j = 0; j < R0; ++j) x[j] = extended(i + R1 * j);
            small_dft<R0, false>(x);
#pragma unroll
            for (int u = 0; u < R0; ++u) col.buf[u * (R1 + 1) + i] = u == 0 ? x[0] : cmul(x[u], rootsD[i * u]);
        }
        __syncthreads();
        for (int blk = t; blk < R0; blk += Col::NL) {
            float2 x[R1];
#pragma unroll
            for (int j = 0; j < R1; ++j) x[j] = col.buf[blk * (R1 + 1) + j];
            small_dft<R1, false>(x);
#pragma unroll
            for (int u = 0; u < R1; ++u) {
                const int k = blk + R0 * u;
                if (live && 2 * k <= D) gh_out[k] = x[u];
            }
        }
    } else {
        col.rows_fwd(twM, extended, [](int, float2 v) { return v; });
        __syncthreads();
        col.cols_fwd(y);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int k = k2 + N2 * (16 * j + tau);
            if (live && 2 * k <= D) gh_out[k] = y[j];
        }
    }
}

hipError_t launch_chirp_lds(const float2 *g, const float2 *w, const float2 *filt, const float2 *twM, const float2 *rootsD,
                            float2 *gp, int BH, int L, int M, hipStream_t st) {
    if (M != chirp_padded_length(L)) return hipErrorInvalidValue;
#define SPECTRE_CHIRP(D, N2, R0, R1)                                                                                       \
    case D:                                                                                                                \
        k_chirp_lds<N2, R0, R1><<<(BH + kChirpHeads<N2> - 1) / kChirpHeads<N2>, 16 * N2 * kChirpHeads<N2>, 0, st>>>(       \
            g, w, filt, twM, rootsD, gp, BH, L);                                                                           \
        break;
    switch (chirp_data_length(L)) {
        SPECTRE_CHIRP(256, 1, 0, 0)
        SPECTRE_CHIRP(320, 2, 20, 16) SPECTRE_CHIRP(400, 2, 20, 20) SPECTRE_CHIRP(448, 2, 28, 16) SPECTRE_CHIRP(512, 2, 0, 0)
        SPECTRE_CHIRP(640, 3, 20, 32) SPECTRE_CHIRP(768, 3, 0, 0)
        SPECTRE_CHIRP(896, 4, 28, 32) SPECTRE_CHIRP(1024, 4, 0, 0)
        SPECTRE_CHIRP(1280, 5, 0, 0) SPECTRE_CHIRP(1536, 6, 0, 0) SPECTRE_CHIRP(1792, 7, 0, 0) SPECTRE_CHIRP(2048, 8, 0, 0)
        default: return hipErrorInvalidValue;
    }
#undef SPECTRE_CHIRP
    return hipGetLastError();
}

hipError_t launch_chirp_pre(const float2 *g, const float2 *w, float2 *A, int BH, int L, int nph, hipStream_t st) {
    const size_t total = (size_t)L * nph * 32;
    k_chirp_pre<<<(unsigned)((total + 255) / 256), 256, 0, st>>>(g, w, A, BH, L, nph, total);
    return hipGetLastError();
}

hipError_t launch_chirp_post(const float2 *U, const float2 *w, float2 *KK, int L, int M, int nph, hipStream_t st) {
    const size_t total = (size_t)M * nph * 32;
    k_chirp_post<<<(unsigned)((total + 255) / 256), 256, 0, st>>>(U, w, KK, L, M, nph, total);
    return hipGetLastError();
}

hipError_t launch_chirp_gate(const float2 *scr, float2 *gp, int BH, int M, int N1, int N2, int ph0, int nphl,
                             hipStream_t st) {
    const size_t total = (size_t)nphl * 32 * N2 * N1;
    k_chirp_gate<<<(unsigned)((total + 255) / 256), 256, 0, st>>>(scr, gp, BH, N1, N2, ph0, 1.0f / (float)M, total);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------ host tables
// Forward DFT of n = 2^a 3^b 5^c 7^d points (decimation in time, smallest prime factor first), out of place.
// root[j] = exp(-j 2 pi j / top) for the top-level length, of which n is a divisor.
static void fft_host(const std::complex<double> *in, size_t stride, size_t n, std::complex<double> *out,
                     const std::vector<std::complex<double>> &root) {
    if (n == 1) {
        out[0] = in[0];
        return;
    }
    const size_t top = root.size();
    size_t p = 2;
    while (n % p != 0) ++p;
    const size_t m = n / p;
    for (size_t r = 0; r < p; ++r) fft_host(in + r * stride, stride * p, m, out + r * m, root);
    std::complex<double> col[7];
    for (size_t k = 0; k < m; ++k) {
        for (size_t r = 0; r < p; ++r) col[r] = out[r * m + k] * root[(r * k) * (top / n)];
        for (size_t q = 0; q < p; ++q) {
            std::complex<double> acc = col[0];
            for (size_t r = 1; r < p; ++r) acc += col[r] * root[((r * q) % p) * (top / p)];
            out[k + q * m] = acc;
        }
    }
}

void chirp_tables_host(int L, int M, int N1, int N2, int P, float2 *w, float2 *filt) {
    std::vector<std::complex<double>> wd(L), f(M, std::complex<double>(0.0, 0.0));
    for (int n = 0; n < L; ++n) {
        const long long sq = ((long long)n * n) % (2LL * L);       // exact phase index
        wd[n] = std::polar(1.0, M_PI * (double)sq / (double)L);
        w[n] = make_float2((float)wd[n].real(), (float)wd[n].imag());
    }
    std::vector<std::complex<double>> ft(M, std::complex<double>(0.0, 0.0));
    ft[0] = std::conj(wd[0]);
    for (int i = 1; i < L; ++i) ft[i] = ft[M - i] = std::conj(wd[i]);
    std::vector<std::complex<double>> root(M);
    for (int j = 0; j < M; ++j) root[j] = std::polar(1.0, -2.0 * M_PI * (double)j / (double)M);
    fft_host(ft.data(), 1, (size_t)M, f.data(), root);
    for (int k2 = 0; k2 < N2; ++k2)
        for (int r = 0; r < N1; ++r) {
            const int k = k2 + N2 * big_position(r, P);
            filt[(size_t)k2 * N1 + r] = make_float2((float)(f[k].real() / M), (float)(f[k].imag() / M));
        }
}

// Loads this translation unit's code object (the runtime loads them on first use): called by spectre_prepare so
// that no compute call is the first to touch it.
hipError_t load_kernels_mix_chirp() {
    hipFuncAttributes a;
    return hipFuncGetAttributes(&a, reinterpret_cast<const void *>(k_chirp_pre));
}

}  // namespace spectre
