// Mixing layer for sequence lengths with no four-step or in-LDS plan (Sec. 3.2 steps 2-4).
//
// By App. B the layer is a circular convolution of every channel with one real kernel per head,
// kappa = irfft_L(gate).  A length-L circular convolution equals the first L outputs of a
// length-M circular convolution (M >= 2L-1 a length the four-step kernels serve) of the zero-padded signal with the
// periodic extension kk of kappa laid out around index 0, so the data go through the
// four-step kernels once, with rfft_M(kk) as their gate.  kappa itself, one sequence per
// head, is an L-point inverse DFT of arbitrary L; it is evaluated by the chirp-z identity
//   exp(+j 2 pi k m / L) = w_k w_m conj(w_{m-k}),  w_n = exp(+j pi n^2 / L)
// which turns it into one more length-M circular convolution, with a fixed chirp filter.
// The heads' gate sequences ride through the same kernels as the 32 channel pairs of
// pseudo-heads (32 heads per pseudo-head, complex fp32 rows).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace spectre {

// Smallest four-step length M >= max(2L-1, 256); 0 if there is none (L > 65536).
int chirp_padded_length(int L);

// A[k][ph][p] = ext(g[bh])[k] * w_k, bh = 32 ph + p (zero for bh >= BH); ext = Hermitian extension
// of the half spectrum with real DC and Nyquist bins.  g [BH, L/2+1], w [L], A [L, nph, 32].
hipError_t launch_chirp_pre(const float2 *g, const float2 *w, float2 *A, int BH, int L, int nph, hipStream_t st);
// kappa[m] = Re(w_m U[m]) / L, laid out as kk over M rows: KK[i] = kappa[i] (i < L),
// kappa[i - (M - L)] (i > M - L), else 0; imaginary parts zero.  U [L, nph, 32], KK [M, nph, 32].
hipError_t launch_chirp_post(const float2 *U, const float2 *w, float2 *KK, int L, int M, int nph, hipStream_t st);
// Forward-transformed pseudo-head columns (scratch layout of the big kernel, pseudo-heads
// ph0 .. ph0+nphl) -> per-head gate planes gp [BH][N2][N1] in the big kernel's register order,
// scaled by 1/M.
hipError_t launch_chirp_gate(const float2 *scr, float2 *gp, int BH, int M, int N1, int N2, int ph0, int nphl,
                             hipStream_t st);

// Length D of the data pass for L <= 1024 (>= 2L-1, at most the padded length); 0: none.  In-LDS lengths of compile-time radices,
// which have a form for half the rows (mix_slab.hip): the padded lengths of the chirp, multiples of 256, are up to a third longer
// (B=64 H=12 fp32: L = 197 on 400 instead of 512 points 53.2 -> 41.8 us, L = 157 on 320 51 -> 32).
constexpr int kChirpDataLengths[] = {256, 320, 400, 448, 512, 640, 768, 896, 1024, 1280, 1536, 1792, 2048};
inline int chirp_data_length(int L) {
    for (int D : kChirpDataLengths)
        if (D >= 2 * L - 1) return D;
    return 0;
}
constexpr bool chirp_uses(int D) {
    for (int x : kChirpDataLengths)
        if (x == D) return true;
    return false;
}
// All of that in one launch for L <= 1024: g [BH, L/2+1] -> gp [BH][D/2+1] in plain bin order, unscaled, the gate argument
// of the in-LDS kernel when it runs the padded convolution.  twM [M] = exp(-j 2 pi m / M), rootsD the same for D.
hipError_t launch_chirp_lds(const float2 *g, const float2 *w, const float2 *filt, const float2 *twM, const float2 *rootsD,
                            float2 *gp, int BH, int L, int M, hipStream_t st);

// Host: chirp w [L] and the chirp filter's M-point spectrum in the big kernel's register order
// ([N2][N1], scaled by 1/M), both evaluated in fp64.
void chirp_tables_host(int L, int M, int N1, int N2, int P, float2 *w, float2 *filt);

}  // namespace spectre
