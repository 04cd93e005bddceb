// Whole columns on one compute unit (bf16 rows, lengths 8192 and 16384): launch declarations.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace spectre {

// io 1 = bf16 rows; the rows move in 16-byte pieces, so tensors that start elsewhere take the four-step route
bool line_supported(int L, int io, const void *v, const void *out);
// v, out = tensors [B, L, H, 64] of bf16; g = gate [B*H, L/2+1]; scratch for the heads bh0 .. bh0 + nbh - 1:
// gp [nbh][L] complex, lines [nbh][32][L] channel pairs; twL = device table [L] of exp(-j 2 pi m / L).
hipError_t launch_mix_line(const void *v, const float2 *g, void *out, float2 *gp, void *lines, const float2 *twL, int L,
                           int H, int bh0, int nbh, hipStream_t st);
hipError_t load_kernels_mix_line();

}  // namespace spectre
