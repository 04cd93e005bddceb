// Short-sequence (whole slab in LDS) mixer path: host-side declarations.
#pragma once
#include <hip/hip_runtime.h>

#include "mix_chirp.h"

namespace spectre {

constexpr int kSlabMaxL = 2048;

// True if L <= kSlabMaxL and L = 2^a 3^b 5^c 7^d.
bool slab_supported(int L);

// Host: bin_of_pos[p] = the bin held by position p after the forward passes (mixed-radix digit reversal).
void slab_bin_order(int L, int *bin_of_pos);

// Whether the kernels of compile-time radices take `rows` rows per sequence for an L-point transform: all of them, or at most half at the
// lengths that have a form which knows which rows are zero, the padded convolution's.  The other form reads and writes L rows.
inline bool slab_ct_rows(int L, int rows) { return rows == L || (2 * rows <= L && chirp_uses(L)); }

// Heads per launch, a multiple of 8, of a kernel with `parts` workgroups of `lanes` lanes to a head: the runtime takes fewer
// than 2^32 lanes a launch (2^21 heads of 448 or 512 points, 230 to 275 GB of bf16 rows in and out, reach that).
inline int slab_launch_heads(int parts, int lanes) {
    return (int)(0xffffffffLL / ((long long)parts * lanes) / 8 * 8);
}

// out = irfft_L(g * rfft_L(v)) for d = 64; roots = device table [L] of exp(-j 2 pi m / L), bin_of_pos = device
// copy of slab_bin_order(L).  With 0 < rows < L the tensors hold `rows` rows per sequence: v is taken as followed
// by L - rows zero rows and only the first `rows` rows of the result are written.
hipError_t launch_mix_slab(int io, const void *v, const float2 *g, void *out, const float2 *roots,
                           const int *bin_of_pos, int B, int L, int H, hipStream_t st, int rows = 0);

}  // namespace spectre
