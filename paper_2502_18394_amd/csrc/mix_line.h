// Whole columns on one compute unit (bf16 rows, lengths 8192 and 16384): launch declarations.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace spectre {

bool line_supported(int L, int io);   // io 1 = bf16 rows
// v, out = tensors [B, L, H, 64] of bf16; g = gate [B*H, L/2+1]; scratch for the heads bh0 .. bh0 + nbh - 1:
// gp [nbh][L] complex, lines [nbh][32][L] channel pairs; twL = device table [L] of exp(-j 2 pi m / L).
hipError_t launch_mix_line(const void *v, const float2 *g, void *out, float2 *gp, void *lines, const float2 *twL, int L,
                           int H, int bh0, int nbh, hipStream_t st);
hipError_t load_kernels_mix_line();

// Heads per launch of launch_mix_line when at most `most` fit its scratch: as few groups as that allows, all but the last a
// multiple of eight heads (an XCD takes every eighth head), and equal as far as that goes.
constexpr int line_group_heads(int BH, int most) {
    if (BH <= most) return BH;
    const int n = (BH + most - 1) / most, equal = (BH + n - 1) / n, eights = (equal + 7) / 8 * 8;
    return eights <= most ? eights : equal;
}

// Workgroups per XCD of the column kernel, two per compute unit at 8192 and one at 16384, but no more than it has lines.
constexpr int line_workgroups(int L, int nbh) {
    const int places = L == 8192 ? 64 : 32, lines = 32 * ((nbh + 7) / 8);
    return lines < places ? lines : places;
}
// Lines [first, first + count) of workgroup j of `wgs` on XCD xcd; line n is pair n % 32 of the XCD's head n / 32, that is
// head 8 (n / 32) + xcd of the group.  Workgroups wgs / 2 apart share a compute unit, so it is the first ones that take one
// more.
struct LineShare {
    int first, count;
};
__host__ __device__ inline LineShare line_share(int xcd, int j, int wgs, int nbh) {
    const int own = 32 * ((nbh - xcd + 7) / 8), q = own / wgs, r = own % wgs;
    return {j * q + (j < r ? j : r), q + (j < r ? 1 : 0)};
}

}  // namespace spectre
