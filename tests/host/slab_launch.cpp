// Host check of slab_launch_heads (csrc/mix_slab.h): every launch of a split call stays below 2^32 lanes, takes whole groups
// of 8 heads, and the launches cover every head once.
#include <stdio.h>

#include "mix_slab.h"

int main() {
    int fails = 0;
    const long long heads[] = {1, 7, 8, 4095, (1 << 21) - 1, 1 << 21, (1 << 21) + 9, 3 << 21, 0x7fffff00};
    for (int parts : {1, 2, 4, 8, 16})
        for (int lanes : {64, 192, 256, 448, 512, 1024}) {
            const long long most = spectre::slab_launch_heads(parts, lanes);
            if (most < 8 || most % 8 != 0) ++fails;
            for (long long BH : heads) {
                long long covered = 0;
                for (long long bh0 = 0; bh0 < BH; bh0 += most) {
                    const long long n = BH - bh0 < most ? BH - bh0 : most, grid = (n + 7) / 8 * 8 * parts;
                    if (grid * lanes >= (1LL << 32) || grid > 0x7fffffff) ++fails;
                    covered += n;
                }
                if (covered != BH) ++fails;
            }
        }
    printf("slab launches: %d failures\n", fails);
    return fails != 0;
}
