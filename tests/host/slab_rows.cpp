// Host check of slab_ct_rows (csrc/mix_slab.h): fewer rows than the transform only at the lengths of the padded convolution, and there
// every sequence length that it is used for.
#include <stdio.h>

#include "mix_slab.h"

int main() {
    int fails = 0;
    for (int L = 1; L <= 1024; ++L) {
        const int D = spectre::chirp_data_length(L);
        if (D < 2 * L - 1 || !spectre::slab_ct_rows(D, L)) ++fails;
    }
    for (int L = 2; L <= spectre::kSlabMaxL; ++L) {
        bool padded = false;
        for (int l = 1; l <= 1024; ++l) padded = padded || spectre::chirp_data_length(l) == L;
        for (int rows = 1; rows < L; ++rows)
            if (spectre::slab_ct_rows(L, rows) && (!padded || 2 * rows > L)) ++fails;
        if (!spectre::slab_ct_rows(L, L)) ++fails;
    }
    printf("slab rows: %d failures\n", fails);
    return fails != 0;
}
