// Host check of how the gate's output layer is launched (csrc/gate.h).  The tiles of the grid cover the weights' rows, and the two
// rows behind the last whole tile ride with another workgroup only where that takes all their sums side by side (four) and
// the compute units then have less to do.  The hidden layer is formed inside that launch only while what its workgroups repeat is
// bounded: 32 MB of chunk sums, and eight dependent trips of a wave through them.
#include <stdio.h>

#include "gate.h"

using namespace spectre;

int main() {
    int fails = 0, cases = 0, rides = 0, inside = 0;
    alignas(16) static float weights[4];
    for (int B : {1, 2, 3, 4, 5, 8, 16, 33, 250, 2048})
        for (int H : {1, 2, 3, 4, 12, 32, 4096})
            for (int Hg : {1, H})
                for (int dg : {37, 64, 100})
                    for (int n : {2, 62, 63, 64, 65, 196, 197, 1024, 8192, 20480, 33000, 131072})
                        for (int off : {0, 1}) {
                            GateDev P = {};
                            P.Hg = Hg, P.d = 64, P.d_g = dg, P.n_fft = n, P.W2 = weights + off;
                            const GateGrid gr = gate_grid(P, B, H);
                            const long long twoF = 2 * (n / 2 + 1), M = Hg == 1 ? (long long)B * H : B;
                            const long long covered = 256LL * gr.gx * gr.rounds + (gr.tail ? 2 : 0), spare = covered - twoF;
                            const bool fast = dg == 64 && off == 0;
                            ++cases;
                            if (gr.gy != Hg || gr.gx < 1 || gr.rounds < 1) ++fails;
                            if (spare < 0 || spare >= 256LL * gr.rounds + 64) ++fails;
                            if (gr.tail && (M > 4 || !fast || (twoF - 2) % 64 || twoF <= 64)) ++fails;
                            const GateGrid own = gate_grid_of((int)(twoF + 63) / 64, gr.gy, false);
                            if (gr.tail && gr.rounds >= own.rounds && gr.per_unit() >= own.per_unit()) ++fails;
                            rides += gr.tail;
                            for (int chunks : {1, 2, 9, 16, 32, 36, 64, 128, 256, 512, 2048}) {
                                if (!gate_prep_inside(P, B, H, chunks)) continue;
                                const long long wgs = gr.workgroups(), last = chunks % 32;
                                if (M > 4 || !fast || wgs > 1024 || (long long)B * H >= 2048) ++fails;
                                if (chunks > 1 && (wgs * M * chunks * 512 > 32 << 20 || M * (chunks / 32 + (last + 3) / 4) > 8)) ++fails;
                                ++inside;
                            }
                        }
    if (rides == 0 || inside == 0) ++fails;
    printf("gate launches: %d cases, %d with riding rows, %d with the hidden layer inside, %d failures\n", cases, rides, inside, fails);
    return fails != 0;
}
