// Gate kernels: host-side launch declarations and the rules of the output layer's launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace spectre {

constexpr int kPoolRows = 256;   // rows summed by one workgroup of the pooling pass

struct GateDev {                 // device pointers; layout as in the public parameter block
    int Hg, d, d_g, n_fft;
    const float *ln_gamma, *ln_beta;
    float ln_eps;
    const float *W1, *b1, *W2, *b2, *modrelu_bias;
    const float2 *toeplitz;      // [Hg, 2r+1] or nullptr
    int toeplitz_r;
};

// Bytes of the pooling partial sums for query rows [B, L, H, d].
size_t gate_partial_bytes(int B, int L, int H, int d);

// sum_q [B,H,d] (double) = sum over the L rows of q [B,L,H,d]; io 0 = fp32, 1 = bf16.
hipError_t launch_pool(int io, const void *q, double *partial, double *sum_q, int B, int L, int H, int d,
                       hipStream_t st);

// sum [B][row] = sum over chunks of partial [B][nchunks][row], added in a fixed order in fp64.
// sum[b][ch] = (accumulate ? sum[b][ch] : 0) + sum over chunks of partial[b][chunk][ch]
hipError_t launch_pool_final(const double *partial, double *sum, int B, int row, int nchunks, hipStream_t st,
                             bool accumulate = false);

// The two halves of launch_pool: partial [B][pool_chunks][H*d]; pool_rows is the least number of rows a chunk stands for.
int pool_rows(int B, int L, int H, int d);
int pool_chunks(int io, int B, int L, int H, int d);
hipError_t launch_pool_partial(int io, const void *q, double *partial, int B, int L, int H, int d, hipStream_t st);

// hid [B,H,d_g] from partial sums [B][nchunks][H*d] of the query rows, or (Wq != nullptr, d = 64) of the rows X that
// W_q [Hw,64,64] turns into queries; sum_q, if not nullptr, receives the pooled query [B,H,d].
hipError_t launch_gate_prep(const double *partial, int nchunks, const float *Wq, int Hw, double *sum_q, double inv_count,
                            const GateDev &P, float *hid, int B, int H, hipStream_t st);
// g from hid: output layer, modReLU, Toeplitz update, phase.
hipError_t launch_gate_out(const float *hid, const GateDev &P, float2 *raw, int B, int H, long long phase, float2 *g,
                           hipStream_t st);
// The whole gate from query rows q [B,L,H,d]; scratch partial (gate_partial_bytes), hid, raw as above.
hipError_t launch_gate(int io, const void *q, double *partial, double inv_count, const GateDev &P, float *hid, float2 *raw,
                       int B, int L, int H, long long phase, float2 *g, hipStream_t st);

// g [B,H,F] from sum_q; hid is scratch [B,H,d_g]; raw is scratch [B,H,F] complex, only used when
// P.toeplitz is set; phase already reduced modulo n_fft.
hipError_t launch_gate_mlp(const double *sum_q, double inv_count, const GateDev &P, float *hid, float2 *raw,
                           int B, int H, long long phase, float2 *g, hipStream_t st);

// Grid of the output layer: workgroups per weight set, tiles per wave.
struct GateGrid {
    int gx, gy, rounds;
    bool tail;                       // the two rows behind the last whole tile ride with the last workgroup
    long long workgroups() const { return (long long)gx * gy; }
    long long per_unit() const { return (workgroups() + 255) / 256; }   // workgroups of the compute unit that has most
};
inline GateGrid gate_grid_of(int ntiles, int gy, bool tail) {
    int gx = (4096 + gy - 1) / gy;                 // about 16 workgroups per compute unit in total (1024: 5 % slower)
    if (gx > (ntiles + 3) / 4) gx = (ntiles + 3) / 4;
    // shrink the grid to the smallest one with the same number of tiles per wave (no ragged last round)
    const int rounds = (ntiles + 4 * gx - 1) / (4 * gx);
    return {(ntiles + 4 * rounds - 1) / (4 * rounds), gy, rounds, tail};
}
// k_gate_out reads W2 in 16-byte pieces
inline bool gate_vec(const GateDev &P) { return P.d_g % 4 == 0 && (reinterpret_cast<uintptr_t>(P.W2) & 15) == 0; }
inline GateGrid gate_grid(const GateDev &P, int B, int H) {
    const int twoF = 2 * (P.n_fft / 2 + 1), gy = P.Hg == 1 ? 1 : H, M = P.Hg == 1 ? B * H : B;
    const GateGrid own = gate_grid_of((twoF + 63) / 64, gy, false);
    // Lengths that are a multiple of 64 have two rows more than whole tiles.  A tile of their own can cost every wave another tile, or,
    // while all workgroups run at once, some compute units a workgroup more than the others have (32 heads of n = 8192: 1056 for 1024
    // places).  Only there do they ride, and only for up to four rows per weight set, which that workgroup takes side by side.  us, own tile /
    // riding: gate of bf16 rows, 32 heads of 131072 271.2 / 267.9, 65536 144.1 / 141.7, 4 x 16 heads of 8192 30.0 / 27.5; layer of 32 heads
    // of 8192 92.9 / 91.7, 4096 55.9 / 55.2; but 512 24.5 / 25.5, and where there are several rounds of workgroups, 24576 248.6 / 250.6.
    // More rows one after the other would stand behind the last tile (from pooled sums: 16 rows over one set n = 20480 12.3 / 14.5, over
    // 32 sets 52.2 / 56.9; 250 over one 27.9 / 31.4).
    if (M > 4 || !gate_vec(P) || P.d_g != 64 || twoF % 64 != 2 || twoF <= 64) return own;
    const GateGrid ride = gate_grid_of(twoF / 64, gy, true);
    return ride.rounds < own.rounds || (ride.workgroups() <= 1024 && ride.per_unit() < own.per_unit()) ? ride : own;
}

// The hidden layer inside every workgroup of the output layer, whose weights are under way meanwhile: one dependent launch less (about
// 2 us), for up to four rows per weight set and while all workgroups run at once, four to a compute unit.  Each forms the layer again:
//  - further rounds of workgroups would pay for it again (32 heads of 131072 bf16 rows, step of gate and mixer, 1236 -> 1262 us);
//  - a wave adds its share of a row's chunk sums eight at a time, what is left over one at a time and the rows one after the other, each
//    trip a round trip to the L2.  us, separate minus inside, over 3 to 14 shapes each: 2 to 4 trips 2 to 3, 6 trips 1, 8 trips 0 to 1, 12
//    trips -1.8, 16 trips -2 to -3, 32 trips -8, 64 trips -24;
//  - the workgroups' reads of the sums add up (one row, 128 chunks of 512 bytes, 512 workgroups +1, 768 -0.9; 256 chunks, 256 workgroups
//    +1, 1024 -3.9), and so does the layer's arithmetic (32 chunks: 2, 3 and 4 rows in 1024 workgroups -0.5, -2 and -2.5, 4 rows in 512 0).
// Pooled sums, which need neither, while the workgroups run at once (gate with a position, B = 4 H = 32 n = 8192 17.9 / 16.2).
// From 2048 heads on the separate launch adds the layer's terms in another order (launch_gate_prep).
inline bool gate_prep_inside(const GateDev &P, int B, int H, int nchunks) {
    const int M = P.Hg == 1 ? B * H : B;
    if (P.d != 64 || P.d_g != 64 || M > 4 || B * H >= 2048 || !gate_vec(P)) return false;
    const long long workgroups = gate_grid(P, B, H).workgroups();
    if (nchunks == 1) return workgroups <= 1024;
    const int trips = M * (nchunks / 32 + (nchunks % 32 + 3) / 4);
    return trips <= 8 && workgroups * M <= 1024 && workgroups * M * nchunks <= 65536;
}

}  // namespace spectre
