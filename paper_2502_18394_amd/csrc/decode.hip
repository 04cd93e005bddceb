// One decode step of the Prefix-FFT cache in two launches (Algorithm 1, DecodeStep) for gfx950.
//
//   k_decode       : everything that only reads the ring state - the running query sum with the new token in and the
//                    evicted one out, LayerNorm, the MLP, modReLU - and the pass over the half spectra (Eq. 5's update
//                    and / or the newest row's readout) with the gate entries of its own bins, which never leave LDS;
//   k_decode_final : adds the chunks' readout sums in a fixed order, writes the output row, and only then brings the
//                    ring buffers and sum_q up to date (every workgroup of k_decode reads their old contents).
//
// What bounds it: the streams of W2 (the gate's output weights) and of the half spectra.  A workgroup owns 128 bins of
// one head, i.e. 64 KB of each stream per sequence, and everything in front of them (64 x 64 first layer, LayerNorm) is
// recomputed by every workgroup from L2: cheaper than the three dependent launches (ring update, hidden layer, output
// layer) and the round trip of the gate through memory that it replaces.
// A chip's workgroups of one round run in step, so what a workgroup waits for outside its two streams is time without
// traffic.  Loads return in order: the first layer's operands are requested before the weights, whose arrival its chain then
// passes behind, and the first rows of the half spectra as soon as the weights' registers are free, ahead of the factors; in
// steps that only read them a row's registers take the one after next when it is used.  Steps that write the rows back do so only where one
// workgroup has a block of weights to itself (B <= 2) or the launch is so small that each takes one sequence (B=2 H=4 N=8192, 14 tokens 191 / 194);
// elsewhere several take turns at one, and the next eight are requested together behind the last
// store (us of two tokens, one by one / together: B=1 H=32 N=32768 277 / 280, B=2 H=20 N=16384 154 / 156; B=3 H=20 N=32768 421 / 413, B=8 H=32
// N=4096 212 / 208).  us, before / now: B=1 H=32, a deferred token, N=4096 18.6 / 16.8, 8192 27.5 / 27.0, 12288 40.8 / 39.0; two that
// update, 4096 48.0 / 44.5, 16384 147 / 144.  (Plain loads, so that both streams stay
// in the memory-side cache from token to token, gain another 2 to 15 % below 268 MB when nothing else runs between, and lose 6 to
// 17 % when the caches and weights of eight layers take turns.)
// Measured against ring update + hidden + output layer + sweep + final: B=1 H=32 N=8192, deferred updates, 39.7 ->
// 30.5 us a token over 16 of them (a reading step moves 134 MB in 24 us, 5.6 TB/s); B=8 H=32 N=32768, every step
// updating, 838 -> 812 us (4.56 GB, 5.6 TB/s).
#include "prefix.h"

#include "common.h"
#include "fold16.h"
#include "gate.h"
#include "prefix_dev.h"

namespace spectre {

struct DecodeRing {                    // the ring state as it was before this token, and the token itself
    const void *v_t, *q_t;             // [B, 1, H, 64]
    float *v_buf, *q_buf;              // [B*H, N, 64]
    double *sum_q;                     // [B*H, 64]
    int slot, evict;
};

// Bins per workgroup.  A window length is a multiple of 256, so its N / 2 bins below Nyquist are whole chunks; the
// Nyquist bin rides with the last one (a chunk of its own was a second round of workgroups at N = 8192: 1056 of them
// for 1024 places).
constexpr int kBins = 128, kBinStride = kBins + 2;
static int decode_chunks(int N) { return N / (2 * kBins); }

// one bin of the output layer to the factors of the pass: u = raw gate without its bias
template <bool LAZY>
__device__ __forceinline__ void decode_factors(float2 *r, float2 *g, float2 bias, bool act, float mb, float ck, float2 w) {
    const float2 u = *r;
    float re = u.x + bias.x, im = u.y + bias.y;
    if (act) {                                                       // modReLU (Sec. 3.2 step 3c)
        const float mag = sqrtf(re * re + im * im);
        const float sc = (mag > 0.0f) ? fmaxf(mag + mb, 0.0f) / mag : 0.0f;
        re *= sc;
        im *= sc;
    }
    const float2 gc = make_float2(re * ck, im * ck);
    if (LAZY) *g = gc;
    *r = cmulc(gc, w);
}

// one entry (bin, two channels) of the pass
template <bool LAZY>
__device__ __forceinline__ void decode_entry(float4 &x, float2 dl, float2 wk, float2 r, float &acc0, float &acc1) {
    if (!LAZY) {
        x.x = fmaf(dl.x, wk.x, x.x);
        x.y = fmaf(dl.x, wk.y, x.y);
        x.z = fmaf(dl.y, wk.x, x.z);
        x.w = fmaf(dl.y, wk.y, x.w);
    }
    acc0 = fmaf(r.x, x.x, fmaf(-r.y, x.y, acc0));
    acc1 = fmaf(r.x, x.z, fmaf(-r.y, x.w, acc1));
}

// 1-D grid over (chunk, head, group of bpw sequences), see below; 256 lanes.
// LAZY = false: X += Delta w_k, stored, and the readout sums of the updated entries (k_sweep<true, true>).
// LAZY = true : X only read, plus the pending tokens' kappa sums (k_sweep_lazy); ps includes this token.
// AT_ONCE: a row's registers take the next row when it is used, see above.
template <typename T, bool LAZY, bool AT_ONCE>
__global__ __launch_bounds__(256, 4) void k_decode(float4 *__restrict__ X, DecodeRing rg, double inv_count, GateDev P,
                                                const float2 *__restrict__ tw, float *__restrict__ partial,
                                                float *__restrict__ kpart, int B, int H, int N, int bpw,
                                                PendingSlots ps, int nchunks) {
    extern __shared__ float lds_dec[];
    float2 *s_w = reinterpret_cast<float2 *>(lds_dec);               // [bins]      w_k
    float2 *s_r = s_w + kBinStride;                                  // [bpw][bins] u, then c_k/N g_k conj(w_k)
    float *s_qb = reinterpret_cast<float *>(s_r + bpw * kBinStride); // [bpw][64]
    float *s_hid = s_qb + bpw * 64;                                  // [bpw][64]
    float *s_part = s_hid + bpw * 64;                                // [bpw][4][64] first layer, then readout sums
    float2 *s_g = reinterpret_cast<float2 *>(s_part + bpw * 256);    // [bpw][bins] LAZY: c_k/N g_k
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, F = N / 2 + 1;
    // the workgroups that share a (chunk, head), and with it a block of W2, get ids 8 apart: they run at the same time
    // on one XCD, and its L2 serves the block to all but the first
    const int nz = (B + bpw - 1) / bpw, idx8 = blockIdx.x >> 3;
    const int unit = (idx8 / nz) * 8 + (blockIdx.x & 7);
    if (unit >= nchunks * H) return;                                 // whole workgroup: units are padded to 8
    const int h = unit / nchunks, chunk = unit - h * nchunks, hp = (P.Hg == 1) ? 0 : h;
    const int b0 = (idx8 % nz) * bpw, nb = min(bpw, B - b0);
    const int k0 = chunk * kBins;
    const bool last = chunk == nchunks - 1;                          // has the Nyquist bin as its bin kBins

    // loads return in the order they are issued: what the first layer needs goes in front of the weights
    const int kl = tid & (kBins - 1), k = k0 + kl;
    const float2 w = tw[mul_mod((unsigned)k, (unsigned)rg.slot, N)];
    float w1[16];                                                    // first layer: 16 of the 64 inputs per wave
#pragma unroll
    for (int i = 0; i < 16; ++i) w1[i] = P.W1[(size_t)hp * 4096 + (16 * wave + i) * 64 + lane];
    const float b1 = P.b1[hp * 64 + lane];
    const bool act = P.modrelu_bias != nullptr;
    const float2 bias = *reinterpret_cast<const float2 *>(P.b2 + ((size_t)hp * F + k) * 2);
    const float mb = act ? P.modrelu_bias[(size_t)hp * F + k] : 0.0f;
    float2 w_ny = make_float2(0.f, 0.f), bias_ny = w_ny;
    float mb_ny = 0.f;
    if (last) {
        w_ny = tw[mul_mod((unsigned)N / 2, (unsigned)rg.slot, N)];
        bias_ny = *reinterpret_cast<const float2 *>(P.b2 + ((size_t)hp * F + N / 2) * 2);
        if (act) mb_ny = P.modrelu_bias[(size_t)hp * F + N / 2];
    }
    float qn = 0.f, qo = 0.f, gam = 0.f, bet = 0.f;
    double sq = 0.0;
    if (wave < nb) {                                                 // bpw <= 4: one sequence per wave, lane = channel
        const int bh = (b0 + wave) * H + h;
        const size_t i = (size_t)bh * 64 + lane;
        qn = load_scalar<T>(static_cast<const T *>(rg.q_t), i);
        qo = rg.q_buf[((size_t)bh * N + rg.slot) * 64 + lane];
        sq = rg.sum_q[i];
        gam = P.ln_gamma[hp * 64 + lane];
        bet = P.ln_beta[hp * 64 + lane];
    }
    __builtin_amdgcn_sched_barrier(0);

    // this wave's 64 rows of W2 (whole rows of 64 weights, 1 KB per instruction), in flight during the first layer
    const float *w2h = P.W2 + (size_t)hp * 2 * F * 64;
    const float4 *w2 = reinterpret_cast<const float4 *>(w2h + (size_t)(2 * k0 + 64 * wave) * 64) + lane;
    float4 a[16], an;
    if (nz > 1 || P.Hg == 1) {                            // read again by others: keep it in the L2
#pragma unroll
        for (int s = 0; s < 16; ++s) a[s] = w2[64 * s];
    } else {
#pragma unroll
        for (int s = 0; s < 16; ++s) a[s] = stream_load(w2 + 64 * s);
    }
    an = reinterpret_cast<const float4 *>(w2h + (size_t)(last ? N : 2 * k0) * 64)[tid & 31];   // the Nyquist bin's two rows
    if (tid < kBins) s_w[kl] = w;
    if (last && tid == kBins) s_w[kBins] = w_ny;

    // LayerNorm of the descriptor
    if (wave < nb) {
        const double x = inv_count * (sq + ((double)qn - (rg.evict ? (double)qo : 0.0)));
        const double dev = x - wave_sum(x) / 64;
        const double rstd = 1.0 / sqrt(wave_sum(dev * dev) / 64 + (double)P.ln_eps);
        s_qb[wave * 64 + lane] = (float)((double)gam * dev * rstd + (double)bet);
    }
    __syncthreads();
    for (int bl = 0; bl < nb; ++bl) {
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc = fmaf(s_qb[bl * 64 + 16 * wave + i], w1[i], acc);
        s_part[(bl * 4 + wave) * 64 + lane] = acc;
    }
    __syncthreads();
    for (int idx = tid; idx < nb * 64; idx += 256) {
        const int bl = idx >> 6, j = idx & 63;
        const float *pp = s_part + bl * 256 + j;
        const float t = b1 + ((pp[0] + pp[64]) + (pp[128] + pp[192]));
        s_hid[idx] = 0.5f * t * (1.0f + erff(t * 0.70710678118654752440f));
    }
    __syncthreads();
    // output layer: a lane's four weights of row 4 s + lane / 16 against the hidden values, summed over 16 lanes
    for (int bl = 0; bl < nb; ++bl) {
        const float4 hv = *reinterpret_cast<const float4 *>(s_hid + bl * 64 + 4 * (lane & 15));
        float *u = reinterpret_cast<float *>(s_r + bl * kBinStride);
        float p[16];
#pragma unroll
        for (int s = 0; s < 16; ++s) p[s] = fmaf(a[s].x, hv.x, fmaf(a[s].y, hv.y, fmaf(a[s].z, hv.z, a[s].w * hv.w)));
        fold16<8>(p, lane);
        fold16<4>(p, lane);
        fold16<2>(p, lane);
        fold16<1>(p, lane);
        u[64 * wave + 4 * (lane & 15) + (lane >> 4)] = p[0];
        if (last && wave == 0) {
            float q = fmaf(an.x, hv.x, fmaf(an.y, hv.y, fmaf(an.z, hv.z, an.w * hv.w)));
            q += partner16<8>(q);
            q += partner16<4>(q);
            q += partner16<2>(q);
            q += partner16<1>(q);
            if (lane == 0 || lane == 16) u[2 * kBins + (lane >> 4)] = q;
        }
    }
    // the pass over the half spectra: 8 bins x 32 lanes, two channels per lane, eight rows of a lane at a time; the weights'
    // registers are free now, and the first rows are under way while the factors are formed
    const int cl = tid & 31, row = tid >> 5;
    constexpr int kU = 8, kHalf = 8 * kU;
    struct Sequence {                                                // what the pass needs besides the rows
        float2 dl, e, rot;
    };
    auto head_of = [&](int bl) { return X + ((size_t)((b0 + bl) * H + h) * F + k0) * 32 + cl; };
    unsigned mult = 0, m_item = 0, step_item = 0;
    if (LAZY) {                                                      // see k_sweep_lazy
        mult = (cl < ps.n) ? (unsigned)((rg.slot - ps.slot[cl] + N) % N) : 0u;
        index_walk((unsigned)(k0 + row), mult, N, m_item, step_item);
    }
    auto load_sequence = [&](int bl) {
        Sequence q = {make_float2(0.f, 0.f), make_float2(1.f, 0.f), make_float2(1.f, 0.f)};
        if (LAZY) {
            q.rot = tw[step_item];
            q.e = tw[m_item];
        } else {
            const size_t i = (size_t)((b0 + bl) * H + h) * 64 + 2 * cl;
            const T *vp = static_cast<const T *>(rg.v_t);
            q.dl = make_float2(load_scalar<T>(vp, i), load_scalar<T>(vp, i + 1));
            const float2 old = *reinterpret_cast<const float2 *>(rg.v_buf + ((size_t)((b0 + bl) * H + h) * N + rg.slot) * 64 + 2 * cl);
            q.dl.x -= rg.evict ? old.x : 0.f;
            q.dl.y -= rg.evict ? old.y : 0.f;
        }
        return q;
    };
    auto load_row = [&](int bl, int kc) { return stream_load(head_of(bl) + (size_t)kc * 32); };
    Sequence sn = load_sequence(0);
    float4 x[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) x[u] = load_row(0, row + 8 * u);
    __syncthreads();
    {
        const float invN = 1.0f / (float)N;
        for (int bl = tid >> 7; bl < nb; bl += 2)
            decode_factors<LAZY>(s_r + bl * kBinStride + kl, s_g + bl * kBinStride + kl, bias, act, mb,
                                 k == 0 ? invN : 2.0f * invN, w);
        if (last && tid < nb) {
            const int i = tid * kBinStride + kBins;
            decode_factors<LAZY>(s_r + i, s_g + i, bias_ny, act, mb_ny, invN, w_ny);
        }
    }
    __syncthreads();

#pragma unroll 1
    for (int bl = 0; bl < nb; ++bl) {
        const Sequence sq_now = sn;
        float2 e = sq_now.e;
        float acc0 = 0.f, acc1 = 0.f, kacc = 0.f;
        float4 *Xp = head_of(bl);
        const float2 *rp = s_r + bl * kBinStride, *gp = s_g + bl * kBinStride;
        // a row's registers take the one after next (half a chunk on, then the next sequence's): at once, or all eight behind the last store
#pragma unroll 1
        for (int half = 0; half < 2; ++half) {
            const int next_bl = half ? bl + 1 : bl, next_k = half ? row : kHalf + row;
            if (half && next_bl < nb) sn = load_sequence(next_bl);
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int kc = kHalf * half + row + 8 * u;
                decode_entry<LAZY>(x[u], sq_now.dl, LAZY ? make_float2(0.f, 0.f) : s_w[kc], rp[kc], acc0, acc1);
                if (!LAZY) stream_store(Xp + (size_t)kc * 32, x[u]);
                if (LAZY) {
                    const float2 gc = gp[kc];
                    kacc = fmaf(gc.x, e.x, fmaf(gc.y, e.y, kacc));   // c_k/N Re(g_k conj(e_k))
                    e = cmul(e, sq_now.rot);
                }
                if (AT_ONCE && next_bl < nb) x[u] = load_row(next_bl, next_k + 8 * u);
            }
            if (!AT_ONCE && next_bl < nb) {
#pragma unroll
                for (int u = 0; u < kU; ++u) x[u] = load_row(next_bl, next_k + 8 * u);
            }
        }
        if (last && row == 0) {                                      // Nyquist
            float4 xn = stream_load(Xp + kBins * 32);
            decode_entry<LAZY>(xn, sq_now.dl, s_w[kBins], rp[kBins], acc0, acc1);
            if (!LAZY) stream_store(Xp + kBins * 32, xn);
            if (LAZY) {
                const float2 en = tw[mul_mod((unsigned)N / 2, mult, N)];
                kacc = fmaf(gp[kBins].x, en.x, fmaf(gp[kBins].y, en.y, kacc));
            }
        }
        acc0 += __shfl_xor(acc0, 32);
        acc1 += __shfl_xor(acc1, 32);
        float2 *red = reinterpret_cast<float2 *>(s_part + bl * 256);
        if (lane < 32) red[wave * 32 + cl] = make_float2(acc0, acc1);
        if (LAZY) {
            kacc += __shfl_xor(kacc, 32);
            if (lane < 32) s_qb[bl * 128 + wave * 32 + cl] = (cl < ps.n) ? kacc : 0.f;   // s_qb and s_hid are free now
        }
    }
    __syncthreads();
    for (int idx = tid; idx < nb * 32; idx += 256) {
        const int bl = idx >> 5, c = idx & 31;
        const size_t at = (size_t)((b0 + bl) * H + h) * nchunks + chunk;
        const float2 *red = reinterpret_cast<const float2 *>(s_part + bl * 256) + c;
        float2 s = red[0];
#pragma unroll
        for (int q = 1; q < 4; ++q) s = s + red[32 * q];
        *reinterpret_cast<float2 *>(partial + at * 64 + 2 * c) = s;
        if (LAZY) {
            const float *kr = s_qb + bl * 128 + c;
            kpart[at * 32 + c] = (kr[0] + kr[32]) + (kr[64] + kr[96]);
        }
    }
}

// grid B*H; 256 lanes = 32 channel pairs x 8 chunk groups.  out[b, 0, h, c] = sum over chunks of partial (LAZY: plus
// sum_i kappa_i Delta_i[c], this token being pending token npend - 1, whose Delta row it also writes), then the ring
// buffers and the running query sum take the token in.
template <typename IO, typename T, bool LAZY>
__global__ __launch_bounds__(256) void k_decode_final(const float *__restrict__ partial, const float *__restrict__ kpart,
                                                      float *__restrict__ pending, DecodeRing rg,
                                                      typename IO::pair_t *__restrict__ out, int nchunks, int N, int BH,
                                                      int npend) {
    __shared__ float2 red[8][32];
    __shared__ float kred[8][32];
    const int p = threadIdx.x & 31, grp = threadIdx.x >> 5, bh = blockIdx.x;
    float2 dnew = make_float2(0.f, 0.f);
    if (grp == 0) {                                                  // lanes 0..31: two channels each
        const size_t i = (size_t)bh * 64 + 2 * p, ring = ((size_t)bh * N + rg.slot) * 64 + 2 * p;
        const T *vp = static_cast<const T *>(rg.v_t), *qp = static_cast<const T *>(rg.q_t);
        const float2 vn = make_float2(load_scalar<T>(vp, i), load_scalar<T>(vp, i + 1));
        const float2 qn = make_float2(load_scalar<T>(qp, i), load_scalar<T>(qp, i + 1));
        float2 vo = make_float2(0.f, 0.f), qo = vo;
        if (rg.evict) {
            vo = *reinterpret_cast<const float2 *>(rg.v_buf + ring);
            qo = *reinterpret_cast<const float2 *>(rg.q_buf + ring);
        }
        dnew = make_float2(vn.x - vo.x, vn.y - vo.y);
        double2 s = *reinterpret_cast<const double2 *>(rg.sum_q + i);
        s.x += (double)qn.x - (double)qo.x;
        s.y += (double)qn.y - (double)qo.y;
        *reinterpret_cast<double2 *>(rg.sum_q + i) = s;
        *reinterpret_cast<float2 *>(rg.v_buf + ring) = vn;
        *reinterpret_cast<float2 *>(rg.q_buf + ring) = qn;
        if (LAZY) *reinterpret_cast<float2 *>(pending + ((size_t)(npend - 1) * BH + bh) * 64 + 2 * p) = dnew;
    }
    // pending tokens grp, grp + 8, ... of the earlier ones: their Delta rows are under way with the chunks' sums
    constexpr int kPer = kMaxPending / 8;
    float2 dlt[LAZY ? kPer : 1];
    if (LAZY) {
#pragma unroll
        for (int m = 0; m < kPer; ++m) {
            const int i = grp + 8 * m;
            dlt[m] = i + 1 < npend ? *reinterpret_cast<const float2 *>(pending + ((size_t)i * BH + bh) * 64 + 2 * p)
                                   : make_float2(0.f, 0.f);
        }
    }
    const float2 *src = reinterpret_cast<const float2 *>(partial + (size_t)bh * nchunks * 64) + p;
    const float *ksrc = LAZY ? kpart + (size_t)bh * nchunks * 32 + p : nullptr;
    float2 s = make_float2(0.f, 0.f);
    float ks = 0.f;
    for (int c = grp; c < nchunks; c += 64) {    // eight loads of each kind in flight, added in chunk order
        float2 v[8];
        float kv[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            v[i] = make_float2(0.f, 0.f);
            kv[i] = 0.f;
            if (c + 8 * i < nchunks) {
                v[i] = src[(size_t)(c + 8 * i) * 32];
                if (LAZY) kv[i] = ksrc[(size_t)(c + 8 * i) * 32];
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            s = s + v[i];
            if (LAZY) ks += kv[i];
        }
    }
    if (LAZY) {
        kred[grp][p] = ks;
        __syncthreads();
        auto kappa = [&](int i) {
            float k = kred[0][i];
#pragma unroll
            for (int r = 1; r < 8; ++r) k += kred[r][i];
            return k;
        };
#pragma unroll
        for (int m = 0; m < kPer; ++m) {
            if (grp + 8 * m + 1 < npend) {
                const float k = kappa(grp + 8 * m);
                s.x = fmaf(k, dlt[m].x, s.x);
                s.y = fmaf(k, dlt[m].y, s.y);
            }
        }
        if (grp == 0) {                          // this token
            const float k = kappa(npend - 1);
            s.x = fmaf(k, dnew.x, s.x);
            s.y = fmaf(k, dnew.y, s.y);
        }
    }
    red[grp][p] = s;
    __syncthreads();
    if (grp == 0) {
        float2 t = red[0][p];
#pragma unroll
        for (int r = 1; r < 8; ++r) t = t + red[r][p];
        out[(size_t)bh * 32 + p] = IO::pack(t);
    }
}

// The fused kernel holds the hidden layer of width 64 and needs whole 16-byte rows of W2; the Toeplitz update couples
// neighbouring bins across workgroups.  Anything else takes the gate kernels and a sweep.
bool decode_fused_supported(const GateDev &P) {
    return P.d == 64 && P.d_g == 64 && !P.toeplitz && (reinterpret_cast<uintptr_t>(P.W2) & 15) == 0 &&
           (reinterpret_cast<uintptr_t>(P.b2) & 7) == 0;
}

template <typename IO, typename T>
static hipError_t decode_t(const DecodeRing &rg, float2 *X, double inv_count, const GateDev &P, const float2 *tw,
                           float *partial, float *kpart, float *pending, void *out, int B, int H, int N,
                           const PendingSlots &ps, hipStream_t st) {
    const int nch = decode_chunks(N);
    const bool lazy = ps.n > 0;
    // Sequences per workgroup.  Several share one block of W2 and one set-up, but long workgroups end raggedly: at B=8
    // H=32 N=32768 an updating step takes 839 / 812 / 818 us with 1 / 2 / 4, a reading one at B=4 N=8192 68 / 61 / 58 us.
    // Fewer while the launch would leave compute units without a fourth workgroup.
    int bpw = lazy ? 4 : 2;
    if (bpw > B) bpw = B;
    while (bpw > 1 && (long long)nch * H * ((B + bpw - 1) / bpw) < 1024) bpw = (bpw + 1) / 2;
    // the same number of workgroups with even shares: five sequences as 3 + 2, not 4 + 1
    bpw = (B + (B + bpw - 1) / bpw - 1) / ((B + bpw - 1) / bpw);
    const long long wgs = ((long long)nch * H + 7) / 8 * 8 * ((B + bpw - 1) / bpw);
    if (wgs > 0x7fffffffLL) return hipErrorInvalidValue;
    const size_t lds = kBinStride * sizeof(float2) +
                       (size_t)bpw * (kBinStride * sizeof(float2) * (lazy ? 2 : 1) + (64 + 64 + 256) * sizeof(float));
    const dim3 grid((unsigned)wgs);
    float4 *X4 = reinterpret_cast<float4 *>(X);
    const auto kern = lazy ? k_decode<T, true, true> : bpw == 1 || bpw == B ? k_decode<T, false, true> : k_decode<T, false, false>;
    kern<<<grid, 256, lds, st>>>(X4, rg, inv_count, P, tw, partial, kpart, B, H, N, bpw, ps, nch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    typename IO::pair_t *o = static_cast<typename IO::pair_t *>(out);
    if (lazy) k_decode_final<IO, T, true><<<B * H, 256, 0, st>>>(partial, kpart, pending, rg, o, nch, N, B * H, ps.n);
    else k_decode_final<IO, T, false><<<B * H, 256, 0, st>>>(partial, nullptr, nullptr, rg, o, nch, N, B * H, 0);
    return hipGetLastError();
}

hipError_t launch_decode(int io, const void *v_t, const void *q_t, float *v_buf, float *q_buf, double *sum_q, int slot,
                         int evict, float2 *X, double inv_count, const GateDev &P, const float2 *tw, float *partial,
                         float *kpart, float *pending, int npend, const int *slots, void *out, int B, int H, int N,
                         hipStream_t st) {
    if (npend < 0 || npend > kMaxPending) return hipErrorInvalidValue;
    PendingSlots ps;
    ps.n = npend;
    for (int i = 0; i < kMaxBatch; ++i) ps.slot[i] = i < npend ? slots[i] : 0;
    const DecodeRing rg = {v_t, q_t, v_buf, q_buf, sum_q, slot, evict};
    return io ? decode_t<IoBf16, uint16_t>(rg, X, inv_count, P, tw, partial, kpart, pending, out, B, H, N, ps, st)
              : decode_t<IoF32, float>(rg, X, inv_count, P, tw, partial, kpart, pending, out, B, H, N, ps, st);
}

// Loads this translation unit's code object (the runtime loads them on first use): called by spectre_prepare so
// that no compute call is the first to touch it.
hipError_t load_kernels_decode() {
    hipFuncAttributes a;
    return hipFuncGetAttributes(&a, reinterpret_cast<const void *>((k_decode<float, false, false>)));
}

}  // namespace spectre
