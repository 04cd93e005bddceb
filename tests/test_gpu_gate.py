"""GPU parity of spectre_gate against the fp64 oracle (Sec. 3.2 step 3; Sec. 3.5 phase)."""
import numpy as np
import pytest
import torch

from gpu_util import TOL, f64, rel_l2, to_device
from paper_2502_18394_amd import synth

pytestmark = pytest.mark.gpu


def run_gate(oracle, B, L, H, d, dg, n, io, shared=False, modrelu=True, phase=0, seed=1, std=0.02, bias_shift=0.0):
    from paper_2502_18394_amd import binding
    p = synth.gate_params(seed, 1 if shared else H, d, n, d_g=dg, modrelu=modrelu, std=std)
    if bias_shift:
        p["modrelu_bias"] = (p["modrelu_bias"] + np.float32(bias_shift)).astype(np.float32)
    vals, store = synth.tokens(seed + 1, (B, L, H, d), io)
    P = binding.GateParams(p)
    g = binding.gate(to_device(store, io), P, 1.0 / L, phase_pos=phase)
    torch.cuda.synchronize()
    want = oracle.gate(oracle.pool_q(vals.astype(np.float64)), 1.0 / L, f64(p), n, phase)
    return g.cpu().numpy(), want


@pytest.mark.parametrize("B,L,H,d,dg,io,shared", [
    (1, 1024, 1, 64, 64, "f32", False),      # config 1
    (1, 8192, 32, 64, 64, "bf16", False),    # config 2 shape
    (3, 512, 5, 64, 64, "f32", True),        # shared weights, 15 rows on the MFMA column side
    (40, 256, 1, 64, 64, "f32", False),      # more than 32 rows: two row tiles
    (5, 256, 12, 64, 64, "bf16", True),      # shared, 60 rows
    (4, 196, 12, 64, 64, "f32", False),      # ViT length: 2F = 198, ragged last tile
    (2, 300, 3, 32, 48, "f32", False),       # other d, d_g not a multiple of 16, odd chunking
    (1, 7, 2, 8, 5, "f32", False),           # tiny everything, odd n
])
def test_gate_matches_oracle(oracle, B, L, H, d, dg, io, shared):
    print(f"case B={B} L={L} H={H} d={d} dg={dg} io={io} shared={shared}", flush=True)
    got, want = run_gate(oracle, B, L, H, d, dg, L, io, shared=shared)
    err = rel_l2(got, want)
    print(f"  rel_l2={err:.3e}", flush=True)
    assert err <= 1e-5   # the gate is fp32 throughout; bf16 only affects the (exactly represented) inputs


def test_gate_large_std_exercises_modrelu_threshold(oracle):
    got, want = run_gate(oracle, 2, 256, 3, 64, 64, 256, "f32", std=0.5, seed=5, bias_shift=-2.0)
    assert rel_l2(got, want) <= 1e-5
    assert (np.abs(want) == 0).any() and (np.abs(want) > 0).any()
    np.testing.assert_array_equal(np.abs(got) == 0, np.abs(want) == 0)


def test_gate_without_modrelu_and_with_phase(oracle):
    got, want = run_gate(oracle, 2, 512, 2, 64, 64, 512, "f32", modrelu=False, phase=777, seed=9)
    assert rel_l2(got, want) <= 1e-5


def test_gate_from_pooled_sum_decode_form(oracle):
    from paper_2502_18394_amd import binding
    B, H, d, N = 3, 4, 64, 4096
    p = synth.gate_params(11, H, d, N)
    sq = np.random.default_rng(12).standard_normal((B, H, d)) * 40.0
    P = binding.GateParams(p)
    for phase in (0, 4097, 123456789):
        g = binding.gate(torch.from_numpy(sq).cuda(), P, 1.0 / N, pooled=True, phase_pos=phase)
        want = oracle.gate(sq, 1.0 / N, f64(p), N, phase)
        assert rel_l2(g.cpu().numpy(), want) <= 1e-5


@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_pooling_kernels_agree_whatever_the_alignment(io):
    """Rows that start on a 16-byte boundary are pooled with 16-byte loads, others pair by pair; both add the rows of
    a channel in the same order, so the gates must be identical bit for bit."""
    from paper_2502_18394_amd import binding
    B, L, H, d = 2, 1000, 3, 64
    P = binding.GateParams(synth.gate_params(31, H, d, L))
    _, store = synth.tokens(32, (B, L, H, d), io)
    q = to_device(store, io)
    shift = 2                                             # elements: 8 bytes (fp32), 4 bytes (bf16)
    flat = torch.empty(q.numel() + shift, dtype=q.dtype, device="cuda")
    q_off = flat[shift:].view(B, L, H, d)
    q_off.copy_(q)
    assert q.data_ptr() % 16 == 0 and q_off.data_ptr() % 16 != 0
    a = binding.gate(q, P, 1.0 / L)
    b = binding.gate(q_off, P, 1.0 / L)
    torch.cuda.synchronize()
    assert torch.equal(torch.view_as_real(a), torch.view_as_real(b))


def test_pooling_of_long_sequence_is_accurate(oracle):
    """128k rows: the pooled mean is ~0.003 and LayerNorm rescales it to O(1), so the sum must be tight."""
    got, want = run_gate(oracle, 1, 131072, 2, 64, 64, 1024, "bf16", seed=21)
    assert rel_l2(got, want) <= 1e-5


@pytest.mark.parametrize("B,L,H,r,shared,modrelu", [(2, 512, 3, 2, False, True), (1, 196, 4, 8, True, True),
                                                     (3, 1024, 2, 0, False, False), (1, 8192, 32, 4, False, True)])
def test_gate_with_toeplitz_update(oracle, B, L, H, r, shared, modrelu):
    """Sec. 3.2 step 3b between the MLP and modReLU."""
    from paper_2502_18394_amd import binding
    d, dg = 64, 64
    Hg = 1 if shared else H
    p = synth.gate_params(50 + r, Hg, d, L, d_g=dg, modrelu=modrelu, std=0.1)
    p["toeplitz"] = synth.toeplitz_taps(60 + r, Hg, r, std=0.3)
    vals, store = synth.tokens(70 + r, (B, L, H, d), "f32")
    P = binding.GateParams(p)
    g = binding.gate(to_device(store, "f32"), P, 1.0 / L, phase_pos=5 if r == 2 else 0)
    torch.cuda.synchronize()
    p64 = f64(p)
    p64["toeplitz"] = p["toeplitz"].astype(np.complex128)
    want = oracle.gate(oracle.pool_q(vals.astype(np.float64)), 1.0 / L, p64, L, 5 if r == 2 else 0)
    err = rel_l2(g.cpu().numpy(), want)
    print(f"  r={r} rel_l2={err:.3e}", flush=True)
    assert err <= 1e-5
    # and it does something: differs from the gate without taps
    p_plain = {k: v for k, v in p64.items() if k != "toeplitz"}
    plain = oracle.gate(oracle.pool_q(vals.astype(np.float64)), 1.0 / L, p_plain, L, 5 if r == 2 else 0)
    assert rel_l2(want, plain) > 1e-3


def _seeded_gate_cases():
    rng = np.random.default_rng(synth.BASE_SEED + 950)
    cases = []
    for _ in range(14):
        B = int(rng.integers(1, 70))
        H = int(rng.integers(1, 6))
        L = int(rng.integers(1, 700))
        d = 2 * int(rng.integers(1, 129))                     # 2 .. 256, even
        dg = int(rng.integers(1, 257))
        n = int(rng.integers(2, 3000))                        # transform length of the gate (even or odd)
        cases.append((B, L, H, d, dg, n, "bf16" if rng.integers(0, 2) else "f32", bool(rng.integers(0, 2)),
                      bool(rng.integers(0, 2)), int(rng.integers(0, 5000)) if rng.integers(0, 2) else 0))
    return cases


@pytest.mark.parametrize("B,L,H,d,dg,n,io,shared,modrelu,phase", _seeded_gate_cases())
def test_gate_seeded_shapes(oracle, B, L, H, d, dg, n, io, shared, modrelu, phase):
    """Channel counts, hidden widths, row counts and transform lengths drawn at random (seeded): every tiling tail of
    the pooling, hidden and output kernels."""
    print(f"case B={B} L={L} H={H} d={d} dg={dg} n={n} io={io} shared={shared} modrelu={modrelu} phase={phase}", flush=True)
    got, want = run_gate(oracle, B, L, H, d, dg, n, io, shared=shared, modrelu=modrelu, phase=phase, seed=960 + B + L)
    err = rel_l2(got, want)
    print(f"  rel_l2={err:.3e}", flush=True)
    assert err <= 1e-5


@pytest.mark.parametrize("B,L,H,Hg,io,taps,pos", [
    (1, 62, 1, 1, "f32", 0, 0),          # the smallest gate of the one-launch kernel: one tile that is all there is
    (3, 63, 2, 2, "bf16", 0, 5),         # last tile moved back over the one before
    (1, 4095, 2, 2, "bf16", 0, 0), (1, 2048, 3, 1, "bf16", 0, 0),   # the longest rows of that kernel, and past them
    (5, 640, 60, 60, "f32", 0, 0), (4, 1024, 64, 1, "f32", 0, 0),   # many heads: the narrow workgroup
    (3, 201, 90, 90, "bf16", 0, 0), (4, 1024, 64, 1, "bf16", 0, 0), # the same with one part per head, and with two
    (2, 300, 3, 3, "f32", 2, 7),         # Toeplitz update and phase behind it
    (256, 130, 1, 1, "f32", 0, 0),       # one head of many sequences
    (33, 1300, 2, 2, "bf16", 0, 0)])     # weights too long for that kernel: the output layer's tiles, of four rows here
def test_gate_one_launch_and_its_edges(oracle, B, L, H, Hg, io, taps, pos):
    from paper_2502_18394_amd import binding
    print(f"case B={B} L={L} H={H} Hg={Hg} io={io} taps={taps} pos={pos}", flush=True)
    q, qs = synth.tokens(70 + L, (B, L, H, 64), io)
    p = synth.gate_params(71 + L, Hg, 64, L)
    if taps:
        p["toeplitz"] = synth.toeplitz_taps(72, Hg, taps)
    got = binding.gate(to_device(qs, io), binding.GateParams(p), 1.0 / L, phase_pos=pos).cpu().numpy()
    p64 = f64(p)
    if taps:
        p64["toeplitz"] = p["toeplitz"].astype(np.complex128)
    want = oracle.gate(oracle.pool_q(q.astype(np.float64)), 1.0 / L, p64, L, pos)
    assert rel_l2(got, want) <= TOL["f32"]


@pytest.mark.parametrize("B,rows", [(455, 8), (911, 16), (1815, 32)])
def test_gate_output_layer_tiles(oracle, B, rows):
    """Many sequences over shared weights: tiles of 8, 16 and 32 rows, the last one ragged."""
    from paper_2502_18394_amd import binding
    H, n, workgroups = 3, 1300, 6                          # 21 tiles of 64 outputs, four to a workgroup
    per = 32
    while per > 4 and B * H > per // 2 and workgroups * -(-B * H // per) < 1024:    # the launch's rule (csrc/gate.hip)
        per //= 2
    assert per == rows and B * H % per
    print(f"case B={B} rows={rows}", flush=True)
    p = synth.gate_params(81, 1, 64, n)
    sq = np.random.default_rng(82).standard_normal((B, H, 64)) * 40.0
    got = binding.gate(torch.from_numpy(sq).cuda(), binding.GateParams(p), 1.0 / n, pooled=True).cpu().numpy()
    assert rel_l2(got, oracle.gate(sq, 1.0 / n, f64(p), n, 0)) <= 1e-5


@pytest.mark.parametrize("B,H,n,d,dg,Hg", [
    (1024, 2, 196, 64, 64, 2), (1030, 2, 64, 256, 200, 1), (700, 3, 130, 32, 100, 3),   # 2048 heads and more: prep of 256 lanes
    (19, 1, 20480, 64, 64, 1), (19, 2, 16384, 64, 64, 2),      # weights beyond 4 MB a set: tiles of 16 rows, a ragged one
    (250, 1, 20480, 64, 64, 1)])                               # the same, enough workgroups with 32 rows
def test_gate_of_many_heads_and_of_large_weights(oracle, B, H, n, d, dg, Hg):
    from paper_2502_18394_amd import binding
    print(f"case B={B} H={H} n={n} d={d} dg={dg} Hg={Hg}", flush=True)
    p = synth.gate_params(83 + n, Hg, d, n, d_g=dg)
    sq = np.random.default_rng(84).standard_normal((B, H, d)) * 40.0
    got = binding.gate(torch.from_numpy(sq).cuda(), binding.GateParams(p), 1.0 / n, pooled=True).cpu().numpy()
    assert rel_l2(got, oracle.gate(sq, 1.0 / n, f64(p), n, 0)) <= 1e-5


@pytest.mark.parametrize("B,H,Hg,n,dg", [(1, 1, 1, 256, 64), (5, 2, 2, 8192, 64), (12, 3, 3, 2560, 64), (7, 20, 1, 4096, 64),
                                         (2, 32, 32, 65536, 64), (3, 4096, 4096, 2048, 64), (1, 4096, 4096, 4096, 64),
                                         (6, 3, 3, 1792, 37), (33, 1, 1, 768, 100), (1, 2, 2, 21, 64)])
def test_positional_phase_turns_the_gate(B, H, Hg, n, dg):
    """The gate with a position against the gate without one, turned in 64 bits: every number of row groups per tile, one and
    several tiles per wave, and so many (17: 4096 heads of 4096 points) that the phase is a pass of its own; positions below and
    far above n.  The turn is one fp32 complex product with a factor rounded once: 3 * 2^-24 of the bin at most, twice that
    here."""
    from paper_2502_18394_amd import binding
    F, s = n // 2 + 1, 0.02
    gen = torch.Generator(device="cuda").manual_seed(n + H)
    r = lambda *shape: torch.randn(shape, generator=gen, device="cuda") * s
    P = binding.GateParams(dict(n_fft=n, ln_eps=synth.LN_EPS, ln_gamma=1 + r(Hg, 64), ln_beta=r(Hg, 64), W1=r(Hg, 64, dg),
                                b1=r(Hg, dg), W2=r(Hg, dg, 2 * F), b2=r(Hg, 2 * F), modrelu_bias=r(Hg, F)))
    q = 30 * torch.randn((B, H, 64), generator=gen, device="cuda", dtype=torch.float64)
    plain = binding.gate(q, P, 1.0 / n, pooled=True).to(torch.complex128)
    for p in (1, n // 2 + 1, n, 10**12 + 7):
        print(f"case B={B} H={H} Hg={Hg} n={n} dg={dg} p={p}", flush=True)
        g = binding.gate(q, P, 1.0 / n, pooled=True, phase_pos=p).to(torch.complex128)
        angle = (torch.arange(F, device="cuda") * (p % n) % n).double() * (2 * np.pi / n)
        err = (g - plain * torch.polar(torch.ones_like(angle), angle)).abs()
        assert bool((err <= 6 * 2.0 ** -24 * plain.abs()).all())


@pytest.mark.parametrize("B,L,H,io,shared,phase", [
    (1, 4096, 1, "f32", False, 0),      # chunks of 16-piece columns; a length with two output reals behind the last whole tile
    (1, 2113, 1, "f32", False, 0),      # odd length, ragged last chunk and tile
    (4, 3008, 1, "bf16", False, 777),   # 8-piece columns, four rows of one weight set inside the output layer, phase on the last bin
    (5, 3008, 1, "bf16", False, 777),   # a fifth: hidden layer in its own launch
    (2, 2500, 5, "bf16", False, 0),     # 40 pieces a row
    (2, 2500, 2, "f32", True, 0),       # shared weights: rows over (b, h)
    (1, 33000, 3, "bf16", True, 0),     # many chunks
    (1, 40960, 32, "bf16", False, 0),   # more workgroups than run at once: hidden layer in its own launch
])
def test_gate_of_rows_summed_in_deep_chunks(oracle, B, L, H, io, shared, phase):
    """Lengths between the one-launch gate and 256 rows a chunk, at any alignment of a channel pair (same bits)."""
    from paper_2502_18394_amd import binding
    print(f"case B={B} L={L} H={H} io={io} shared={shared} phase={phase}", flush=True)
    p = synth.gate_params(41, 1 if shared else H, 64, L)
    vals, store = synth.tokens(42, (B, L, H, 64), io)
    P = binding.GateParams(p)
    q = to_device(store, io)
    got = binding.gate(q, P, 1.0 / L, phase_pos=phase)
    flat = torch.empty(q.numel() + 2, dtype=q.dtype, device="cuda")
    off = flat[2:].view(B, L, H, 64)
    off.copy_(q)
    assert torch.equal(binding.gate(off, P, 1.0 / L, phase_pos=phase), got)
    want = oracle.gate(oracle.pool_q(vals.astype(np.float64)), 1.0 / L, f64(p), L, phase)
    assert rel_l2(got.cpu().numpy(), want) <= 1e-5


@pytest.mark.parametrize("phase", [0, 777])
@pytest.mark.parametrize("B,H,Hg,n", [(1, 1, 1, 128), (3, 2, 2, 1600), (4, 1, 1, 8192), (5, 1, 1, 8192), (2, 2, 1, 65), (9, 3, 3, 2048),
                                      (33, 2, 1, 1024), (4, 4, 4, 4096), (4, 16, 16, 4096), (2, 2048, 2048, 512)])
def test_last_bin_of_every_row(oracle, B, H, Hg, n, phase):
    """Lengths whose last bin lies behind the last whole tile of the output layer: as a tile of its own, and with the last workgroup (up to
    four rows per weight set; the last two cases, with the hidden layer inside the launch and in front of it)."""
    from paper_2502_18394_amd import binding
    print(f"case B={B} H={H} Hg={Hg} n={n} phase={phase}", flush=True)
    p = synth.gate_params(61, Hg, 64, n)
    sq = np.random.default_rng(62).standard_normal((B, H, 64)) * 40.0
    got = binding.gate(torch.from_numpy(sq).cuda(), binding.GateParams(p), 1.0 / n, pooled=True, phase_pos=phase).cpu().numpy()
    want = oracle.gate(sq, 1.0 / n, f64(p), n, phase)
    assert rel_l2(got, want) <= 1e-5 and rel_l2(got[:, :, -1], want[:, :, -1]) <= 1e-5


@pytest.mark.parametrize("B,L,H,io,shared,phase", [
    (4, 4096, 2, "f32", False, 777),    # 64 chunks of four rows: the most that the output layer's workgroups add up themselves
    (1, 8192, 4, "bf16", True, 777),    # 128 of them: hidden layer in its own launch
    (1, 65536, 8, "f32", False, 0),     # rows of 2 KB in chunks of 128: the pass of whole rows
])
def test_gate_on_both_sides_of_what_workgroups_repeat(oracle, B, L, H, io, shared, phase):
    test_gate_of_rows_summed_in_deep_chunks(oracle, B, L, H, io, shared, phase)
