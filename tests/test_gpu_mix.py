"""GPU parity of spectre_mix_forward against the fp64 oracle (Sec. 3.2 Eq. 3-4).

Bars (relative L2 over the whole output): 1e-5 for fp32 I/O, 2e-2 for bf16 I/O.
"""
import numpy as np
import pytest
import torch

from gpu_util import TOL, assert_close_elementwise, rel_l2
from paper_2502_18394_amd import synth

pytestmark = pytest.mark.gpu




def to_device(vals, store, io):
    if io == "bf16":
        return torch.from_numpy(store.view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(store).cuda()


def from_device(t):
    if t.dtype == torch.bfloat16:
        return synth.bf16_bits_to_f32(t.view(torch.int16).cpu().numpy().view(np.uint16))
    return t.cpu().numpy()


def run_case(oracle, B, L, H, d, io, seed, gate="random", flags=0):
    from paper_2502_18394_amd import binding
    vals, store = synth.tokens(seed, (B, L, H, d), io)
    if isinstance(gate, str):
        g = synth.random_gate(seed + 1, B, H, L)
    else:
        g = gate
    out = binding.mix_forward(to_device(vals, store, io), torch.from_numpy(g).cuda(), flags=flags)
    torch.cuda.synchronize()
    got = from_device(out)
    want = oracle.mix_forward(vals.astype(np.float64), g.astype(np.complex128))
    return got, want, vals


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("B,L,H", [(1, 256, 1), (2, 512, 3), (1, 1024, 1), (1, 2048, 2), (2, 4096, 2),
                                   (1, 8192, 3), (1, 16384, 1), (1, 32768, 2), (4, 8192, 32), (3, 16384, 11)])
def test_mix_forward_matches_oracle(oracle, B, L, H, io):
    print(f"case B={B} L={L} H={H} io={io}", flush=True)
    got, want, _ = run_case(oracle, B, L, H, 64, io, seed=synth.BASE_SEED + L + H)
    err = rel_l2(got, want)
    print(f"  rel_l2={err:.3e}", flush=True)
    assert err <= TOL[io]
    assert_close_elementwise(got, want, io, L)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("B,H", [(3, 5), (1, 32), (1, 1)])
def test_one_kernel_path_at_4096_and_the_three_kernel_path_behind_it(oracle, options, B, H, io):
    """L = 4096 runs as a single kernel (whole columns in LDS; head counts that are and are not multiples of the
    eight workgroup slots per round).  With the fused-4096 option off the same call takes the three four-step kernels
    (N1 = 256, N2 = 16), which keeps that plan covered by a mixer test; both must match the oracle."""
    from paper_2502_18394_amd import binding
    L = 4096
    print(f"case B={B} H={H} io={io}", flush=True)
    assert binding.mix_workspace_bytes(B, L, H, 64, binding.BF16) == 256
    got, want, _ = run_case(oracle, B, L, H, 64, io, seed=synth.BASE_SEED + 11 * H)
    options(binding.OPT_FUSED_4096, 0)
    assert binding.mix_workspace_bytes(B, L, H, 64, binding.BF16) > B * H * L * 8
    got3, _, _ = run_case(oracle, B, L, H, 64, io, seed=synth.BASE_SEED + 11 * H)
    e1, e3 = rel_l2(got, want), rel_l2(got3, want)
    print(f"  one kernel {e1:.3e}  three kernels {e3:.3e}", flush=True)
    assert e1 <= TOL[io] and e3 <= TOL[io]


@pytest.mark.parametrize("B,L,H", [(1, 8192, 3), (2, 12288, 2), (1, 32768, 5), (1, 131072, 1)])
def test_bf16_scratch_option_stays_within_the_bf16_bar(oracle, B, L, H):
    """Flag SPECTRE_MIX_BF16_SCRATCH: the three four-step kernels exchange bfloat16 pairs instead of fp32 pairs (opt-in, bf16
    rows only).  Two more roundings to 8 mantissa bits: the error against the oracle must stay well inside the bar
    for bf16 rows; fp32 rows ignore the switch and keep the fp32 bar."""
    from paper_2502_18394_amd import binding
    seed = synth.BASE_SEED + 13 * H
    plain, want, _ = run_case(oracle, B, L, H, 64, "bf16", seed=seed)
    got, _, _ = run_case(oracle, B, L, H, 64, "bf16", seed=seed, flags=binding.MIX_BF16_SCRATCH)
    e0, e1 = rel_l2(plain, want), rel_l2(got, want)
    print(f"case B={B} L={L} H={H}: fp32 scratch {e0:.3e}  bf16 scratch {e1:.3e}", flush=True)
    assert e0 <= TOL["bf16"] and e1 <= 5e-3
    assert not np.array_equal(plain, got)                     # the switch did take the other kernels
    if L <= 12288:
        got32, want32, _ = run_case(oracle, B, L, H, 64, "f32", seed=seed, flags=binding.MIX_BF16_SCRATCH)
        assert rel_l2(got32, want32) <= TOL["f32"]


@pytest.mark.parametrize("B,H,mb,one_lane", [(1, 11, 9, False), (1, 7, 9, False), (3, 1, 3, False), (1, 3, 3, True),
                                              (2, 5, 2, False), (1, 13, 9, True)])
def test_head_groups_of_any_size_give_the_same_rows(oracle, options, B, H, mb, one_lane):
    """Long calls take their heads in groups (one stream, or two streams with an even number of groups whose sizes
    differ by at most one head, some of them empty when there are fewer heads than groups).  Every head is
    transformed on its own, so the grouping must not change a bit; the scratch-size option shrinks the groups far enough
    to get several of them at a small length.  The same groupings with the bfloat16 scratch stay within its bar."""
    L, io = 6144, "bf16"                      # 1.5 MB a head
    seed = synth.BASE_SEED + 17 * H + B
    from paper_2502_18394_amd import binding
    plain, want, _ = run_case(oracle, B, L, H, 64, io, seed=seed)
    assert rel_l2(plain, want) <= TOL[io]
    options(binding.OPT_SCRATCH_MB, mb)
    if one_lane:
        options(binding.OPT_LANES, 1)
    got, _, _ = run_case(oracle, B, L, H, 64, io, seed=seed)
    print(f"case B={B} H={H} chunk_mb={mb} one_lane={one_lane}: identical {np.array_equal(got, plain)}", flush=True)
    assert np.array_equal(got, plain)
    got16, _, _ = run_case(oracle, B, L, H, 64, io, seed=seed, flags=binding.MIX_BF16_SCRATCH)
    options(binding.OPT_SCRATCH_MB, -1)
    options(binding.OPT_LANES, -1)
    plain16, _, _ = run_case(oracle, B, L, H, 64, io, seed=seed, flags=binding.MIX_BF16_SCRATCH)
    assert np.array_equal(got16, plain16) and rel_l2(got16, want) <= 5e-3


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("B,H", [(64, 8), (43, 12), (171, 3)])
def test_patch_grid_length_with_many_heads_takes_its_own_kernel(oracle, options, B, H, io):
    """L = 196 (14 x 14 patches) with many heads: the compile-time form of the in-LDS kernel for many heads against the general
    kernel (the compile-time option, switched off, forces that one).  Both must match the oracle and, to the rounding of two fp32
    transforms, each other."""
    L = 196
    seed = synth.BASE_SEED + 19 * H + B
    from paper_2502_18394_amd import binding
    got, want, _ = run_case(oracle, B, L, H, 64, io, seed=seed)
    options(binding.OPT_SLAB_COMPILE_TIME, 0)
    general, _, _ = run_case(oracle, B, L, H, 64, io, seed=seed)
    e1, e2, e12 = rel_l2(got, want), rel_l2(general, want), rel_l2(got, general)
    print(f"case B={B} H={H} io={io}: own kernel {e1:.3e}  general {e2:.3e}  between {e12:.3e}", flush=True)
    assert e1 <= TOL[io] and e2 <= TOL[io] and e12 <= (1e-6 if io == "f32" else 2e-3)


@pytest.mark.parametrize("B,L,H,io", [(1, 8192, 8, "f32"), (2, 7168, 12, "bf16"), (1, 6144, 16, "bf16"), (3, 5120, 8, "bf16")])
def test_head_affine_placement_changes_no_bit(oracle, options, B, L, H, io):
    """Four-step lengths up to 8192 with a multiple of 8 heads in a call place every workgroup of a head on one XCD
    and walk the heads up, down, up through the three kernels (L2 reuse).  It is only a renumbering of workgroups:
    the rows must equal those of the plain numbering (head-affine option off) bit for bit, and match the oracle."""
    seed = synth.BASE_SEED + 23 * H + L
    from paper_2502_18394_amd import binding
    got, want, _ = run_case(oracle, B, L, H, 64, io, seed=seed)
    options(binding.OPT_HEAD_AFFINE, 0)
    plain, _, _ = run_case(oracle, B, L, H, 64, io, seed=seed)
    err = rel_l2(got, want)
    print(f"case B={B} L={L} H={H} io={io}: rel_l2 {err:.3e} identical {np.array_equal(got, plain)}", flush=True)
    assert err <= TOL[io] and np.array_equal(got, plain)


@pytest.mark.parametrize("B,H,io", [(1, 8, "f32"), (2, 8, "bf16")])
def test_head_affine_placement_of_4096_point_columns_changes_no_bit(oracle, options, B, H, io):
    """The same at 12288 points on 4096-point columns, which mix_forward_static takes there (mix_forward has 1024-point ones)."""
    from paper_2502_18394_amd import binding
    L = 12288
    print(f"case B={B} H={H} io={io}", flush=True)
    vals, store = synth.tokens(synth.BASE_SEED + 24 * H + B, (B, L, H, 64), io)
    gate = synth.random_gate(synth.BASE_SEED + 25, B, H, L)
    v, g = to_device(vals, store, io), torch.from_numpy(gate).cuda()
    got = from_device(binding.mix_forward_static(v, g))
    options(binding.OPT_HEAD_AFFINE, 0)
    plain = from_device(binding.mix_forward_static(v, g))
    assert np.array_equal(got, plain)
    assert rel_l2(got, oracle.mix_forward(vals.astype(np.float64), gate.astype(np.complex128))) <= TOL[io]


@pytest.mark.parametrize("L,most", [(1792, 585), (2048, 512)])
def test_bf16_rows_beyond_the_memory_side_cache_take_the_four_step_kernels(oracle, L, most):
    """bf16 rows of 1792 and 2048 points: the largest call in LDS (2^20 positions) and the first on the four-step route.  Other
    kernels, so not the same bits, but the same rows to a bf16 step; the first and the last head against the oracle.  fp32 rows
    stay in LDS: the same bits on both sides."""
    from paper_2502_18394_amd import binding
    print(f"case L={L} most={most}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(L)
    v = torch.randn((1, L, most + 1, 64), generator=gen, device="cuda")
    g = torch.view_as_complex(torch.randn((1, most + 1, L // 2 + 1, 2), generator=gen, device="cuda"))
    f32 = binding.mix_forward(v, g)
    assert torch.equal(binding.mix_forward(v[:, :, :most].contiguous(), g[:, :most].contiguous()), f32[:, :, :most])
    v = v.bfloat16()
    many = binding.mix_forward(v, g)
    few = binding.mix_forward(v[:, :, :most].contiguous(), g[:, :most].contiguous())
    assert not torch.equal(many[:, :, :most], few)
    diff = torch.linalg.vector_norm(many[:, :, :most].float() - few.float()) / torch.linalg.vector_norm(few.float())
    assert float(diff) <= 2e-3
    for out, h in ((few, 0), (few, most - 1), (many, 0), (many, most)):
        want = oracle.mix_forward(v[:, :, h:h + 1].float().cpu().numpy().astype(np.float64),
                                  g[:, h:h + 1].cpu().numpy().astype(np.complex128))
        assert_close_elementwise(from_device(out[:, :, h:h + 1].contiguous()), want, "bf16", L)


@pytest.mark.parametrize("B,L,H,io", [(1, 7168, 8, "bf16"), (2, 2048 * 3, 3, "f32"), (1, 16384, 5, "f32"), (1, 131072, 2, "bf16")])
def test_lane_shuffle_exchange_changes_no_bit(oracle, options, B, L, H, io):
    """The column kernel can move values between the 16 lanes of a sub-transform with cross-lane (DPP) moves instead
    of through LDS (both 256-point columns, where every exchange is of that kind, and 4096-point ones, where the
    inner two are).  It is data movement only: same rows bit for bit, and they match the oracle."""
    from paper_2502_18394_amd import binding
    seed = synth.BASE_SEED + 29 * H + L
    got, want, _ = run_case(oracle, B, L, H, 64, io, seed=seed)
    options(binding.OPT_LANE_SHUFFLES, 1)
    shuffled, _, _ = run_case(oracle, B, L, H, 64, io, seed=seed)
    err = rel_l2(shuffled, want)
    print(f"case B={B} L={L} H={H} io={io}: rel_l2 {err:.3e} identical {np.array_equal(got, shuffled)}", flush=True)
    assert err <= TOL[io] and np.array_equal(got, shuffled)


def test_identity_gate_returns_input_on_gpu(oracle):
    B, L, H, d = 1, 4096, 2, 64
    g = np.ones((B, H, L // 2 + 1), np.complex64)
    got, want, vals = run_case(oracle, B, L, H, d, "f32", seed=7, gate=g)
    assert rel_l2(got, vals) <= 1e-5
    assert rel_l2(got, want) <= 1e-5


def test_pure_phase_gate_shifts_on_gpu(oracle):
    B, L, H, d, s = 1, 1024, 2, 64, 137
    k = np.arange(L // 2 + 1)
    g = np.broadcast_to(np.exp(-2j * np.pi * ((k * s) % L) / L), (B, H, L // 2 + 1)).astype(np.complex64)
    got, want, vals = run_case(oracle, B, L, H, d, "f32", seed=8, gate=np.ascontiguousarray(g))
    assert rel_l2(got, np.roll(vals, s, axis=1)) <= 1e-5


def test_run_to_run_bitwise_identical():
    from paper_2502_18394_amd import binding
    vals, store = synth.tokens(3, (1, 8192, 4, 64), "bf16")
    g = torch.from_numpy(synth.random_gate(4, 1, 4, 8192)).cuda()
    v = to_device(vals, store, "bf16")
    a = binding.mix_forward(v, g).view(torch.int16).clone()
    b = binding.mix_forward(v, g).view(torch.int16)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("B,L,H", [(2, 196, 3), (1, 2, 1), (3, 4, 2), (2, 8, 2), (1, 49, 2), (2, 60, 1), (1, 105, 3),
                                   (2, 128, 2), (1, 360, 2), (1, 500, 1), (1, 175, 2), (16, 256, 16), (8, 512, 32),
                                   (1, 2048, 32), (4, 2000, 8), (1, 1920, 3), (50, 700, 6), (1, 1024, 64), (3, 1215, 2),
                                   (2, 1029, 40), (1, 2048, 1)])
def test_short_and_mixed_radix_lengths(oracle, B, L, H, io):
    """Whole-slab path: non-power-of-two lengths (4*7*7 = 196 of the ViT grid, odd lengths), short ones, and
    lengths up to 2048 with few heads (4 to 32 channel pairs per workgroup)."""
    print(f"case B={B} L={L} H={H} io={io}", flush=True)
    got, want, _ = run_case(oracle, B, L, H, 64, io, seed=synth.BASE_SEED + 7 * L + H)
    err = rel_l2(got, want)
    print(f"  rel_l2={err:.3e}", flush=True)
    assert err <= TOL[io]
    assert_close_elementwise(got, want, io, L)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("B,L,H", [(1, 196, 9), (5, 196, 27), (1, 256, 3), (3, 256, 43), (1, 320, 9), (1, 400, 9), (1, 448, 3),
                                   (1, 512, 7), (1, 640, 3), (3, 768, 3), (1, 896, 2), (1, 1024, 8), (1, 1024, 9), (1, 1280, 3),
                                   (1, 1536, 3), (1, 1792, 9), (1, 2048, 3)])
def test_lengths_of_compile_time_radices(oracle, options, B, L, H, io):
    """Every split of the kernel whose radices are compile-time constants, in its forms for few and for many heads and with
    head counts that are no multiple of 8, against the oracle and the general kernel.  Between the two: the rounding of two
    fp32 transforms, 2.5e-7 each, or one bf16 step of a few of the rows."""
    from paper_2502_18394_amd import binding
    print(f"case B={B} L={L} H={H} io={io}", flush=True)
    seed = synth.BASE_SEED + 29 * L + H
    got, want, _ = run_case(oracle, B, L, H, 64, io, seed=seed)
    assert rel_l2(got, want) <= (1e-6 if io == "f32" else 2e-3)
    assert_close_elementwise(got, want, io, L)
    options(binding.OPT_SLAB_COMPILE_TIME, 0)
    general, _, _ = run_case(oracle, B, L, H, 64, io, seed=seed)
    assert rel_l2(got, general) <= (1e-6 if io == "f32" else 2e-3)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("L,most", [(144, 64), (196, 64), (144, 128), (196, 128), (256, 64), (448, 32), (576, 42), (768, 32), (784, 32), (896, 32),
                                    (1024, 16), (1280, 32), (1536, 16), (1792, 16)])
def test_forms_for_few_and_for_many_heads(oracle, options, L, most, io):
    """The last call that takes the form for few heads and the first that takes the other, against the general kernel (bounds as
    above), and the first head of both against the oracle."""
    from paper_2502_18394_amd import binding
    for H in (most, most + 1):
        print(f"case L={L} H={H} io={io}", flush=True)
        vals, store = synth.tokens(synth.BASE_SEED + 41 * L, (1, L, H, 64), io)
        gate = synth.random_gate(synth.BASE_SEED + 41 * L + 1, 1, H, L)
        v, g = to_device(vals, store, io), torch.from_numpy(gate).cuda()
        got = from_device(binding.mix_forward(v, g))
        options(binding.OPT_SLAB_COMPILE_TIME, 0)
        general = from_device(binding.mix_forward(v, g))
        options(binding.OPT_SLAB_COMPILE_TIME, -1)
        assert rel_l2(got, general) <= (1e-6 if io == "f32" else 2e-3)
        want = oracle.mix_forward(np.ascontiguousarray(vals[:, :, :1]).astype(np.float64),
                                  np.ascontiguousarray(gate[:, :1]).astype(np.complex128))
        assert_close_elementwise(got[:, :, :1], want, io, L)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("L", [144, 196, 256])
def test_patch_grids_whose_rows_pass_the_caches_by(oracle, L, io):
    """More than 100 MB in and out: rows on a 128-byte boundary bypass the caches, others do not, fp32 rows of 196 also change
    the pairs per workgroup.  All the same bits as a part of the heads below that size; first and last head against the oracle."""
    from paper_2502_18394_amd import binding
    B, H = -(-120_000_000 // (L * 12 * 256 * (2 if io == "f32" else 1))), 12
    print(f"case B={B} L={L} H={H} io={io}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(L)
    v = torch.randn((B, L, H, 64), generator=gen, device="cuda").to(torch.float32 if io == "f32" else torch.bfloat16)
    g = torch.view_as_complex(torch.randn((B, H, L // 2 + 1, 2), generator=gen, device="cuda"))
    out = binding.mix_forward(v, g)
    n = B // 3
    assert torch.equal(binding.mix_forward(v[:n].contiguous(), g[:n].contiguous()), out[:n])
    aside = torch.empty(v.numel() + 16, dtype=v.dtype, device="cuda")[16:].view(v.shape)
    aside.copy_(v)
    assert aside.data_ptr() % 128 != 0 and torch.equal(binding.mix_forward(aside, g, out=torch.empty_like(v)), out)
    for b, h in ((0, 0), (B - 1, H - 1)):
        want = oracle.mix_forward(v[b:b + 1, :, h:h + 1].float().cpu().numpy().astype(np.float64),
                                  g[b:b + 1, h:h + 1].cpu().numpy().astype(np.complex128))
        assert_close_elementwise(from_device(out[b:b + 1, :, h:h + 1].contiguous()), want, io, L)


@pytest.mark.parametrize("B,L,H,io", [(1, 12288, 3, "f32"), (1, 12288, 8, "bf16"), (1, 20480, 1, "f32"), (3, 24576, 3, "bf16"),
                                      (1, 28672, 2, "f32"), (1, 32768, 5, "bf16"), (1, 24576, 27, "f32")])
def test_columns_of_1024_points(oracle, B, L, H, io):
    """The plan with 1024-point columns, with plane counts that are no multiple of 8 and a call of two head groups.  1e-6:
    1.9e-7 measured for fp32 rows."""
    print(f"case B={B} L={L} H={H} io={io}", flush=True)
    got, want, _ = run_case(oracle, B, L, H, 64, io, seed=synth.BASE_SEED + 31 * L + H)
    assert rel_l2(got, want) <= (1e-6 if io == "f32" else 2e-3)
    assert_close_elementwise(got, want, io, L)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("B,H", [(1, 1), (2, 8), (1, 17), (3, 11)])
def test_4096_points_with_few_and_many_heads(oracle, options, B, H, io):
    """Two and four pairs per workgroup (up to 16 heads and above), from tensors off a 16-byte boundary as well, against the
    oracle and the three kernels of the four-step route."""
    from paper_2502_18394_amd import binding
    L = 4096
    print(f"case B={B} H={H} io={io}", flush=True)
    seed = synth.BASE_SEED + 37 * H + B
    got, want, _ = run_case(oracle, B, L, H, 64, io, seed=seed)
    assert rel_l2(got, want) <= (1e-6 if io == "f32" else 2e-3)
    assert_close_elementwise(got, want, io, L)
    vals, store = synth.tokens(seed, (B, L, H, 64), io)
    v = to_device(vals, store, io)
    g = torch.from_numpy(synth.random_gate(seed + 1, B, H, L)).cuda()
    off = torch.empty(v.numel() + 2, dtype=v.dtype, device="cuda")[2:].view_as(v)
    off.copy_(v)
    assert off.data_ptr() % 16 != 0 and np.array_equal(from_device(binding.mix_forward(off, g)), got)
    options(binding.OPT_FUSED_4096, 0)
    three, _, _ = run_case(oracle, B, L, H, 64, io, seed=seed)
    assert rel_l2(got, three) <= (1e-6 if io == "f32" else 2e-3)


@pytest.mark.parametrize("L", [196, 256])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_streamed_rows_change_no_bit(L, dtype):
    """Calls too large for the memory-side cache read and write their rows past the caches, from tensors on a line boundary:
    the same bits as a part of the batch alone, and as from a tensor off that boundary."""
    from paper_2502_18394_amd import binding
    B, H = 256, 12
    print(f"case L={L} {dtype}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(L)
    v = torch.randn((B, L, H, 64), generator=gen, device="cuda").to(dtype)
    g = torch.view_as_complex(torch.randn((B, H, L // 2 + 1, 2), generator=gen, device="cuda"))
    out = binding.mix_forward(v, g)
    assert torch.equal(binding.mix_forward(v[64:96].contiguous(), g[64:96].contiguous()), out[64:96])
    off = torch.empty(v.numel() + 16, dtype=dtype, device="cuda")[16:].view_as(v)
    off.copy_(v)
    assert off.data_ptr() % 128 != 0 and torch.equal(binding.mix_forward(off, g), out)


@pytest.mark.parametrize("L", [127, 131, 157, 163, 199, 211, 223, 227, 251, 257, 319, 331, 383, 389, 443, 449, 509, 521])
def test_lengths_at_the_edges_of_the_padded_ones(oracle, L):
    """Lengths on both sides of every length that the data pass of the padded convolution has up to 1024 points."""
    got, want, _ = run_case(oracle, 1, L, 3, 64, "f32", seed=synth.BASE_SEED + L)
    print(f"case L={L} rel_l2={rel_l2(got, want):.3e}", flush=True)
    assert rel_l2(got, want) <= 1e-6


def test_vit_config_full_size(oracle):
    """Config 5 at its real size: B=256, L=196, H=12, fp32."""
    c = synth.CONFIGS["vit_196"]
    got, want, _ = run_case(oracle, c["B"], c["L"], c["H"], c["d"], c["io"], seed=synth.BASE_SEED + 5)
    err = rel_l2(got, want)
    print(f"  rel_l2={err:.3e}", flush=True)
    assert err <= 1e-5
    assert_close_elementwise(got, want, c["io"], c["L"])


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("B,L,H", [(1, 11, 1), (2, 197, 3), (1, 1, 2), (1, 1000, 2), (1, 1031, 1), (2, 3000, 2),
                                   (1, 12289, 1), (3, 640, 40), (1, 3 * 4096, 2), (2, 1021, 2), (1, 509, 3),
                                   (3, 257, 5), (16, 197, 12)])
def test_any_other_length(oracle, B, L, H, io):
    """Lengths with neither a four-step nor an in-LDS plan (primes, 197 = 14*14 patches + a class token):
    zero-padded convolution with a chirp-z evaluated kernel; padded lengths up to 2048 (L <= 1024: 11, 197, 257,
    509, 1021) run the data pass in the in-LDS kernel, longer ones (1031, 3000, 12289) in the four-step kernels."""
    print(f"case B={B} L={L} H={H} io={io}", flush=True)
    got, want, _ = run_case(oracle, B, L, H, 64, io, seed=synth.BASE_SEED + 11 * L + H)
    err = rel_l2(got, want)
    print(f"  rel_l2={err:.3e}", flush=True)
    assert err <= TOL[io]
    assert_close_elementwise(got, want, io, 16 * L)        # padded transform, and the kernel came through two more


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("B,L,H", [(1, 768, 2), (2, 1280, 1), (1, 1792, 3), (1, 1536, 2), (1, 2560, 1), (2, 3072, 2),
                                   (1, 3584, 1), (1, 5120, 2), (1, 6144, 3), (1, 7168, 1), (1, 12288, 2), (1, 20480, 1),
                                   (1, 28672, 2), (1, 49152, 1), (1, 98304, 1), (1, 114688, 1)])
def test_four_step_with_an_odd_factor(oracle, B, L, H, io):
    """L = N1 * N2 with N1 = 256 or 4096 and N2 = 3, 5, 7 times a power of two (<= 28): the same four-step
    kernels as the power-of-two lengths, the small in-register transform by the prime-factor algorithm."""
    print(f"case B={B} L={L} H={H} io={io}", flush=True)
    got, want, _ = run_case(oracle, B, L, H, 64, io, seed=synth.BASE_SEED + 13 * L + H)
    err = rel_l2(got, want)
    print(f"  rel_l2={err:.3e}", flush=True)
    assert err <= TOL[io]
    assert_close_elementwise(got, want, io, L)


def test_any_other_length_identity_and_shift(oracle):
    B, L, H, d, s = 1, 1000, 2, 64, 333
    k = np.arange(L // 2 + 1)
    g = np.ones((B, H, L // 2 + 1), np.complex64)
    got, want, vals = run_case(oracle, B, L, H, d, "f32", seed=9, gate=g)
    assert rel_l2(got, vals) <= 1e-5
    g = np.broadcast_to(np.exp(-2j * np.pi * ((k * s) % L) / L), (B, H, L // 2 + 1)).astype(np.complex64)
    got, want, vals = run_case(oracle, B, L, H, d, "f32", seed=10, gate=np.ascontiguousarray(g))
    assert rel_l2(got, np.roll(vals, s, axis=1)) <= 1e-5


def test_unsupported_lengths_are_refused():
    from paper_2502_18394_amd import binding
    v = torch.zeros((1, 65537, 1, 64), device="cuda")
    g = torch.zeros((1, 1, 32769), dtype=torch.complex64, device="cuda")
    with pytest.raises(binding.SpectreError) as e:
        binding.mix_forward(v, g)
    assert e.value.code == binding.EUNSUPPORTED
    assert not binding.length_supported(3 * 131072, 64) and binding.length_supported(196, 64)


def _route_boundary_cases():
    """Seeded draw of shapes around the points where the mixer changes kernels: the in-LDS limit (2048), the
    one-kernel length (4096), four-step lengths and their neighbours, head counts around multiples of eight."""
    rng = np.random.default_rng(synth.BASE_SEED + 900)
    anchors = [2048, 4096, 8192, 1024, 512, 256, 3 * 256, 5 * 256, 7 * 256, 3 * 4096 // 4, 196, 1000]
    cases = []
    for i in range(24):
        a = int(anchors[i % len(anchors)])
        L = max(1, a + int(rng.integers(-2, 3)))
        B = int(rng.integers(1, 4))
        H = int(rng.choice([1, 2, 3, 5, 7, 8, 9, 16, 17]))
        cases.append((B, L, H, "bf16" if rng.integers(0, 2) else "f32"))
    return cases


@pytest.mark.parametrize("B,L,H,io", _route_boundary_cases())
def test_shapes_around_the_route_boundaries(oracle, B, L, H, io):
    print(f"case B={B} L={L} H={H} io={io}", flush=True)
    got, want, _ = run_case(oracle, B, L, H, 64, io, seed=synth.BASE_SEED + 17 * L + H + B)
    err = rel_l2(got, want)
    print(f"  rel_l2={err:.3e}", flush=True)
    assert err <= TOL[io]
    assert_close_elementwise(got, want, io, 16 * L)


@pytest.mark.parametrize("H", [(1 << 19) - 1, 1 << 19])
def test_rows_4_gb_apart(H):
    """The last number of heads of 512 bf16 rows whose lanes' offsets fit 32 bits and the first that needs 64 (34 GB of rows): the first,
    a middle and the last head bit for bit as in a call of a few of them."""
    from paper_2502_18394_amd import binding
    L, at = 512, [0, H // 2, H - 1]
    v = torch.empty((1, L, H, 64), dtype=torch.bfloat16, device="cuda")
    g = torch.empty((1, H, L // 2 + 1), dtype=torch.complex64, device="cuda")
    few = torch.randn(1, L, 200, 64, device="cuda").to(torch.bfloat16)
    gate = torch.view_as_complex(torch.randn(1, 200, L // 2 + 1, 2, device="cuda"))
    for i, h in enumerate(at):
        v[:, :, h], g[:, h] = few[:, :, i], gate[:, i]
    want = binding.mix_forward(few, gate)
    got = binding.mix_forward(v, g)
    for i, h in enumerate(at):
        assert torch.equal(got[:, :, h], want[:, :, i])


@pytest.mark.parametrize("L,io,heads", [
    (8192, "bf16", (31, 32)), (16384, "bf16", (15, 16)),                  # lines through the L2 from 32 MB on
    (5120, "f32", (12, 13, 44, 45)), (7168, "bf16", (9, 10, 73, 74)),     # scalar addresses up to 16 MB, and from 56 and 128 MB on
    (6144, "f32", (10, 11, 20)), (28672, "f32", (2, 3, 5)),               # scalar addresses of 24 and 28 fp32 rows at every size
    (3072, "f32", (24, 32, 48)), (49152, "f32", (1, 2, 3)),               # columns through the L2 but for 24 to 32 and 20 to 26 MB
])
def test_forms_by_the_size_of_the_scratch_change_no_bit(L, io, heads):
    from paper_2502_18394_amd import binding
    gen = torch.Generator(device="cuda").manual_seed(L)
    v = torch.randn((1, L, max(heads), 64), generator=gen, device="cuda").to(torch.bfloat16 if io == "bf16" else torch.float32)
    g = torch.view_as_complex(torch.randn((1, max(heads), L // 2 + 1, 2), generator=gen, device="cuda"))
    few = [binding.mix_forward(v[:, :, h:h + 1].contiguous(), g[:, h:h + 1].contiguous()) for h in (0, min(heads) - 1)]
    for H in heads:
        print(f"case L={L} io={io} H={H}", flush=True)
        got = binding.mix_forward(v[:, :, :H].contiguous(), g[:, :H].contiguous())
        for h, want in zip((0, min(heads) - 1), few):
            assert torch.equal(got[:, :, h:h + 1], want)


@pytest.mark.parametrize("H", [(1 << 21) - 1, 1 << 21])
@pytest.mark.parametrize("L", [256, 101])
def test_streamed_and_padded_rows_4_gb_apart(L, H):
    """As above for rows that pass the caches by (256 points in 16 x 16, 69 GB of rows) and padded rows (101 on the same, 27 GB)."""
    from paper_2502_18394_amd import binding
    at = [0, H // 2, H - 1]
    gen = torch.Generator(device="cuda").manual_seed(L)
    v = torch.empty((1, L, H, 64), dtype=torch.bfloat16, device="cuda")
    g = torch.empty((1, H, L // 2 + 1), dtype=torch.complex64, device="cuda")
    few = torch.randn((1, L, 200, 64), generator=gen, device="cuda").to(torch.bfloat16)
    gate = torch.view_as_complex(torch.randn((1, 200, L // 2 + 1, 2), generator=gen, device="cuda"))
    for i, h in enumerate(at):
        v[:, :, h], g[:, h] = few[:, :, i], gate[:, i]
    want = binding.mix_forward(few, gate)
    print(f"case L={L} H={H}", flush=True)
    got = binding.mix_forward(v, g)
    for i, h in enumerate(at):
        assert torch.equal(got[:, :, h], want[:, :, i])
