"""spectre_layer_forward (projection, pooled query, gate, mixer and the optional wavelet refinement in one call)
against the oracle's functions chained, Sec. 3.2 steps 1-4 and Sec. 3.5, and against the library's own separate calls.

On the four-step route with bf16 rows the call projects inside the row transforms (V never exists in memory) and
feeds the refinement from block sums the mixer emits; every other shape runs the separate kernels with V in the
workspace.  The oracle side adds no arithmetic: project -> pool -> gate -> mix -> level gates -> refinement."""
import numpy as np
import pytest
import torch

from gpu_util import TOL, f64, from_device, rel_l2, to_device
from paper_2502_18394_amd import synth

pytestmark = pytest.mark.gpu


def oracle_chain(oracle, x, Wq, Wv, p, wp, J):
    B, L, H, d = x.shape
    Q, V = oracle.project(x, Wq, Wv)
    sum_q = oracle.pool_q(Q)
    g = oracle.gate(sum_q, 1.0 / L, p, L, 0)
    out = oracle.mix_forward(V, g)
    if wp is not None:
        out = oracle.wrm_apply(out, oracle.wrm_gates(sum_q, 1.0 / L, wp, J), J)
    return out


def run_layer(oracle, B, L, H, io, J, seed, Hw=None):
    from paper_2502_18394_amd import binding
    d = 64
    Hw = H if Hw is None else Hw
    vals, store = synth.tokens(seed, (B, L, H, d), io)
    rng = np.random.default_rng(seed + 1)
    Wq = (0.125 * rng.standard_normal((Hw, d, d))).astype(np.float32)
    Wv = (0.125 * rng.standard_normal((Hw, d, d))).astype(np.float32)
    p = synth.gate_params(seed + 2, H, d, L)
    wp = synth.wrm_params(seed + 3, H, d, J) if J is not None else None
    P = binding.GateParams(p)
    W = binding.WrmParams(wp) if wp is not None else None
    x_d = to_device(store, io)
    Wq_d, Wv_d = torch.from_numpy(Wq).cuda(), torch.from_numpy(Wv).cuda()
    out = binding.layer_forward(x_d, Wq_d, Wv_d, P, W)
    # the same chain through the separate entry points
    v, _, sq = binding.project(x_d, Wq_d, Wv_d)
    g = binding.gate(sq, P, 1.0 / L, pooled=True)
    ref = binding.mix_forward(v, g)
    if W is not None:
        ref = binding.wrm_apply(ref, binding.wrm_gates(sq, W, 1.0 / L, pooled=True))
    torch.cuda.synchronize()
    bq = Wq if Hw == H else np.broadcast_to(Wq, (H, d, d))
    bv = Wv if Hw == H else np.broadcast_to(Wv, (H, d, d))
    want = oracle_chain(oracle, vals.astype(np.float64), bq.astype(np.float64), bv.astype(np.float64), f64(p),
                        f64(wp) if wp is not None else None, J)
    return from_device(out), from_device(ref), want


# bf16 rows on the four-step route, where the row transforms project: columns of 256, 1024 and 4096 points, one and several head
# groups, shared projection weights, refinement depths below and above the 8 levels a tile holds (an odd number of rows per
# lane, and with it a ragged last group of the matrix-core prologue: the many heads of 1792 points below; 768 runs in LDS).
@pytest.mark.parametrize("B,L,H,J,Hw", [(1, 8192, 8, None, None), (2, 8192, 3, 13, None), (1, 16384, 5, 6, None),
                                         (1, 768, 2, 8, None), (1, 12288, 2, 12, 1), (1, 32768, 4, 15, None),
                                         (1, 131072, 2, 17, None), (3, 2560, 2, 9, None), (1, 7168, 1, None, 1)])
def test_fused_layer_matches_oracle_chain_bf16(oracle, B, L, H, J, Hw):
    print(f"case B={B} L={L} H={H} J={J} Hw={Hw}", flush=True)
    got, ref, want = run_layer(oracle, B, L, H, "bf16", J, seed=synth.BASE_SEED + 500 + L + H, Hw=Hw)
    err, e_ref = rel_l2(got, want), rel_l2(got, ref)
    print(f"  vs oracle chain {err:.3e}  vs separate calls {e_ref:.3e}  differing {np.mean(got != ref):.2e}", flush=True)
    assert err <= TOL["bf16"]
    # same V bits, same kernels behind; the pooled query is summed in another order (1e-7 on the gate), and the
    # refinement's coarse sums are added in another order: a bf16 step here and there
    assert e_ref <= 2e-3 and np.mean(got != ref) < 2e-2


# every other shape runs the separate kernels inside the call: fp32 rows, the in-LDS lengths, 4096, padded lengths
@pytest.mark.parametrize("B,L,H,io,J", [(1, 8192, 2, "f32", 13), (2, 196, 3, "f32", 2), (2, 196, 3, "bf16", None),
                                        (1, 4096, 4, "bf16", 12), (1, 1000, 2, "bf16", 3), (1, 1024, 1, "f32", None),
                                        (1, 512, 32, "bf16", 9)])
def test_layer_on_the_other_routes_matches_oracle_chain(oracle, B, L, H, io, J):
    print(f"case B={B} L={L} H={H} io={io} J={J}", flush=True)
    got, ref, want = run_layer(oracle, B, L, H, io, J, seed=synth.BASE_SEED + 600 + L + H)
    err = rel_l2(got, want)
    print(f"  vs oracle chain {err:.3e}  identical to separate calls {np.array_equal(got, ref)}", flush=True)
    assert err <= (TOL["bf16"] if io == "bf16" else 2e-5)     # fp32: the gate's 1e-5 bar and the mixer's, chained
    assert np.array_equal(got, ref)                           # the very same kernels in the same order


@pytest.mark.parametrize("B,L,H,J", [(18, 1792, 32, None), (19, 1792, 31, 8), (32, 2048, 16, 11), (19, 2048, 28, 11)])
def test_layer_of_many_heads_of_1792_and_2048_points(oracle, B, L, H, J):
    """bf16 rows on both sides of 2^20 positions, from which these lengths take the projecting row transforms: 16 * 7 tile rows at
    1792 points, no multiple of the 32 of a matrix instruction.  Sampled heads against the oracle chain, and the whole against
    the separate calls."""
    from paper_2502_18394_amd import binding
    print(f"case B={B} L={L} H={H} J={J}", flush=True)
    d, seed = 64, synth.BASE_SEED + 730 + L + H
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((B, L, H, d), generator=gen, device="cuda").bfloat16()
    rng = np.random.default_rng(seed + 1)
    Wq, Wv = ((0.125 * rng.standard_normal((H, d, d))).astype(np.float32) for _ in range(2))
    p, wp = synth.gate_params(seed + 2, H, d, L), synth.wrm_params(seed + 3, H, d, J) if J is not None else None
    P, W = binding.GateParams(p), binding.WrmParams(wp) if wp is not None else None
    Wq_d, Wv_d = torch.from_numpy(Wq).cuda(), torch.from_numpy(Wv).cuda()
    out = binding.layer_forward(x, Wq_d, Wv_d, P, W)
    v, _, sq = binding.project(x, Wq_d, Wv_d)
    ref = binding.mix_forward(v, binding.gate(sq, P, 1.0 / L, pooled=True))
    if W is not None:
        ref = binding.wrm_apply(ref, binding.wrm_gates(sq, W, 1.0 / L, pooled=True))
    e_ref = float(torch.linalg.vector_norm(out.float() - ref.float()) / torch.linalg.vector_norm(ref.float()))
    print(f"  vs separate calls {e_ref:.3e}", flush=True)
    assert e_ref <= 2e-3                                       # bf16 steps of the rows, from sums in another order
    one = lambda q, h: {k: (a[h:h + 1] if isinstance(a, np.ndarray) else 1 if k == "Hg" else a) for k, a in q.items()}
    for b, h in ((0, 0), (B - 1, H - 1), (B // 2, H // 2)):
        rows = x[b:b + 1, :, h:h + 1].float().cpu().numpy().astype(np.float64)
        want = oracle_chain(oracle, rows, Wq[h:h + 1].astype(np.float64), Wv[h:h + 1].astype(np.float64), f64(one(p, h)),
                            f64(one(wp, h)) if wp is not None else None, J)
        assert rel_l2(from_device(out[b:b + 1, :, h:h + 1].contiguous()), want) <= TOL["bf16"]


def test_layer_of_many_heads(oracle):
    """2048 heads: the gate's preparation, with the query projection in it, in workgroups of 256 lanes."""
    got, ref, want = run_layer(oracle, 256, 60, 8, "f32", None, seed=synth.BASE_SEED + 700)
    assert rel_l2(got, want) <= 2e-5 and rel_l2(got, ref) <= 1e-6


@pytest.mark.parametrize("L", [256, 197])
def test_layer_of_a_length_that_is_not_ready_enqueues_nothing(L):
    """With only 512 points prepared the roots of unity of 256 points exist (as those of its columns), and those of the padded
    length of 197, but not the other tables of either length: the layer has to say so before its projection runs."""
    import ctypes
    from paper_2502_18394_amd import binding
    H, d = 2, 64
    print(f"case L={L}", flush=True)
    P = binding.GateParams(synth.gate_params(720, H, d, L))
    x, Wm = torch.ones((1, L, H, d), device="cuda"), torch.ones((H, d, d), device="cuda")
    out = torch.full_like(x, 7.0)
    torch.cuda.synchronize()
    binding.shutdown()
    binding.prepare(512, d)
    lib = binding.lib()
    ws = torch.full((lib.spectre_layer_workspace_bytes(1, L, H, d, binding.F32, ctypes.byref(P.c), None) + 256,), 7,
                    dtype=torch.uint8, device="cuda")
    at = ws.data_ptr() + (-ws.data_ptr()) % 256
    rc = lib.spectre_layer_forward(x.data_ptr(), Wm.data_ptr(), Wm.data_ptr(), H, ctypes.byref(P.c), None, out.data_ptr(), 1, L, H,
                                   d, binding.F32, at, ws.numel() - 256, None)
    torch.cuda.synchronize()
    assert rc == binding.ENOTREADY and b"spectre_prepare" in lib.spectre_last_error()
    assert bool((ws == 7).all()) and bool((out == 7.0).all())


def test_layer_rejects_bad_arguments():
    from paper_2502_18394_amd import binding
    d = 64
    x = torch.zeros((1, 1024, 2, d), device="cuda")
    Wm = torch.zeros((2, d, d), device="cuda")
    P_wrong = binding.GateParams(synth.gate_params(1, 2, d, 512))
    with pytest.raises(binding.SpectreError) as e:
        binding.layer_forward(x, Wm, Wm, P_wrong)              # gate built for another length
    assert e.value.code in (binding.EINVAL, binding.EUNSUPPORTED)
    P = binding.GateParams(synth.gate_params(1, 2, d, 1024))
    W_bad = binding.WrmParams(synth.wrm_params(2, 2, d, 11))   # 2^11 does not divide 1024
    with pytest.raises(binding.SpectreError):
        binding.layer_forward(x, Wm, Wm, P, W_bad)
    with pytest.raises(binding.SpectreError) as e:
        binding.layer_forward(x, Wm, Wm, P, out=x)             # out overlaps x
    assert e.value.code == binding.EINVAL
