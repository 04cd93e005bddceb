"""GPU parity of the decode step.  The two-launch form at the edges of its tiling: one chunk of 128 bins and many, window
lengths with an odd factor, one and several sequences per workgroup, shared and per-head gate weights.  And the form of
separate launches that gates of another width, with taps or off their alignment take."""
import numpy as np
import pytest
import torch

from gpu_util import TOL, f64, from_device, rel_l2, to_device
from paper_2502_18394_amd import synth

pytestmark = pytest.mark.gpu


def run_steps(oracle, B, H, N, Hg, io, defer, modrelu=True, steps=7, d_g=64, taps=0, shift=0):
    """Steps while the window fills up and wraps, each compared, and the state after them."""
    from paper_2502_18394_amd import binding
    d, T0 = 64, N - 3
    print(f"case B={B} H={H} N={N} Hg={Hg} io={io} defer={defer} modrelu={modrelu} d_g={d_g} taps={taps} shift={shift}", flush=True)
    c, oc = binding.PrefixCache(B, H, d, N, defer=defer), oracle.PrefixCache(B, H, d, N)
    v, vs = synth.tokens(800 + N, (B, T0 + steps, H, d), io)
    q, qs = synth.tokens(801 + N, (B, T0 + steps, H, d), io)
    p = synth.gate_params(802 + B, Hg, d, N, d_g=d_g, modrelu=modrelu)
    if taps:
        p["toeplitz"] = synth.toeplitz_taps(803, Hg, taps, std=0.3)
    P = binding.GateParams(p)
    if shift:                                         # W2 `shift` floats off the start of its allocation
        w2 = torch.empty(P.t["W2"].numel() + shift, device="cuda")
        w2[shift:] = P.t["W2"].reshape(-1)
        P.t["W2"] = w2
        P.c.W2 = w2.data_ptr() + 4 * shift
    cut = lambda a, i, j: np.ascontiguousarray(a[:, i:j])
    c.update(to_device(cut(vs, 0, T0), io), to_device(cut(qs, 0, T0), io))
    oc.prefill(cut(v, 0, T0).astype(np.float64), cut(q, 0, T0).astype(np.float64))
    for i in range(T0, T0 + steps):
        out = c.step(to_device(cut(vs, i, i + 1), io), to_device(cut(qs, i, i + 1), io), P)
        oc.update(cut(v, i, i + 1).astype(np.float64), cut(q, i, i + 1).astype(np.float64))
        assert rel_l2(from_device(out), oc.readout_newest(oracle.gate(oc.sum_q, 1.0 / N, f64(p), N, 0))) <= TOL[io]
    c.flush()
    assert rel_l2(c.prefix_fft.cpu().numpy(), oc.spec) <= 1e-5
    assert rel_l2(c.sum_q.cpu().numpy(), oc.sum_q) <= 1e-12
    assert np.array_equal(c.v_buf.cpu().numpy(), oc.v_buf.astype(np.float32))
    assert np.array_equal(c.q_buf.cpu().numpy(), oc.q_buf.astype(np.float32))


@pytest.mark.parametrize("B,H,N,Hg,io,defer,modrelu", [
    (1, 1, 256, 1, "f32", 0, True), (5, 3, 256, 3, "bf16", 0, True), (3, 2, 768, 2, "f32", 0, False),
    (9, 1, 1280, 1, "f32", 0, True), (4, 32, 2048, 1, "bf16", 0, True),
    (1, 1, 256, 1, "f32", 4, True), (5, 3, 512, 3, "bf16", 3, True), (2, 3, 1792, 1, "f32", 32, False),
    (9, 32, 1024, 32, "f32", 2, True)])
def test_decode_step(oracle, B, H, N, Hg, io, defer, modrelu):
    run_steps(oracle, B, H, N, Hg, io, defer, modrelu)


@pytest.mark.parametrize("B,H,N,Hg,io,defer,per_wg", [
    (3, 32, 5120, 1, "bf16", 0, 2), (3, 32, 4096, 32, "f32", 0, 2),     # eager: two, and one in the last workgroup
    (3, 32, 5120, 32, "bf16", 5, 2), (5, 32, 5120, 1, "f32", 3, 3),     # pending tokens: two and one, three and two
    (7, 32, 4096, 32, "f32", 4, 4), (3, 32, 8192, 1, "f32", 4, 3)])     # four and three; all three in one workgroup
def test_decode_step_of_several_sequences_per_workgroup(oracle, B, H, N, Hg, io, defer, per_wg):
    n = min(4 if defer else 2, B)
    while n > 1 and N // 256 * H * -(-B // n) < 1024:                   # the launch's rule (csrc/decode.hip)
        n = (n + 1) // 2
    assert -(-B // -(-B // n)) == per_wg
    run_steps(oracle, B, H, N, Hg, io, defer, steps=4)


@pytest.mark.parametrize("Hg,io", [(32, "f32"), (1, "bf16")])
def test_decode_step_of_all_sequences_in_one_workgroup(oracle, Hg, io):
    """Updating steps of two sequences whose rows one workgroup takes: the rows are requested one by one, also across the sequences."""
    run_steps(oracle, 2, 32, 8192, Hg, io, 0, steps=3)


@pytest.mark.parametrize("B,H,N,Hg,io,defer,modrelu,d_g,taps,shift", [
    (2, 3, 768, 3, "f32", 0, True, 48, 0, 0), (2, 3, 768, 1, "bf16", 3, False, 48, 0, 0),       # another width
    (1, 2, 512, 2, "bf16", 0, True, 64, 2, 0), (2, 2, 1280, 1, "f32", 4, True, 64, 3, 0),       # Toeplitz taps
    (2, 2, 256, 2, "f32", 0, True, 64, 0, 1), (1, 3, 512, 3, "f32", 3, True, 64, 0, 2),         # W2 off a 16-byte boundary
    (1, 2, 1792, 2, "f32", 32, True, 33, 1, 0)])                                                # all at once, never full
def test_decode_step_of_other_gates(oracle, B, H, N, Hg, io, defer, modrelu, d_g, taps, shift):
    run_steps(oracle, B, H, N, Hg, io, defer, modrelu, d_g=d_g, taps=taps, shift=shift)
