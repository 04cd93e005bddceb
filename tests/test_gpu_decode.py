"""GPU parity of the two-launch decode step at the edges of its tiling: one chunk of 128 bins and many, window lengths
with an odd factor, sequence counts around the two and four a workgroup takes, shared and per-head gate weights."""
import numpy as np
import pytest

from gpu_util import TOL, f64, from_device, rel_l2, to_device
from paper_2502_18394_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,N,Hg,io,defer,modrelu", [
    (1, 1, 256, 1, "f32", 0, True), (5, 3, 256, 3, "bf16", 0, True), (3, 2, 768, 2, "f32", 0, False),
    (9, 1, 1280, 1, "f32", 0, True), (4, 32, 2048, 1, "bf16", 0, True),
    (1, 1, 256, 1, "f32", 4, True), (5, 3, 512, 3, "bf16", 3, True), (2, 3, 1792, 1, "f32", 32, False),
    (9, 32, 1024, 32, "f32", 2, True)])
def test_decode_step(oracle, B, H, N, Hg, io, defer, modrelu):
    from paper_2502_18394_amd import binding
    d, steps, T0 = 64, 7, N - 3                       # the window fills up and wraps while the steps run
    print(f"case B={B} H={H} N={N} Hg={Hg} io={io} defer={defer} modrelu={modrelu}", flush=True)
    c, oc = binding.PrefixCache(B, H, d, N, defer=defer), oracle.PrefixCache(B, H, d, N)
    v, vs = synth.tokens(800 + N, (B, T0 + steps, H, d), io)
    q, qs = synth.tokens(801 + N, (B, T0 + steps, H, d), io)
    p = synth.gate_params(802 + B, Hg, d, N, modrelu=modrelu)
    P = binding.GateParams(p)
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
