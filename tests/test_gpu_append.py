"""GPU parity of appends of several tokens around the 64 that one sweep over the cache takes, and on rings shorter than
such a batch (memory rows in front), where a batch evicts its own tokens."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import rel_l2, to_device
from paper_2502_18394_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N_mem,N_max,T0,appends,io", [
    (0, 256, 100, (63, 64, 65), "f32"), (0, 512, 510, (127, 128, 129), "bf16"), (0, 256, 0, (1, 2, 66), "f32"),
    (240, 16, 10, (15, 16, 17, 40), "f32"), (193, 63, 63, (64, 130), "bf16"),
    (255, 1, 1, (2, 64, 65), "f32"), (253, 3, 2, (2, 3, 4, 63), "bf16"), (504, 8, 3, (64, 100), "f32")])
def test_append(oracle, N_mem, N_max, T0, appends, io):
    from paper_2502_18394_amd import binding
    B, H, d = 2, 3, 64
    print(f"case N_mem={N_mem} N_max={N_max} T0={T0} appends={appends} io={io}", flush=True)
    c, oc = binding.PrefixCache(B, H, d, N_max, N_mem=N_mem), oracle.MemoryPrefixCache(B, H, d, N_mem, N_max)
    M = np.random.default_rng(900).standard_normal((B, H, N_mem, d)).astype(np.float32)
    if N_mem:
        c.set_memory(torch.from_numpy(M).cuda())
    v, vs = synth.tokens(901, (B, max(T0, 1), H, d), io)
    q, qs = synth.tokens(902, (B, max(T0, 1), H, d), io)
    if T0:
        c.update(to_device(vs, io), to_device(qs, io))
        oc.prefill(M.astype(np.float64), v.astype(np.float64), q.astype(np.float64))
    else:
        oc.prefill(M.astype(np.float64))
    for j, T in enumerate(appends):
        v, vs = synth.tokens(903 + 2 * j, (B, T, H, d), io)
        q, qs = synth.tokens(904 + 2 * j, (B, T, H, d), io)
        c.update(to_device(vs, io), to_device(qs, io))
        for i in range(T):
            oc.update(v[:, i:i + 1].astype(np.float64), q[:, i:i + 1].astype(np.float64))
        assert c.t == oc.t
        assert rel_l2(c.prefix_fft.cpu().numpy(), oc.spec) <= 1e-5
        assert rel_l2(c.sum_q.cpu().numpy(), oc.sum_q) <= 1e-12
        assert np.array_equal(c.v_buf.cpu().numpy(), oc.v_buf.astype(np.float32))
        assert np.array_equal(c.q_buf.cpu().numpy()[:, :, N_mem:], oc.q_buf.astype(np.float32)[:, :, -N_max:])


@pytest.mark.parametrize("N_mem,N,T0", [(0, 256, 250), (0, 768, 3), (0, 1792, 1785), (16, 256, 200), (7, 256, 1)])
def test_append_groups_of_16_tokens(oracle, N_mem, N, T0):
    """Batches at the edges of the groups of 16 tokens that a sweep folds, in windows with and without an odd factor, around
    the wrap of the ring; rings behind memory rows take the other sweep where a batch wraps.  1e-6: fp32 sums of at most 64
    terms per bin and append, 1.4e-7 measured."""
    from paper_2502_18394_amd import binding
    B, H, d = 2, 2, 64
    print(f"case N_mem={N_mem} N={N} T0={T0}", flush=True)
    c, oc = binding.PrefixCache(B, H, d, N - N_mem, N_mem=N_mem), oracle.MemoryPrefixCache(B, H, d, N_mem, N - N_mem)
    M = np.random.default_rng(950).standard_normal((B, H, N_mem, d)).astype(np.float32)
    if N_mem:
        c.set_memory(torch.from_numpy(M).cuda())
    x, _ = synth.tokens(951, (B, T0, H, d))
    c.update(to_device(x, "f32"), to_device(x, "f32"))
    oc.prefill(M.astype(np.float64), x.astype(np.float64), x.astype(np.float64))
    for T in (2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 64):
        x, _ = synth.tokens(952 + T, (B, T, H, d))
        c.update(to_device(x, "f32"), to_device(x, "f32"))
        for i in range(T):
            oc.update(x[:, i:i + 1].astype(np.float64), x[:, i:i + 1].astype(np.float64))
        assert rel_l2(c.prefix_fft.cpu().numpy(), oc.spec) <= 1e-6, T


@pytest.mark.parametrize("N_max", [1, 8, 16, 63, 256])
@pytest.mark.parametrize("T,batches", [(32, 1), (64, 1), (65, 2)])
def test_append_takes_64_tokens_per_sweep_on_any_ring(N_max, T, batches):
    """A sweep moves the whole cache, so the number of them must not grow as the ring gets shorter: an append is two
    launches (ring buffers, sweep) per 64 tokens, counted as the nodes of a captured call."""
    from paper_2502_18394_amd import binding
    n = 256
    print(f"case N_max={N_max} T={T}", flush=True)
    c = binding.PrefixCache(1, 1, 64, N_max, N_mem=n - N_max)
    x = torch.ones((1, T, 1, 64), device="cuda")
    c.update(x[:, :1].contiguous(), x[:, :1].contiguous())          # set-up happens here, not under capture
    c.update(x, x)
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        c.update(x, x)
    nodes = ctypes.c_size_t(0)
    assert binding.lib().hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
    assert nodes.value == 2 * batches


def off_by_one(t):
    """The same values one element further on than an allocation starts."""
    flat = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")
    flat[1:] = t.reshape(-1)
    return flat[1:].view(t.shape)


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("T", [1, 2, 65, 159])
def test_rows_and_sums_need_no_more_than_the_alignment_of_an_element(T, io):
    """Appended rows are read in pairs and pooled sums two at a time: the state and the gate are the same, bit for bit,
    wherever the elements lie (the cache's own arrays are on 16-byte boundaries)."""
    from paper_2502_18394_amd import binding
    B, H, N = 2, 3, 256
    print(f"case T={T} io={io}", flush=True)
    _, vs = synth.tokens(910, (B, 2 + T, H, 64), io)
    _, qs = synth.tokens(911, (B, 2 + T, H, 64), io)
    P = binding.GateParams(synth.gate_params(912, H, 64, N))
    states = []
    for place in (lambda t: t, off_by_one):
        c = binding.PrefixCache(B, H, 64, N)
        cut = lambda a, i, j: place(to_device(np.ascontiguousarray(a[:, i:j]), io))
        for i, j in ((1, 2), (2, 2 + T)):                           # an empty cache would be pre-filled
            c.update(cut(vs, i, j), cut(qs, i, j))
        out = c.step(cut(vs, 0, 1), cut(qs, 0, 1), P)
        g = binding.gate(place(c.sum_q), P, 1.0 / N, pooled=True)
        states.append([c.prefix_fft, c.v_buf, c.q_buf, c.sum_q, out, g])
    for a, b in zip(*states):
        assert torch.equal(torch.view_as_real(a) if a.is_complex() else a, torch.view_as_real(b) if b.is_complex() else b)


@pytest.mark.parametrize("N,T", [(2560, 1023), (2560, 1024), (2560, 2560), (3072, 2561)])
def test_prompts_around_the_sizes_whose_query_rows_stay_cached(N, T):
    """fp32 prompts of 64 and 160 MiB of query rows, and one token to the other side of either: ring buffers bit for bit, sums of
    fp64 terms in another order, and the spectra of two heads in 64 bits (bound as in test_append)."""
    from paper_2502_18394_amd import binding
    B, H = 8, 32
    print(f"case N={N} T={T}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    v, q = (torch.randn((B, T, H, 64), generator=gen, device="cuda") for _ in range(2))
    c = binding.PrefixCache(B, H, 64, N)
    c.update(v, q)
    assert torch.equal(c.v_buf[:, :, :T], v.transpose(1, 2)) and torch.equal(c.q_buf[:, :, :T], q.transpose(1, 2))
    assert not bool(c.v_buf[:, :, T:].any()) and not bool(c.q_buf[:, :, T:].any())
    assert rel_l2(c.sum_q.cpu().numpy(), q.double().sum(1).cpu().numpy()) <= 1e-12
    for b, h in ((0, 0), (B - 1, H - 1)):
        assert rel_l2(c.prefix_fft[b, h].cpu().numpy(), np.fft.rfft(c.v_buf[b, h].cpu().numpy().astype(np.float64), axis=0)) <= 1e-5
