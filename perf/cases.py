"""The work that users of the library have it do, as cases that can be timed and compared.

Every case goes through ``paper_2502_18394_amd.binding``, the public entry points, with the buffers a serving
program keeps between calls (gate weights, workspaces, output tensors, the Prefix-FFT cache).  d = 64 channels per
head and a gate MLP of width 64 throughout, as in every configuration of ``synth``.

Kinds of work
  step     gate from the query rows, then the mixer: one mixing layer whose V and Q are already projected
  mix      the mixer alone with a gate that is given
  layer    the whole layer from its input X (projection, pooled query, gate, mixer), optionally with the wavelet
           refinement over all the levels its length has
  decode   single-token steps of a cache that is filled to the brim, T tokens a pass; defer > 0 leaves updates pending
  prefill  a new prompt into a cache that held another sequence: reset, then all tokens at once
  turn     T tokens appended to a running sequence, its gate, and the readout of the whole window
"""
import math

import torch

from paper_2502_18394_amd import binding, synth

D, DG = 64, synth.D_GATE


def listed():
    return [
        # one head on its own: the smallest call there is, launches and latency only
        dict(name="one_head_1k", kind="step", B=1, H=1, L=1024, io="f32", shared=False),
        # the Llama head shape at the ends and the middle of its length sweep: short prompts ...
        dict(name="llama_512", kind="step", B=1, H=32, L=512, io="bf16", shared=False),
        dict(name="llama_4k", kind="step", B=1, H=32, L=4096, io="bf16", shared=False),
        # ... the ordinary context length ...
        dict(name="llama_8k", kind="step", B=1, H=32, L=8192, io="bf16", shared=False),
        # ... and the longest one
        dict(name="llama_128k", kind="step", B=1, H=32, L=131072, io="bf16", shared=False),
        # a whole layer with the refinement, a long document of a length with an odd factor
        dict(name="layer_24k", kind="layer", B=1, H=32, L=24576, io="bf16", shared=False, refine=True),
        # image classification: 14 x 14 patches, a large batch of short sequences
        dict(name="vit_196", kind="step", B=256, H=12, L=196, io="f32", shared=False),
        # the same patches with a class token: a length no plan divides
        dict(name="vit_197", kind="mix", B=64, H=12, L=197, io="f32"),
        # generation for a batch of long sequences, every step updating the cache
        dict(name="decode_32k", kind="decode", B=8, H=32, N=32768, io="f32", T=1, defer=0, shared=False),
        # generation for one user at an ordinary context length, updates deferred, 16 tokens
        dict(name="decode_8k", kind="decode", B=1, H=32, N=8192, io="bf16", T=16, defer=16, shared=False),
        # a batch of new prompts, as long as documents happen to be, into caches that served others before
        dict(name="prefill_32k", kind="prefill", B=8, H=32, N=32768, io="bf16", T=20011),
        # a chat turn: a few dozen tokens in, the whole window out
        dict(name="turn_8k", kind="turn", B=4, H=32, N=8192, io="bf16", T=57, shared=False),
    ]


def _plan_lengths():
    return sorted({n1 * m * (1 << a) for n1 in (256, 4096) for m in (1, 3, 5, 7) for a in range(6)
                   if m * (1 << a) <= 32})


def _smooth(n):
    for p in (2, 3, 5, 7):
        while n % p == 0:
            n //= p
    return n == 1


PLAN = _plan_lengths()                                            # 256 .. 131072: lengths with a four-step plan
SMOOTH = [n for n in range(48, 2049) if _smooth(n)]               # short lengths with prime factors up to 7
MAX_TOKENS = 32 * 131072                                          # B * H * L of the longest listed layer


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _nearest(values, x):
    return min(values, key=lambda v: abs(math.log(v / x)))


def _batch(rng, H, L, most):
    """Sequences per call: any number that stays within `most` head rows."""
    return max(1, int(_log_uniform(rng, 1, max(1.001, min(256, most / (H * L))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "mix", "layer", "decode", "decode", "prefill", "turn"])
    io = rng.choice(["bf16", "f32"])
    H = rng.choice([1, 4, 8, 12, 16, 20, 32, 32])
    shared = rng.random() < 0.25
    most = MAX_TOKENS if io == "bf16" else MAX_TOKENS // 2
    if kind in ("step", "mix", "layer"):
        form = rng.choice(["plan", "plan", "smooth", "any"])
        if form == "plan":
            L = _nearest(PLAN, _log_uniform(rng, 256, 131072))
        elif form == "smooth":
            L = _nearest(SMOOTH, _log_uniform(rng, 48, 2048))
        else:
            L = int(_log_uniform(rng, 100, 65536))
            most //= 8                                            # padded to at least twice the length
        c = dict(kind=kind, B=_batch(rng, H, L, most), H=H, L=L, io=io)
        if kind != "mix":
            c["shared"] = shared
        if kind == "layer":
            c["refine"] = rng.random() < 0.5
        return c
    N = _nearest(PLAN, _log_uniform(rng, 512, 65536))
    most = 8 * 32 * 32768
    if kind == "decode":
        B = min(16, _batch(rng, H, N, most))
        T = max(1, int(_log_uniform(rng, 1, max(1.001, min(32.0, most / (B * H * N))))))
        return dict(kind=kind, B=B, H=H, N=N, io=io, T=T, defer=rng.choice([0, 0, 8, 16, 32]), shared=shared)
    B = min(16, _batch(rng, H, N, most if kind == "prefill" else most // 4))
    if kind == "prefill":
        return dict(kind=kind, B=B, H=H, N=N, io=io, T=max(2, int(_log_uniform(rng, N / 16, N))))
    return dict(kind=kind, B=B, H=H, N=N, io=io, T=max(2, int(_log_uniform(rng, 2, min(2048, N)))), shared=shared)


# ------------------------------------------------------------------------------------------ inputs
class _Draw:
    """Normal tensors on the GPU from one seed."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def __call__(self, *shape, std=1.0, dtype=torch.float32):
        return (torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.float32) * std).to(dtype)


def _gate_params(nrm, Hg, n):
    F = n // 2 + 1
    s = 0.02
    return binding.GateParams(dict(
        n_fft=n, ln_eps=synth.LN_EPS, ln_gamma=1.0 + nrm(Hg, D, std=s), ln_beta=nrm(Hg, D, std=s),
        W1=nrm(Hg, D, DG, std=s), b1=nrm(Hg, DG, std=s), W2=nrm(Hg, DG, 2 * F, std=s), b2=nrm(Hg, 2 * F, std=s),
        modrelu_bias=nrm(Hg, F, std=s)))


def _wrm_params(nrm, Hg, levels):
    s, nout = 0.02, (levels + 1) * D
    return binding.WrmParams(dict(
        levels=levels, ln_eps=synth.LN_EPS, ln_gamma=1.0 + nrm(Hg, D, std=s), ln_beta=nrm(Hg, D, std=s),
        W1=nrm(Hg, D, DG, std=s), b1=nrm(Hg, DG, std=s), W2=nrm(Hg, DG, nout, std=0.5), b2=nrm(Hg, nout, std=0.5)))


def _buffer(nbytes):
    return torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")


def _levels(case):
    return synth.max_wavelet_levels(case["L"]) if case.get("refine") else 0


def prepare(case, seed):
    nrm = _Draw(seed)
    kind, B, H = case["kind"], case["B"], case["H"]
    dtype = torch.bfloat16 if case["io"] == "bf16" else torch.float32
    s = dict(kind=kind, case=case)
    Hg = 1 if case.get("shared") else H
    if kind in ("step", "mix", "layer"):
        L = case["L"]
        s["x"] = nrm(B, L, H, D, dtype=dtype)
        s["out"] = torch.empty_like(s["x"])
        binding.prepare(L, D)
        if kind in ("step", "mix"):
            s["ws"] = _buffer(binding.mix_workspace_bytes(B, L, H, D, binding.BF16 if case["io"] == "bf16" else binding.F32))
        if kind == "mix":
            s["g"] = torch.view_as_complex(nrm(B, H, L // 2 + 1, 2))
        else:
            s["P"] = _gate_params(nrm, Hg, L)
        if kind == "step":
            s["q"] = nrm(B, L, H, D, dtype=dtype)
            s["g"] = torch.empty((B, H, L // 2 + 1), dtype=torch.complex64, device="cuda")
            s["ws_gate"] = _buffer(binding.gate_workspace_bytes(B, L, H, s["P"]))
        if kind == "layer":
            s["Wq"], s["Wv"] = nrm(Hg, D, D, std=0.125), nrm(Hg, D, D, std=0.125)
            s["W"] = _wrm_params(nrm, Hg, _levels(case)) if case["refine"] else None
            s["ws"] = None                                   # allocated per call by the binding, as for any torch op
        return s
    N, T = case["N"], case["T"]
    s["cache"] = cache = binding.PrefixCache(B, H, D, N, defer=case.get("defer", 0))
    if kind != "prefill":
        s["P"] = _gate_params(nrm, Hg, N)
        # a running sequence: the window is full, so every new token evicts one
        cache.update(nrm(B, N, H, D, dtype=dtype), nrm(B, N, H, D, dtype=dtype))
    if kind == "decode":
        s["v"] = [nrm(B, 1, H, D, dtype=dtype) for _ in range(T)]
        s["q"] = [nrm(B, 1, H, D, dtype=dtype) for _ in range(T)]
        s["out"] = [torch.empty((B, 1, H, D), dtype=dtype, device="cuda") for _ in range(T)]
    else:
        s["v"], s["q"] = nrm(B, T, H, D, dtype=dtype), nrm(B, T, H, D, dtype=dtype)
    s["dtype"] = dtype
    return s


# ------------------------------------------------------------------------------------------ one pass
def _cache_state(cache):
    return [cache.prefix_fft, cache.v_buf, cache.q_buf, cache.sum_q]


def run(s):
    kind = s["kind"]
    if kind == "step":
        binding.gate(s["q"], s["P"], 1.0 / s["q"].shape[1], g_out=s["g"], ws=s["ws_gate"])
        binding.mix_forward(s["x"], s["g"], out=s["out"], ws=s["ws"])
        return [s["out"], s["g"]]
    if kind == "mix":
        return binding.mix_forward(s["x"], s["g"], out=s["out"], ws=s["ws"])
    if kind == "layer":
        return binding.layer_forward(s["x"], s["Wq"], s["Wv"], s["P"], W=s["W"], out=s["out"], ws=s["ws"])
    cache = s["cache"]
    if kind == "decode":
        for v, q, out in zip(s["v"], s["q"], s["out"]):
            cache.step(v, q, s["P"], out=out)
        return s["out"] + _cache_state(cache)
    if kind == "prefill":
        cache.reset()
        cache.update(s["v"], s["q"])
        return _cache_state(cache)
    cache.update(s["v"], s["q"])
    g = binding.gate(cache.sum_q, s["P"], 1.0 / cache.N, pooled=True, phase_pos=cache.t)
    return [cache.readout(g, binding.READ_WINDOW, dtype=s["dtype"])] + _cache_state(cache)


# ------------------------------------------------------------------------------------------ what it costs at least
def _gate_work(case, n, pooled):
    """Weights, gate and the query side of one gate evaluation."""
    B, H, F = case["B"], case["H"], n // 2 + 1
    Hg = 1 if case.get("shared") else H
    e = 2 if case["io"] == "bf16" else 4
    weights = Hg * (4 * (D * DG + DG + 2 * D + DG * 2 * F + 2 * F + F))
    rows = B * H * D * 8 if pooled else B * n * H * D * e
    return weights + rows + 8 * B * H * F, 2 * B * H * DG * (D + 2 * F) + (0 if pooled else B * n * H * D)


def work(case):
    kind, B, H = case["kind"], case["B"], case["H"]
    e = 2 if case["io"] == "bf16" else 4
    n = case.get("L") or case["N"]
    F = n // 2 + 1
    row = B * H * D * e                                       # one token of every sequence and head
    fft = 2.5 * n * math.log2(n) * B * H * D                  # one real transform of every channel
    gate = 8 * B * H * F
    if kind == "mix":
        return {"bytes": 2 * n * row + gate, "flops": 2 * fft + 6 * B * H * F * D}
    if kind == "step":
        b, f = _gate_work(case, n, False)
        return {"bytes": 2 * n * row + gate + b, "flops": 2 * fft + 6 * B * H * F * D + f}
    if kind == "layer":                                       # the gate stays inside the call; X is read once
        b, f = _gate_work(case, n, True)
        levels = _levels(case)
        refine = 4 * H * (levels + 1) * D * DG if case["refine"] else 0
        return {"bytes": 2 * n * row + b - gate + refine,
                "flops": 2 * fft + 6 * B * H * F * D + f + 2 * n * B * H * D * D + (6 * n * B * H * D if levels else 0)}
    state = 8 * B * H * F * D                                 # the half spectra of every channel
    ring = 4 * B * H * D                                      # one row of a ring buffer
    T = case["T"]
    if kind == "decode":
        b, f = _gate_work(case, n, True)
        cap = case["defer"]
        # a deferred step only reads the half spectra; they are written once every `cap` tokens
        traffic = state * (2 * T if not cap else T * (1 + 1 / cap))
        return {"bytes": traffic + T * (b - gate + 3 * row + 4 * ring), "flops": T * (8 * B * H * F * D * 2 + f)}
    if kind == "prefill":                                     # prompt in, spectra and both ring buffers out
        return {"bytes": 2 * T * row + state + 2 * n * ring, "flops": fft}
    b, f = _gate_work(case, n, True)
    return {"bytes": 2 * T * row + 4 * T * ring + 2 * state + b - gate + n * row,
            "flops": min(T * 8 * B * H * F * D, fft) + f + fft + 6 * B * H * F * D}


def tolerance(case):
    # About four times the distance to the same path in 64 bits.  fp32 rows: 1.3e-7 (gate, half spectra) to 3.0e-7
    # (a window's spectra after many appended tokens); bf16 rows: 1.66e-3, the rounding of the stored rows.
    return {"rel": 1.2e-6} if case["io"] == "f32" else {"rel": 7e-3}
