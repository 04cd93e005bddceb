"""GPU parity of the window transform and the full-window readout over the plans whose column kernels hold a plane with
its Hermitian partner (256- and 1024-point columns), and one length above them that keeps the separate kernels."""
import numpy as np
import pytest
import torch

from gpu_util import TOL, from_device, rel_l2, to_device
from paper_2502_18394_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B,H,io", [
    (256, 1, 1, "f32"),        # one plane, its own partner; fewer units than the 8 the grid is padded to
    (512, 2, 3, "bf16"), (768, 1, 3, "f32"), (1280, 1, 2, "bf16"),      # self-paired planes with and without a second one
    (8192, 1, 2, "f32"),       # the most planes of 256-point columns
    (12288, 1, 1, "bf16"), (28672, 1, 1, "f32"), (32768, 1, 2, "bf16"),  # 1024-point columns
    (40960, 1, 1, "f32"),      # 4096-point columns
])
def test_window_transform_and_readout(oracle, N, B, H, io):
    from paper_2502_18394_amd import binding
    d, T = 64, N - N // 5
    print(f"case N={N} B={B} H={H} io={io}", flush=True)
    v, vs = synth.tokens(1300 + N, (B, T, H, d), io)
    c = binding.PrefixCache(B, H, d, N)
    c.update(to_device(vs, io), to_device(vs, io))
    rows = np.zeros((B, H, N, d))
    rows[:, :, :T] = v.astype(np.float64).transpose(0, 2, 1, 3)
    spec = np.fft.rfft(rows, axis=2)
    got = c.prefix_fft.cpu().numpy()
    assert rel_l2(got, spec.reshape(got.shape)) <= 1e-6        # fp32 transform: 2e-7 measured
    rng = np.random.default_rng(N)
    g = (rng.standard_normal((B, H, N // 2 + 1)) + 1j * rng.standard_normal((B, H, N // 2 + 1))).astype(np.complex64)
    out = c.readout(torch.from_numpy(g).cuda(), binding.READ_WINDOW, dtype=torch.bfloat16 if io == "bf16" else torch.float32)
    y = g[..., None].astype(np.complex128) * spec
    y[:, :, [0, -1]] = y[:, :, [0, -1]].real
    want = np.fft.irfft(y, n=N, axis=2)[:, :, N - T:].transpose(0, 2, 1, 3)
    assert rel_l2(from_device(out), want) <= TOL[io]


@pytest.mark.parametrize("N,heads", [(4096, (17, 18, 32, 33)), (2048, (40, 70)), (16384, (4, 5, 14))])
def test_readout_at_the_sizes_where_its_stores_change(N, heads):
    """Columns through the L2 below 18 MB and above 32 MB, plain between (256-point columns from 2560 slots on, else always through), and the window's
    row transforms on both sides of 16 and 56 MB: the same bits as for two heads."""
    from paper_2502_18394_amd import binding
    gen = torch.Generator(device="cuda").manual_seed(N)
    rows = [torch.randn((1, N + N // 8, max(heads), 64), generator=gen, device="cuda") for _ in range(2)]
    g = torch.view_as_complex(torch.randn((1, max(heads), N // 2 + 1, 2), generator=gen, device="cuda"))

    def window(H):
        c = binding.PrefixCache(1, H, 64, N)
        for part in (slice(0, N), slice(N, None)):                  # a prompt, then so many tokens that the window is transformed anew
            c.update(*(r[:, part, :H].contiguous() for r in rows))
        return c.prefix_fft, c.readout(g[:, :H].contiguous(), binding.READ_WINDOW)

    spec, out = window(2)
    for H in heads:
        print(f"case N={N} H={H}", flush=True)
        got_spec, got = window(H)
        assert torch.equal(got_spec[:, :2], spec) and torch.equal(got[:, :, :2], out)
