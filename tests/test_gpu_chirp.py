"""GPU parity of the one-launch gate of the padded convolution (lengths without a plan, padded length 256 .. 2048): the
shortest and the longest length of every padded length, head counts that do and do not fill a workgroup."""
import numpy as np
import pytest
import torch

from gpu_util import TOL, assert_close_elementwise, rel_l2
from paper_2502_18394_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [11, 127, 131, 254, 257, 383, 386, 509, 514, 631, 641, 761, 769, 894, 898, 1022])
@pytest.mark.parametrize("B,H", [(1, 1), (3, 3)])
def test_short_padded_lengths(oracle, B, H, L):
    from paper_2502_18394_amd import binding
    print(f"case B={B} L={L} H={H}", flush=True)
    v, _ = synth.tokens(1100 + L, (B, L, H, 64), "f32")
    g = synth.random_gate(1101 + L, B, H, L)
    got = binding.mix_forward(torch.from_numpy(v).cuda(), torch.from_numpy(g).cuda()).cpu().numpy()
    want = oracle.mix_forward(v.astype(np.float64), g.astype(np.complex128))
    assert rel_l2(got, want) <= TOL["f32"]
    assert_close_elementwise(got, want, "f32", 16 * L)         # padded transform, and the gate came through two more
