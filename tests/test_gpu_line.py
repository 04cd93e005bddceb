"""GPU parity of the whole-column mixer (bf16 rows, L = 8192 and 16384): head counts that are and are not multiples of
the eight XCDs, workgroups with no line, one, several and unequal shares of them, heads taken in several groups."""
import numpy as np
import pytest
import torch

from gpu_util import TOL, assert_close_elementwise, from_device, rel_l2, to_device
from paper_2502_18394_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,L,H,mb", [(1, 8192, 1, 0), (3, 8192, 3, 0), (1, 8192, 32, 0), (2, 8192, 9, 8),
                                      (1, 16384, 1, 0), (2, 16384, 5, 0), (1, 16384, 16, 16),
                                      (1, 8192, 20, 0), (5, 8192, 13, 0),       # shares of 1 or 2 lines, of 4 or 5
                                      (1, 16384, 20, 0), (3, 16384, 11, 0)])    # of 2 or 3, of 4 or 5
def test_whole_column_mixer(oracle, options, B, L, H, mb):
    from paper_2502_18394_amd import binding
    print(f"case B={B} L={L} H={H} mb={mb}", flush=True)
    if mb:
        options(binding.OPT_SCRATCH_MB, mb)
    v, vs = synth.tokens(1000 + L + H, (B, L, H, 64), "bf16")
    g = synth.random_gate(1001 + H, B, H, L)
    got = from_device(binding.mix_forward(to_device(vs, "bf16"), torch.from_numpy(g).cuda()))
    want = oracle.mix_forward(v.astype(np.float64), g.astype(np.complex128))
    assert rel_l2(got, want) <= TOL["bf16"]
    assert_close_elementwise(got, want, "bf16", L)


@pytest.mark.parametrize("shift_in,shift_out", [(2, 0), (0, 2), (6, 2)])
def test_tensors_off_a_16_byte_boundary_give_the_same_rows(oracle, shift_in, shift_out):
    """Channel pairs are 4 bytes and that is all a caller owes: same result bit for bit, and not a byte outside the output."""
    from paper_2502_18394_amd import binding
    B, L, H = 1, 8192, 2
    print(f"case shifts {shift_in} {shift_out} elements", flush=True)
    v, vs = synth.tokens(77, (B, L, H, 64), "bf16")
    g = synth.random_gate(78, B, H, L)
    n = B * L * H * 64
    src = torch.zeros(n + 16, dtype=torch.bfloat16, device="cuda")
    src[shift_in:shift_in + n] = to_device(vs, "bf16").reshape(-1)
    dst = torch.full((n + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
    got = from_device(binding.mix_forward(src[shift_in:shift_in + n].view(B, L, H, 64), torch.from_numpy(g).cuda(),
                                          out=dst[shift_out:shift_out + n].view(B, L, H, 64)))
    want = oracle.mix_forward(v.astype(np.float64), g.astype(np.complex128))
    assert rel_l2(got, want) <= TOL["bf16"]
    assert_close_elementwise(got, want, "bf16", L)
    assert np.array_equal(got, from_device(binding.mix_forward(to_device(vs, "bf16"), torch.from_numpy(g).cuda())))
    rest = torch.cat([dst[:shift_out], dst[shift_out + n:]]).float()
    assert bool((rest == 7.0).all())
