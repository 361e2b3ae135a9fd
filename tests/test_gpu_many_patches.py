"""A level over so many patches that the softmax weights of a chunk of eight channels span more than 2^32 bytes, on the GPU."""
import pytest
import torch

import paper_2506_21411_amd as dchag

from .test_gpu_products import say

pytestmark = pytest.mark.gpu


def test_softmax_weights_of_a_chunk_beyond_32_bit_offsets():
    """One member a group, 8 heads, D 256: the weights of the chunk's channel 7 (padding, zero) begin 56 pitches of 4 bytes behind those of
    channel 0, past 2^32 from 19,173,962 patches on.  65,536 tokens repeated 295 times give 295 times the output of the 65,536."""
    base, times, D, heads = 65536, 295, 256, 8
    assert 7 * heads * base * times * 4 > 2 ** 32
    gen = torch.Generator(device="cuda").manual_seed(5)
    r = lambda *s, std=1.0: (torch.randn(*s, generator=gen, device="cuda") * std).to(torch.bfloat16)
    lv = dchag.LevelWeights(1, r(1, D), *(r(1, D, D, std=D ** -0.5) for _ in range(4)), *(r(1, D, std=D ** -0.5) for _ in range(4)))
    few = r(1, 1, base, D)
    say("level of 65,536 patches")
    want = dchag.dchag_aggregate_level(few, lv, heads)
    say(f"level of {base * times} patches")
    got = dchag.dchag_aggregate_level(few.repeat(1, 1, times, 1), lv, heads)
    ref = (few[0, 0].float() @ lv.Wv[0].float().T + lv.bv[0].float()) @ lv.Wo[0].float().T + lv.bo[0].float()
    assert (want[0, 0].float() - ref).norm() < 2e-2 * ref.norm()
    assert torch.equal(got.view(times, base, D), want.view(1, base, D).expand(times, -1, -1))
