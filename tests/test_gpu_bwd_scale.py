"""The gradient scale of the backward: the largest |dO| of each (batch, K/V
head) is found wherever it sits, also where the partial maxima are capped (more
than 256 chunks of 16384 elements per K/V head) and chunks get longer."""
import pytest
import torch

from gpu_util import announce, device_inputs, need_gpu
from paper_2609_13612_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,Hkv,S,D", [(1, 1, 1, 1, 64), (2, 2, 1, 77, 64), (2, 4, 2, 129, 128),
                                         (1, 16, 1, 2305, 128), (1, 8, 1, 9000, 64)])
@pytest.mark.parametrize("where", ["first", "last"])
def test_largest_element_is_found(B, H, Hkv, S, D, where):
    """One dO element of 2^20 (fp16 holds up to 65504): a scale that missed it would overflow the fp16 copy of dO to
    inf.  The gradients are finite, and those of dO 2^-30 are exactly 2^-30 times them."""
    need_gpu()
    announce(f"bwd scale {B} {H}/{Hkv} {S} {D} {where}")
    _, d = device_inputs(B, H, Hkv, S, D, seed=S, with_do=True)
    q, k, v, do = (d[n] for n in ("q", "k", "v", "do"))
    flat = do.view(B, Hkv, -1)
    flat[0, -1, 0 if where == "first" else -1] = 2.0 ** 20
    kw = dict(rope="neox", mask="causal")
    o, lse = api.attnfuse_fwd(q, k, v, **kw)
    big = api.attnfuse_bwd(q, k, v, o, do, lse, **kw)
    small = api.attnfuse_bwd(q, k, v, o, (do.float() * 2.0 ** -30).bfloat16(), lse, **kw)
    for a, b in zip(big, small):
        assert torch.isfinite(a).all()
        assert torch.equal(a.float() * 2.0 ** -30, b.float())
