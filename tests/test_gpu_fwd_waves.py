"""The dense forward's four-wave and eight-wave workgroups give the same bits: a
batch of a size that takes one form against its heads in calls of the other."""
import pytest
import torch

from gpu_util import announce, device_inputs, need_gpu
from paper_2609_13612_amd import _lib, api

pytestmark = pytest.mark.gpu
MASK = {"none": 0, "causal": 1, "sliding_window": 2}


@pytest.mark.parametrize("B,H,G,S,D,rope,mask,window,bias,parts", [
    (2, 14, 1, 2050, 64, "none", "none", None, None, 2), (2, 14, 1, 2111, 64, "none", "none", None, "key", 2),
    (1, 16, 4, 2400, 128, "none", "none", None, "key", 2), (2, 32, 4, 2048, 128, "none", "causal", None, "key", 4),
    (6, 16, 8, 400, 128, "neox", "none", None, None, 2), (3, 12, 1, 1000, 64, "interleaved", "none", None, None, 3),
    (12, 8, 4, 500, 128, "neox", "causal", None, None, 2), (3, 32, 4, 512, 128, "neox", "sliding_window", 100, None, 4)])
def test_same_bits(monkeypatch, B, H, G, S, D, rope, mask, window, bias, parts):
    need_gpu()
    announce(f"fwd waves {B} {H}/{H // G} {S} {D} {rope} {mask} {bias}")
    _, d = device_inputs(B, H, H // G, S, D, seed=S)
    q, k, v = d["q"], d["k"], d["v"]
    bt = torch.randn(B, 1, 1, S, device="cuda") if bias else None
    monkeypatch.setattr(api, "_native", None)
    monkeypatch.setattr(api, "_fwd_scratch", lambda *a, **kw: None)   # rotated in the loop

    def call(q, k, v, b):
        return api.attnfuse_fwd_bias_norm(q.contiguous(), k.contiguous(), v.contiguous(), bias=b, rope=rope, mask=mask,
                                          window=window)

    def waves(b, h):
        return _lib.load().af_fwd_waves(b, h, h // G, S, D, api.ROPE[rope], MASK[mask], window or 0, int(bool(bias)))

    n = H // parts
    assert waves(B, H) == 8 and waves(1, n) == 4, "the case is meant to compare the two forms"
    o, lse = call(q, k, v, bt)
    for b in range(B):
        for h in range(0, H, n):
            x, y = call(q[b:b + 1, h:h + n], k[b:b + 1, h // G:(h + n) // G], v[b:b + 1, h // G:(h + n) // G],
                        None if bt is None else bt[b:b + 1])
            assert torch.equal(o[b:b + 1, h:h + n], x) and torch.equal(lse[b:b + 1, h:h + n], y)
