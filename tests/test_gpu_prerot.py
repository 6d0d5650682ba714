"""The forward on keys rotated once into scratch equals the one that rotates
them in its loop, bit for bit (both round the same fp32 rotation to fp16 once),
over the forms the scratch path accepts."""
import pytest
import torch

from gpu_util import announce, device_inputs, need_gpu
from paper_2609_13612_amd import api, blockmask, inputs

pytestmark = pytest.mark.gpu


def _both(monkeypatch, call, k):
    scratch = torch.empty(k.numel() * 2, dtype=torch.uint8, device="cuda")
    res = []
    monkeypatch.setattr(api, "_native", None)   # marshalled where the scratch can be chosen
    for s in (None, scratch):
        monkeypatch.setattr(api, "_fwd_scratch", lambda *a, s=s, **kw: s)
        res.append(call())
    torch.cuda.synchronize()
    assert torch.equal(res[0][0], res[1][0])
    if res[0][1] is not None:
        assert torch.equal(res[0][1], res[1][1])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rope", ["neox", "interleaved"])
@pytest.mark.parametrize("mask,window", [("none", None), ("causal", None), ("sliding_window", 70)])
@pytest.mark.parametrize("B,H,Hkv,S", [(1, 2, 2, 1), (2, 8, 2, 127), (1, 5, 5, 321), (1, 16, 1, 600)])
def test_dense(monkeypatch, B, H, Hkv, S, D, rope, mask, window):
    need_gpu()
    announce(f"prerot dense {B} {H}/{Hkv} {S} {D} {rope} {mask}")
    _, d = device_inputs(B, H, Hkv, S, D, seed=S)
    kw = dict(rope=rope, mask=mask, window=window)
    slopes = inputs.alibi_slopes(H).cuda()
    for a in (None, slopes):
        _both(monkeypatch, lambda: api.attnfuse_fwd(d["q"], d["k"], d["v"], alibi_slopes=a, **kw), d["k"])
    bias = torch.randn(B, H, S, S, device="cuda")
    for norm in ("softmax", "relu"):
        for b in (None, bias):
            _both(monkeypatch, lambda: api.attnfuse_fwd_bias_norm(d["q"], d["k"], d["v"], bias=b, norm=norm, **kw), d["k"])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rope", ["neox", "interleaved"])
@pytest.mark.parametrize("mask", ["none", "causal"])
@pytest.mark.parametrize("B,H,Hkv,S", [(1, 2, 2, 130), (2, 8, 2, 700)])
def test_block_sparse(monkeypatch, B, H, Hkv, S, D, rope, mask):
    need_gpu()
    announce(f"prerot sparse {B} {H}/{Hkv} {S} {D} {rope} {mask}")
    _, d = device_inputs(B, H, Hkv, S, D, seed=S)
    bm = blockmask.block_mask_from_dense(inputs.random_blocks(blockmask.num_blocks(S), 0.5, seed=1, empty_rows=(1,)), S,
                                         "cuda")
    _both(monkeypatch, lambda: api.attnfuse_fwd_blocksparse(d["q"], d["k"], d["v"], bm, rope=rope, mask=mask), d["k"])


def test_public_call_takes_the_scratch_path():
    """A long prompt through the public entry point, on a side stream, eager and captured."""
    need_gpu()
    announce("prerot public")
    B, H, Hkv, S, D = 1, 32, 8, 4096, 128
    kw = dict(rope="neox", mask="causal")
    assert api._fwd_scratch(torch.empty(0, device="cuda", dtype=torch.bfloat16), B, H, Hkv, S, D, 1, 1, 0) is not None
    _, d = device_inputs(B, H, Hkv, S, D, seed=3)
    api.attnfuse_fwd(d["q"], d["k"], d["v"], **kw)   # the table
    outs = []
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        for _ in range(3):
            outs.append(api.attnfuse_fwd(d["q"], d["k"], d["v"], **kw))
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        outs.append(api.attnfuse_fwd(d["q"], d["k"], d["v"], **kw))
    for _ in range(3):
        outs[-1][0].zero_()
        g.replay()
        torch.cuda.synchronize()
        for o, lse in outs:
            assert torch.equal(o, outs[0][0]) and torch.equal(lse, outs[0][1])
