"""The dK/dV pass where several workgroups share a key block (fp32 partials and
a reduction): gradients against the fp64 oracle at sizes whose steps do not
divide evenly, with ragged last blocks, every RoPE kind and mask, ALiBi, a bias
and relu weights, and nothing written past the workspace."""
import pytest
import torch

import oracle
from gpu_util import announce, assert_bf16_close, assert_fp32_close, device_inputs, f64, need_gpu
from paper_2609_13612_amd import _lib, api, blockmask, inputs

pytestmark = pytest.mark.gpu

CASES = [(1, 8, 2, 600, 128, "neox", "causal", None, None), (2, 4, 1, 333, 128, "neox", "none", None, "softmax"),
         (1, 8, 2, 1001, 64, "interleaved", "causal", None, None), (1, 6, 1, 515, 128, "none", "causal", None, None),
         (2, 6, 1, 300, 64, "neox", "none", None, "relu"), (1, 8, 1, 700, 128, "interleaved", "sliding_window", 333, None)]


@pytest.mark.parametrize("B,H,Hkv,S,D,rope,mask,window,norm", CASES, ids=lambda x: str(x))
def test_split_gradients(B, H, Hkv, S, D, rope, mask, window, norm):
    need_gpu()
    announce(f"bwd splits {B} {H}/{Hkv} {S} {D} {rope} {mask} {norm}")
    cpu, d = device_inputs(B, H, Hkv, S, D, seed=S, with_do=True)
    kw = dict(rope=rope, mask=mask, window=window)
    okw = dict(kw, theta=10000.0)
    fwd, bwd = api.attnfuse_fwd, api.attnfuse_bwd
    if norm:
        bias = torch.randn(B, 1, 1, S, generator=torch.Generator().manual_seed(S))
        scale = (1.0 if norm == "softmax" else 1.0 / S) / D ** 0.5
        if norm == "relu":
            bias = bias / S
        kw.update(norm=norm, bias=bias.cuda(), scale=scale)
        okw.update(norm=norm, bias=f64(bias.expand(B, H, S, S)), scale=scale)
        if norm == "relu":
            okw["relu_gate"] = "fp16"
        fwd, bwd = api.attnfuse_fwd_bias_norm, api.attnfuse_bwd_bias_norm
    elif rope == "none":
        kw["alibi_slopes"] = inputs.alibi_slopes(H).cuda()
        okw["alibi_slopes"] = f64(inputs.alibi_slopes(H))
    n = api.attnfuse_bwd_workspace_bytes(B, H, Hkv, S, D, rope)
    unsplit = 2 * B * S * D * (H + (H + Hkv if rope != "none" else 0)) + 8 * B * H * S + 16384
    assert n > unsplit + 2 * 8 * B * Hkv * S * D - 1, "the case is meant to split"
    o, lse = fwd(d["q"], d["k"], d["v"], **kw)
    ws = torch.full((n + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    g = bwd(d["q"], d["k"], d["v"], o, d["do"], lse, workspace=ws[:n], **kw)
    torch.cuda.synchronize()
    assert (ws[n:] == 0x5A).all(), "written past the workspace"
    ref = oracle.attention_backward(*[f64(cpu[x]) for x in ("q", "k", "v", "do")], **okw)
    for name, a, r in zip(("dQ", "dK", "dV"), g, ref):
        assert_bf16_close(a, r, name)


@pytest.mark.parametrize("B,H,Hkv,S,D,rope,mask,window", [
    (1, 8, 2, 1001, 64, "neox", "causal", None), (1, 16, 2, 700, 128, "none", "none", None),
    (2, 8, 1, 650, 128, "interleaved", "sliding_window", 300)])
def test_split_gradients_under_a_block_mask(B, H, Hkv, S, D, rope, mask, window):
    """Lists of very different lengths (a global block, a band, an empty column): some shares hold nothing."""
    need_gpu()
    announce(f"bwd splits sparse {B} {H}/{Hkv} {S} {D} {rope} {mask}")
    cpu, d = device_inputs(B, H, Hkv, S, D, seed=S, with_do=True)
    nb = blockmask.num_blocks(S)
    active = torch.from_numpy(inputs.bigbird_blocks(nb, n_random=1)).clone()
    active[:, 3] = False
    bm = blockmask.block_mask_from_dense(active.cuda(), S)
    assert bm.col_tiles == blockmask.block_mask_from_dense(active, S).col_tiles
    n = _lib.load().af_bwd_splits(B, H, Hkv, S, D, api.MASK[mask], window or 0, *bm.col_tiles[mask != "none"], 1 << 40)
    assert n > 1, "the case is meant to split"
    kw = dict(rope=rope, mask=mask, window=window)
    o, lse = api.attnfuse_fwd_blocksparse(d["q"], d["k"], d["v"], bm, **kw)
    g = api.attnfuse_bwd_blocksparse(d["q"], d["k"], d["v"], o, d["do"], lse, bm, **kw)
    ref = oracle.attention_backward(*[f64(cpu[x]) for x in ("q", "k", "v", "do")], theta=10000.0,
                                    block_mask=bm.as_oracle(), **kw)
    for name, a, r in zip(("dQ", "dK", "dV"), g, ref):
        assert_bf16_close(a, r, name)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_smaller_workspaces(dtype):
    """One workspace of the longest sequence's size serves shorter ones that would share more, one without room for any
    partials works too, and neither is written past its end."""
    need_gpu()
    B, H, Hkv, D = 1, 8, 2, 64
    size = lambda S: api.attnfuse_bwd_workspace_bytes(B, H, Hkv, S, D, "neox")
    unsplit = lambda S: 2 * B * S * D * (2 * H + Hkv) + 8 * B * H * S + 4096   # (4096: the small sections, with slack)
    room = lambda S, n: _lib.load().af_bwd_splits(B, H, Hkv, S, D, 1, 0, 0, -1, max(0, n - unsplit(S)))
    longest = size(700)
    assert room(1000, unsplit(1000)) == 1 < room(1000, unsplit(1000) + 3 * 8 * B * Hkv * 1000 * D) < room(1000, 1 << 40)
    for S, n in ((700, longest), (300, longest), (1000, unsplit(1000)), (1000, unsplit(1000) + 3 * 8 * B * Hkv * 1000 * D)):
        announce(f"bwd workspace {dtype} {S} {n}")
        cpu, d = device_inputs(B, H, Hkv, S, D, dtype=dtype, seed=S, with_do=True)
        o, lse = api.attnfuse_fwd(d["q"], d["k"], d["v"], rope="neox")
        ws = torch.full((n + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        g = api.attnfuse_bwd(d["q"], d["k"], d["v"], o, d["do"], lse, rope="neox", workspace=ws[:n])
        torch.cuda.synchronize()
        assert (ws[n:] == 0x5A).all(), "written past the workspace"
        ref = oracle.attention_backward(*[f64(cpu[x]) for x in ("q", "k", "v", "do")], rope="neox", theta=10000.0,
                                        mask="causal")
        for name, a, r in zip(("dQ", "dK", "dV"), g, ref):
            (assert_bf16_close if dtype == "bf16" else assert_fp32_close)(a, r, name)
