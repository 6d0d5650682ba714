"""The native marshalling (native/binding.cpp) against the Python one: the same
bits, the same outputs given back, the same refusals, and None for what it
does not take."""
import pytest
import torch

from gpu_util import announce, device_inputs, need_gpu
from paper_2609_13612_amd import api, autograd, blockmask, inputs

pytestmark = pytest.mark.gpu
B, H, HKV, S, D = 2, 8, 2, 200, 64


def _calls(d):
    q, k, v, do = (d[n] for n in ("q", "k", "v", "do"))
    slopes = inputs.alibi_slopes(H).cuda()
    bias = torch.randn(B, 1, 1, S, device="cuda")
    bm = blockmask.block_mask_from_dense(inputs.random_blocks(4, 0.6, seed=1), S, "cuda")
    lens = torch.tensor([S, 3], dtype=torch.int32, device="cuda")
    qd = q[:, :, 5].contiguous()
    for rope, mask, window in (("neox", "causal", None), ("interleaved", "none", None), ("none", "sliding_window", 30)):
        kw = dict(rope=rope, theta=500000.0, mask=mask, window=window)
        for s in (None, slopes):
            o, lse = api.attnfuse_fwd(q, k, v, alibi_slopes=s, **kw)
            yield lambda s=s, kw=kw: api.attnfuse_fwd(q, k, v, alibi_slopes=s, scale=0.1, **kw)
            yield lambda s=s, kw=kw, o=o, lse=lse: api.attnfuse_bwd(q, k, v, o, do, lse, alibi_slopes=s, **kw)
            yield lambda s=s, kw=kw: api.attnfuse_decode(qd, k, v, lens, alibi_slopes=s, **kw)
            yield lambda s=s, kw=kw: api.attnfuse_decode_noalloc(qd, k, v, alibi_slopes=s, **kw)
            yield lambda s=s, kw=kw: api.attnfuse_fwd_blocksparse(q, k, v, bm, alibi_slopes=s, **kw)
            yield lambda s=s, kw=kw, o=o, lse=lse: api.attnfuse_bwd_blocksparse(q, k, v, o, do, lse, bm, alibi_slopes=s, **kw)
        for norm in ("softmax", "relu"):
            for b in (None, bias):
                o, lse = api.attnfuse_fwd_bias_norm(q, k, v, bias=b, norm=norm, **kw)
                assert (lse is None) == (norm == "relu")
                yield lambda b=b, norm=norm, kw=kw: api.attnfuse_fwd_bias_norm(q, k, v, bias=b, norm=norm, **kw)[:1]
                yield lambda b=b, norm=norm, kw=kw, o=o, lse=lse: api.attnfuse_bwd_bias_norm(
                    q, k, v, o, do, lse, bias=b, norm=norm, **kw)
    for rope in ("neox", "interleaved"):
        yield lambda rope=rope: api.attnfuse_rope(q, k, rope=rope)
        yield lambda rope=rope: api.attnfuse_rope(q, rope=rope)[:1]
        yield lambda rope=rope: api.attnfuse_rope_bwd(q, k, rope=rope)


def test_same_bits_as_the_python_marshalling(monkeypatch):
    need_gpu()
    announce("native against python marshalling")
    assert api._native is not None, "the native binding is not built"
    _, d = device_inputs(B, H, HKV, S, D, seed=1, with_do=True)
    n = 0
    for call in _calls(d):
        call()                                             # builds the table
        taken = []
        real = api._native

        class Spy:
            def __getattr__(self, name):
                def f(*a):
                    taken.append(getattr(real, name)(*a))
                    return taken[-1]
                return f
        with monkeypatch.context() as m:
            m.setattr(api, "_native", Spy())
            a = call()
        assert len(taken) == 1 and taken[0] is not None, "declined"
        with monkeypatch.context() as m:
            m.setattr(api, "_native", None)
            b = call()
        assert all(torch.equal(x, y) for x, y in zip(a, b))
        n += 1
    assert n > 40


def test_given_outputs_come_back_and_streams_are_kept():
    need_gpu()
    announce("native outputs and streams")
    _, d = device_inputs(B, H, HKV, S, D, seed=2, with_do=True)
    q, k, v = d["q"], d["k"], d["v"]
    out, lse = torch.empty_like(q), torch.empty(B, H, S, device="cuda")
    tab = api.rope_table(D, 10000.0, S)
    o, l = api.attnfuse_fwd(q, k, v, rope="neox", out=out, lse=lse, rope_table=tab)
    assert o is out and l is lse
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        big = torch.randn(4096, 4096, device="cuda")
        for _ in range(10):
            big = big @ big * 1e-3
        q2 = q.clone()                                     # ordered after the products on st
        o2, _ = api.attnfuse_fwd(q2, k, v, rope="neox", rope_table=tab)
    st.synchronize()
    assert torch.equal(o2, out)


def test_refusals_are_the_same():
    need_gpu()
    announce("native refusals")
    _, d = device_inputs(B, H, HKV, S, D, seed=3, with_do=True)
    q, k, v = d["q"], d["k"], d["v"]
    bad = [(ValueError, dict(out=torch.empty(B, H, S, D, device="cuda"))),
           (ValueError, dict(lse=torch.empty(B, H, S + 1, device="cuda"))),
           (ValueError, dict(alibi_slopes=torch.ones(H + 1, device="cuda"))),
           (ValueError, dict(rope="neox", rope_table=torch.empty(S - 1, D // 2, 2, device="cuda"))),
           (KeyError, dict(rope="half")), (KeyError, dict(mask="upper")),
           (api.AttnFuseError, dict(mask="sliding_window")), (api.AttnFuseError, dict(scale=-1.0)),
           (api.AttnFuseError, dict(scale=float("nan"))), (api.AttnFuseError, dict(out=q)),
           (api.AttnFuseError, dict(rope="neox", theta=-2.0))]
    for exc, kw in bad:
        with pytest.raises(exc):
            api.attnfuse_fwd(q, k, v, **kw)
    for a in ((q.transpose(1, 2), k, v), (q, k.float(), v), (q, k.cpu(), v), (q, k[:, :, :-1], v), (q.half(), k, v)):
        with pytest.raises(ValueError):
            api.attnfuse_fwd(*a)
    with pytest.raises(api.AttnFuseError):                 # too small a workspace
        api.attnfuse_bwd(q, k, v, q.clone(), d["do"], torch.zeros(B, H, S, device="cuda"),
                         workspace=torch.empty(16, device="cuda"))
    with pytest.raises(TypeError):
        api.attnfuse_bwd(q, k, v, q.clone(), d["do"], None)


def test_other_kinds_of_argument_still_run():
    """Values and tensors the native marshalling declines: numpy scalars, a float window, a subclass, a Parameter."""
    import numpy as np
    need_gpu()
    announce("native declined arguments")
    _, d = device_inputs(B, H, HKV, S, D, seed=4, with_do=True)
    q, k, v = d["q"], d["k"], d["v"]
    ref = api.attnfuse_fwd(q, k, v, rope="neox", theta=10000.0, mask="sliding_window", window=31, scale=0.125)

    class Sub(torch.Tensor):
        pass
    for qq, th, w, sc in ((q, np.float32(10000.0), 31, 0.125), (q, 10000, 31.0, 0.125), (q, 10000.0, np.int64(31), np.float64(0.125)),
                          (q.as_subclass(Sub), 10000.0, 31, None), (torch.nn.Parameter(q), 10000.0, 31, 0.125)):
        o, lse = api.attnfuse_fwd(qq, k, v, rope="neox", theta=th, mask="sliding_window", window=w, scale=sc)
        assert torch.equal(o, ref[0]) and torch.equal(lse, ref[1])


def test_gradients_through_saved_tensor_hooks():
    need_gpu()
    announce("native under saved-tensor hooks")
    _, d = device_inputs(B, H, HKV, S, D, seed=5, with_do=True)
    leaves = [d[n].clone().requires_grad_() for n in ("q", "k", "v")]
    want = torch.autograd.grad(autograd.attention(*leaves, rope="neox"), leaves, d["do"])
    with torch.autograd.graph.save_on_cpu():
        o = autograd.attention(*leaves, rope="neox")
    got = torch.autograd.grad(o, leaves, d["do"])
    assert all(torch.equal(x, y) for x, y in zip(want, got))


def test_same_bits_where_the_forward_takes_scratch(monkeypatch):
    """The calls with the longest argument list (scratch, a bias's strides, a block mask's lists), each against the Python
    marshalling and against the keys rotated in the loop."""
    need_gpu()
    announce("native against python marshalling, with scratch")
    B, H, HKV, S, D = 2, 16, 4, 2048, 128
    _, d = device_inputs(B, H, HKV, S, D, seed=6)
    q, k, v = d["q"], d["k"], d["v"]
    nb = blockmask.num_blocks(S)
    bm = blockmask.block_mask_from_dense(inputs.random_blocks(nb, 0.9, seed=1), S, "cuda")
    g = torch.Generator("cuda").manual_seed(1)
    biases = [torch.randn(s, generator=g, device="cuda") for s in ((B, 1, 1, S), (1, H, 1, S), (1, 1, S, S))]
    slopes = inputs.alibi_slopes(H).cuda()
    norms = [(n, b) for n in ("softmax", "relu") for b in [None] + biases]
    for rope, mask, window in (("neox", "causal", None), ("interleaved", "none", None), ("neox", "sliding_window", 1500)):
        kw = dict(rope=rope, theta=500000.0, mask=mask, window=window)
        calls = [(0, s is not None, 0, lambda s=s: api.attnfuse_fwd(q, k, v, alibi_slopes=s, **kw)) for s in (None, slopes)]
        calls += [(0, s is not None, bm.k_idx.numel(),
                   lambda s=s: api.attnfuse_fwd_blocksparse(q, k, v, bm, alibi_slopes=s, **kw)) for s in (None, slopes)]
        calls += [(api.NORM[n], b is not None, 0, lambda n=n, b=b: api.attnfuse_fwd_bias_norm(q, k, v, norm=n, bias=b, **kw))
                  for n, b in norms]
        for norm, extra, blocks, call in calls:
            assert api._fwd_scratch_bytes(B, H, HKV, S, D, 0, api.ROPE[rope], api.MASK[mask], window or 0, norm, int(extra),
                                          blocks) > 0
            a = call()
            with monkeypatch.context() as m:
                m.setattr(api, "_native", None)
                b = call()
                m.setattr(api, "_fwd_scratch", lambda *a, **kw: None)
                c = call()
            for x, y, z in zip(a, b, c):
                assert (x is None and y is None and z is None) or (torch.equal(x, y) and torch.equal(x, z))
