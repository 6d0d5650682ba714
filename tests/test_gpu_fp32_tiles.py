"""The fp32 kernels at the edges of their 16-row tiles and of the four waves
that share a tile's rows: forward and backward against the fp64 oracle.

Bound: 1e-5 on O, dQ, dK, dV relative to the largest value (a sum of n fp32
terms rounds to within n 2^-24 of the sum of their magnitudes; here n is at
most S D = 1.7e4, and random signs leave about sqrt(n) 2^-24 = 8e-6), 1e-5
absolute plus that on the LSE."""
import numpy as np
import pytest

import oracle
from gpu_util import announce, device_inputs, f64, need_gpu
from paper_2609_13612_amd import api, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 15, 16, 17, 64, 65, 131])
@pytest.mark.parametrize("H,Hkv,D,rope,mask,window,alibi", [
    (2, 2, 64, "neox", "causal", None, False), (6, 2, 128, "interleaved", "none", None, False),
    (4, 1, 64, "none", "sliding_window", 18, True), (2, 2, 128, "neox", "sliding_window", 1, False)])
def test_fp32_tile_edges(S, H, Hkv, D, rope, mask, window, alibi):
    need_gpu()
    announce(f"fp32 tiles S={S} H={H}/{Hkv} D={D} {rope} {mask}")
    cpu, dev = device_inputs(2, H, Hkv, S, D, dtype="fp32", seed=S, with_do=True)
    slopes = inputs.alibi_slopes(H) if alibi else None
    kw = dict(rope=rope, theta=10000.0, mask=mask, window=window)
    o, lse = api.attnfuse_fwd(dev["q"], dev["k"], dev["v"], alibi_slopes=slopes.cuda() if alibi else None, **kw)
    g = api.attnfuse_bwd(dev["q"], dev["k"], dev["v"], o, dev["do"], lse,
                         alibi_slopes=slopes.cuda() if alibi else None, **kw)
    okw = dict(kw, alibi_slopes=f64(slopes) if alibi else None)
    a = [f64(cpu[n]) for n in ("q", "k", "v")]
    O, L = oracle.attention_forward(*a, **okw)
    ref = oracle.attention_backward(*a, f64(cpu["do"]), **okw)
    assert np.abs(f64(lse) - L).max() <= 1e-5 * (1 + np.abs(L).max())
    for name, x, r in (("O", o, O), ("dQ", g[0], ref[0]), ("dK", g[1], ref[1]), ("dV", g[2], ref[2])):
        assert np.abs(f64(x) - r).max() <= 1e-5 * max(1.0, np.abs(r).max()), name
