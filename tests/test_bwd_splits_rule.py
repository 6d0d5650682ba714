"""How many workgroups share a key block of the dK/dV pass under a block mask
(CPU): by the lengths of the mask's lists, never more than the dense call of the
sizes takes, and one where they are not known."""
import numpy as np
import pytest
import torch

from paper_2609_13612_amd import _lib, blockmask, inputs


ROOM = 1 << 40   # any number of partials fits


def _dense(B, H, Hkv, S, D, mask, room=ROOM):
    return _lib.load().af_bwd_splits(B, H, Hkv, S, D, mask, 0, 0, -1, room)


def _sparse(B, H, Hkv, S, D, mask, active, window=0):
    bm = blockmask.block_mask_from_dense(torch.from_numpy(np.array(active)), S)
    longest, tiles = bm.col_tiles[mask != 0]
    return _lib.load().af_bwd_splits(B, H, Hkv, S, D, mask, window, longest, tiles, ROOM)


def _mask(kind, nb):
    i = np.arange(nb)
    band = abs(i[:, None] - i[None])
    return {"diag": band == 0, "band": band <= 1, "random": np.random.default_rng(1).random((nb, nb)) < 0.1,
            "bigbird": inputs.bigbird_blocks(nb, n_random=1), "all": band >= 0}[kind]


# whole backward unsplit / as the dense call, us: 55 / 81, 59 / 83, 87 / 96, 73 / 90, 65 / 83, 46 / 58
@pytest.mark.parametrize("B,H,Hkv,S,D,kind", [(1, 8, 8, 2000, 128, "diag"), (1, 8, 8, 2000, 128, "band"),
                                              (1, 8, 8, 2000, 128, "random"), (1, 32, 8, 2048, 128, "diag"),
                                              (1, 4, 1, 8000, 128, "diag"), (1, 2, 1, 16000, 64, "diag")])
def test_short_lists_are_not_split(B, H, Hkv, S, D, kind):
    assert _dense(B, H, Hkv, S, D, 1) > 1
    assert _sparse(B, H, Hkv, S, D, 1, _mask(kind, blockmask.num_blocks(S))) == 1


# 325 / 143, 397 / 95, 332 / 152
@pytest.mark.parametrize("B,H,Hkv,S,D,kind", [(1, 32, 8, 2048, 128, "bigbird"), (1, 8, 2, 4000, 64, "bigbird"),
                                              (1, 4, 1, 8000, 128, "random")])
def test_long_lists_are(B, H, Hkv, S, D, kind):
    assert 1 < _sparse(B, H, Hkv, S, D, 1, _mask(kind, blockmask.num_blocks(S))) <= _dense(B, H, Hkv, S, D, 1)


@pytest.mark.parametrize("S", [1, 64, 129, 333, 600, 1000, 2049])
@pytest.mark.parametrize("mask,window", [(0, 0), (1, 0), (2, 200)])
def test_all_active_is_the_dense_call(S, mask, window):
    lib = _lib.load()
    for B, H, Hkv in ((1, 8, 2), (1, 1, 1), (3, 16, 16)):
        for D in (64, 128):
            want = lib.af_bwd_splits(B, H, Hkv, S, D, mask, window, 0, -1, ROOM)
            assert _sparse(B, H, Hkv, S, D, mask, _mask("all", blockmask.num_blocks(S)), window) == want


def test_unknown_lists_are_not_split():
    assert _dense(1, 32, 8, 2048, 128, 1) > 1
    assert _lib.load().af_bwd_splits(1, 32, 8, 2048, 128, 1, 0, 0, 0, ROOM) == 1


@pytest.mark.parametrize("S,density", [(64, 1.0), (65, 0.5), (600, 0.3), (1000, 0.0), (2111, 0.1)])
def test_list_lengths(S, density):
    nb = blockmask.num_blocks(S)
    active = inputs.random_blocks(nb, density, seed=S)
    bm = blockmask.block_mask_from_dense(torch.from_numpy(active), S)
    for got, a in zip(bm.col_tiles, (active, np.tril(active))):
        n = [a[:, j:j + 2].any(axis=1).sum() for j in range(0, nb, 2)]
        assert got == (max(n), sum(n))
    assert bm.to("cpu").col_tiles == bm.col_tiles


@pytest.mark.parametrize("B,H,Hkv,S,D,mask", [(1, 32, 8, 512, 128, 1), (1, 8, 2, 4000, 64, 1), (3, 16, 4, 1777, 128, 0)])
def test_as_many_as_the_workspace_holds(B, H, Hkv, S, D, mask):
    n, part = _dense(B, H, Hkv, S, D, mask), 8 * B * Hkv * S * D
    assert n > 1
    for room, want in ((0, 1), (part, 1), (2 * part - 1, 1), (2 * part, 2), (n * part - 1, n - 1), (n * part, n)):
        assert _dense(B, H, Hkv, S, D, mask, room) == want


def _unsplit_bytes(B, H, Hkv, S, D, rope):
    """What the backward needs without partials, section by section."""
    up = lambda x: (x + 255) & ~255
    n = 2 * up(4 * B * H * S) + up(2 * B * H * S * D) + up(4 * B * Hkv)
    n += up(4 * B * Hkv * -(-(H // Hkv) * S * D // 16384))
    return n + (up(2 * B * H * S * D) + up(2 * B * Hkv * S * D) if rope else 0)


@pytest.mark.parametrize("B,H,Hkv,S,D", [(1, 32, 8, 512, 128), (1, 8, 2, 4000, 64), (3, 16, 4, 1777, 128),
                                         (1, 32, 8, 8192, 128)])
@pytest.mark.parametrize("rope", [0, 1])
def test_room_for_partials_is_not_required(B, H, Hkv, S, D, rope):
    """A workspace without room for partials is accepted in both types: with it the call is refused later, for a bias
    together with slopes (bf16) or a bias (fp32), and one byte less is an invalid argument."""
    lib = _lib.load()
    need = _unsplit_bytes(B, H, Hkv, S, D, rope)
    assert need <= lib.attnfuse_bwd_workspace_bytes(B, H, Hkv, S, D, rope)
    p = [0x1000000 * i for i in range(1, 14)]

    def code(dtype, nbytes):
        return lib.attnfuse_bwd_bias_norm(*p[:9], p[10], 0, 0, 0, 0, p[9], nbytes, B, H, Hkv, S, D, dtype, rope, 1e4,
                                          p[11], S, 1, 0, p[12], 0.1, None)
    for dtype in (0, 1):
        assert code(dtype, need) == -2
        assert code(dtype, need - 1) == -1
