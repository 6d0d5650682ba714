"""The binding's forward on keys rotated once: which calls it takes, and its
argument checks (CPU; validation fails before any HIP call)."""
import pytest

from paper_2609_13612_amd import _lib

FAKE = 0x10000


def _bytes(B=1, H=32, Hkv=8, S=8192, D=128, dtype=0, rope=1, mask=1, window=0, norm=0, extra=0, blocks=0):
    return _lib.load().af_fwd_workspace_bytes(B, H, Hkv, S, D, dtype, rope, mask, window, norm, extra, blocks)


def test_long_rotated_prompts_take_the_scratch():
    for rope in (1, 2):
        assert _bytes(rope=rope) == 2 * 8 * 8192 * 128
    assert _bytes(B=4, mask=2, window=1024) == 2 * 4 * 8 * 8192 * 128
    assert _bytes(B=4, H=12, Hkv=12, S=4096, D=64, mask=0, blocks=377) == 2 * 4 * 12 * 4096 * 64


@pytest.mark.parametrize("kw", [
    dict(rope=0), dict(dtype=1), dict(S=128), dict(S=512, norm=1), dict(S=0), dict(B=0), dict(H=6, Hkv=4), dict(D=96), dict(S=(1 << 20) + 1),
    dict(H=12, Hkv=12, B=4, S=512, D=64)])
def test_other_calls_do_not(kw):
    assert _bytes(**kw) == 0


@pytest.mark.parametrize("kw,takes", [
    # measured in the loop / rotated once, us: 49.4 / 52.8, 83.0 / 85.6, 33.3 / 35.8, 26.2 / 28.1, 26.2 / 27.7, 19.3 / 20.9
    (dict(B=2, H=16, Hkv=16, S=2048, D=64, mask=0), False), (dict(H=12, Hkv=12, S=4096, D=64, mask=0), False),
    (dict(B=2, H=16, Hkv=16, S=1347, D=64, mask=0, rope=2), False), (dict(B=2, H=16, Hkv=4, S=2048, mask=2, window=300), False),
    (dict(H=8, Hkv=2, S=5066, D=64, mask=2, window=827), False), (dict(H=16, Hkv=16, S=915, D=64, mask=2, window=588), False),
    # 93.8 / 90.5, 45.1 / 44.1, 44.5 / 40.3, 39.3 / 28.8
    (dict(B=2, H=8, Hkv=2, S=4085, D=64, mask=0), True), (dict(B=2, H=16, Hkv=4, S=2048, mask=2, window=1024), True),
    (dict(B=2, H=16, Hkv=16, S=2048, D=64), True), (dict(S=1000, mask=0), True)])
def test_the_faster_form_is_taken(kw, takes):
    assert bool(_bytes(**kw)) == takes


# in the loop / rotated once, us: 37.8 / 26.2, 26.1 / 19.0, 24.1 / 17.9, 27.9 / 22.5, 28.3 / 24.2
@pytest.mark.parametrize("kw,plain", [
    (dict(H=2, Hkv=2, S=1165, D=64, mask=2, window=538), False), (dict(H=8, Hkv=1, S=891, D=64, rope=2, mask=0), True),
    (dict(H=2, Hkv=2, S=656, D=64, mask=2, window=491), False), (dict(B=4, H=2, Hkv=2, S=942, D=64, rope=2), True),
    (dict(H=12, Hkv=12, S=640, D=64), False)])
def test_alibi_and_bias_take_it_earlier(kw, plain):
    assert _bytes(extra=1, **kw) > 0
    assert (_bytes(**kw) > 0) == plain


@pytest.mark.parametrize("kw,takes", [
    # measured in the loop / rotated once, us: 72.5 / 86.8, 27.9 / 31.3, 27.0 / 31.0, 13.0 / 16.2, 15.7 / 17.4, 38.5 / 42.9
    (dict(B=2, S=6316, mask=2, window=25, blocks=2939), False), (dict(B=3, H=8, Hkv=2, S=4910, D=64, blocks=610), False),
    (dict(H=8, Hkv=8, S=3653, mask=2, window=39, blocks=971), False), (dict(B=2, H=8, Hkv=1, S=6016, D=64, mask=2, window=80, blocks=840), False),
    (dict(B=3, H=2, Hkv=2, S=2047, D=64, mask=0, blocks=307), False), (dict(H=16, Hkv=16, S=3498, D=64, mask=0, blocks=323), False),
    # 48.2 / 39.7, 116.8 / 77.2, 85.4 / 62.5
    (dict(H=12, Hkv=4, S=2245, mask=0, blocks=209), True), (dict(B=2, H=16, Hkv=16, S=7209, D=64, mask=2, window=81, blocks=337), True),
    (dict(H=1, Hkv=1, S=4564, mask=0, blocks=425), True),
    (dict(B=4, H=8, Hkv=1, S=3317, D=64, rope=2, mask=0, blocks=811), True)])   # 60.2 / 52.6
def test_the_faster_form_is_taken_under_a_block_mask(kw, takes):
    assert bool(_bytes(**kw)) == takes


BASE = dict(Q=FAKE, K=FAKE + 0x100, V=FAKE + 0x200, O=FAKE + 0x300, LSE=FAKE + 0x400, qp=None, ki=None, bias=None, sb=0,
            sh=0, sq=0, norm=0, ws=FAKE + 0x500, n=1 << 20, B=1, H=4, Hkv=2, S=16, D=64, dtype=0, rope=1, theta=1e4,
            table=0x40000, rows=4096, mask=1, window=0, slopes=None, scale=0.125, stream=None)


@pytest.mark.parametrize("kw", [
    dict(ws=None), dict(ws=FAKE + 0x508), dict(ws=FAKE), dict(ws=FAKE + 0x300), dict(ws=0x40000), dict(n=2 * 2 * 16 * 64 - 1),
    dict(rope=0), dict(dtype=1), dict(Q=None), dict(S=0), dict(qp=FAKE + 0x600), dict(ki=FAKE + 0x600),
    dict(qp=FAKE + 0x602, ki=FAKE + 0x700), dict(qp=FAKE + 0x300, ki=FAKE + 0x700),
    dict(qp=FAKE + 0x600, ki=FAKE + 0x700, S=64 * 2048 + 1), dict(rows=8), dict(scale=0.0), dict(norm=2)])
def test_bad_arguments_are_refused(kw):
    assert _lib.load().af_fwd_ws(*{**BASE, **kw}.values()) == -1
