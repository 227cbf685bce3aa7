"""Host logic of the float32 plans: the call with a workspace and krul_pair_similarity_static agree, and 96-row tiles cost no caller memory."""
import ctypes
import math
import random

import pytest

import paper_2507_08045_amd as kr

MODELS = [(32, 32, 8, 128), (80, 64, 8, 128), (32, 32, 32, 128), (24, 16, 16, 128), (28, 24, 8, 96), (36, 20, 4, 80), (16, 16, 4, 72),
          (12, 8, 8, 104), (24, 16, 4, 64)]


def between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def shape(B, L, Hq, Hkv, d, S, Tq, flags=0):
    return kr.KrulShape(B, L, Hq, Hkv, d, S, Tq, kr.KRUL_F32, 0.0, flags)


def shapes(n, seed=7):
    rng = random.Random(seed)
    for _ in range(n):
        L, Hq, Hkv, d = rng.choice(MODELS)
        yield between(rng, 1, 8), L, Hq, Hkv, d, between(rng, 64, 8192), between(rng, 1, 1024 * Hkv // Hq)


def test_static_call_takes_the_plan_of_the_call_with_a_workspace():
    """The same bits are promised wherever the workspace's size is at most the static area's.  (162 tokens over 664 keys: 96-row tiles would
    fit the area where the plans that they replace do not.)"""
    seen = 0
    for sz in [(3, 32, 32, 8, 128, 664, 162), *shapes(6000)]:
        for flags in (0, kr.KRUL_FLAG_CAUSAL):
            sh = shape(*sz, flags)
            if (sz[5] >= sz[6] or not flags) and kr.workspace_bytes(sh) <= kr.KRUL_STATIC_SCRATCH_BYTES:
                assert kr.plan(sh) == kr.plan(sh, static=True), sz
                seen += kr.plan(sh)["rows_per_tile"] == 96
    assert seen >= 20


def status(sh, ws_bytes):
    """Of a call that gets past the workspace's check only to find misaligned keys: nothing runs."""
    vp = ctypes.c_void_p
    return kr.lib().krul_pair_similarity(ctypes.byref(sh), vp(0x1000), vp(0x2008), vp(0x3000), None, None, vp(0x10000), ctypes.c_size_t(ws_bytes), None)


# (the longer history takes 96-row tiles and few records, the shorter one not)
@pytest.mark.parametrize("model,longer,shorter", [((8, 24, 16, 16, 128, 77), 173, 45), ((4, 32, 32, 8, 128, 19), 159, 98), ((2, 32, 32, 8, 128, 18), 397, 194),
                                                  ((2, 32, 32, 32, 128, 66), 143, 46)], ids=lambda v: str(v))
def test_memory_for_a_history_serves_a_shorter_one(model, longer, shorter):
    B, L, Hq, Hkv, d, Tq = model
    sh = shape(B, L, Hq, Hkv, d, longer, Tq)
    assert kr.plan(sh)["rows_per_tile"] == 96
    assert status(sh, kr.workspace_bytes(sh)) == kr.KRUL_EINVAL
    assert status(shape(B, L, Hq, Hkv, d, shorter, Tq), kr.workspace_bytes(sh)) == kr.KRUL_EINVAL


# calls that 32-row tiles are estimated to be fastest for among 32 and 64 rows, and 96-row tiles faster still
@pytest.mark.parametrize("size", [(1, 32, 32, 8, 128, 7260, 17), (4, 24, 16, 16, 128, 2224, 70), (6, 28, 24, 8, 96, 166, 22), (2, 80, 64, 8, 128, 786, 9),
                                  (8, 24, 16, 16, 128, 1081, 84), (3, 24, 16, 16, 128, 131, 83)], ids=lambda s: f"{s[0]}x{s[6]}-over-{s[5]}")
def test_one_row_block_is_not_given_up_for_three(size):
    """A wave with one row block sums the small terms of its products apart from the large ones, one with two or three does not."""
    assert kr.plan(shape(*size))["rows_per_tile"] == 32
