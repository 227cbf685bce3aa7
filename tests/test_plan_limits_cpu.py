"""Host logic of the plans: what the workspace queries ask for stays within the limit on a plan's records."""
import math
import random

import pytest

import paper_2507_08045_amd as kr

MODELS = [(32, 32, 8, 128), (80, 64, 8, 128), (80, 40, 40, 128), (24, 16, 4, 64), (28, 24, 8, 96), (36, 20, 4, 80), (2048, 2, 1, 64)]


def ceil_div(a, b):
    return -(-a // b)


def bound(B, L, Hq, Hkv, Tq, ir):
    """512 MB of records, or those of a round of 256 workgroups of 128 rows, or of all rows -- padded to the widest tile -- in the
    four splits that row tiles in patches of eight take; a quarter more for the Initial-Recent test's; the head values."""
    rows = B * Hkv * ceil_div(Hq // Hkv * Tq, 256) * 256
    heads = 3 * (B * L * Hq * 4 + 256)
    return max(512 << 20, 16 * L * max(256 * 128, 4 * rows)) * (5 if ir else 4) // 4 + heads + 1024


def sizes():
    rng = random.Random(3)

    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    named = [(8, (80, 64, 8, 128), 16384, 100), (8, (80, 64, 8, 128), 16384, 150), (1, (80, 64, 8, 128), 32768, 700),
             (5, (32, 32, 8, 128), 19169, 1727), (4, (80, 64, 8, 128), 14998, 292), (27, (32, 32, 8, 192), 37099, 132)]
    return named + [(spread(1, 64), rng.choice(MODELS), spread(100, 131072), spread(1, 2048)) for _ in range(600)]


# (a decode step keeps a record per row and key tile whatever their number: under 1 % of the keys it reads)
@pytest.mark.parametrize("dtype", [kr.KRUL_BF16, kr.KRUL_F32], ids=["bf16", "f32"])
@pytest.mark.parametrize("flags", [0, kr.KRUL_FLAG_CAUSAL], ids=["all keys", "causal"])
def test_workspace_stays_within_the_limit(dtype, flags):
    for B, (L, Hq, Hkv, d), S, Tq in sizes():
        if S < Tq or (dtype == kr.KRUL_BF16 and d <= 128 and Hq // Hkv * Tq <= 64):
            continue
        shp = kr.KrulShape(B, L, Hq, Hkv, d, S, Tq, dtype, 0.0, flags)
        assert 0 < kr.workspace_bytes(shp) <= bound(B, L, Hq, Hkv, Tq, False), (B, L, Hq, Hkv, d, S, Tq)
        assert 0 < kr.workspace_bytes_ir(shp) <= bound(B, L, Hq, Hkv, Tq, True), (B, L, Hq, Hkv, d, S, Tq)


def test_named_workspaces():
    """No gigabytes for a few per cent of the time, and none for a plan on keys in place that a turn on dense keys does not take."""
    def need(B, L, Hq, Hkv, S, Tq):
        return kr.workspace_bytes(kr.KrulShape(B, L, Hq, Hkv, 128, S, Tq, kr.KRUL_BF16, 0.0, 0))
    assert need(8, 80, 64, 8, 16384, 100) < 400 << 20
    assert need(1, 80, 64, 8, 32768, 700) < 520 << 20


def test_plans_do_not_obey_the_static_areas_size():
    """A call with a workspace fills the chip whether or not its plan would fit krul_pair_similarity_static's 40 MB."""
    def plan(B, L, Hq, Hkv, S, Tq):
        return kr.plan(kr.KrulShape(B, L, Hq, Hkv, 128, S, Tq, kr.KRUL_BF16, 0.0, 0))
    assert plan(2, 80, 64, 8, 7967, 129)["n_workgroups"] >= 256      # (not one key split in 144)
    assert plan(8, 80, 64, 8, 16384, 16)["form"] == 1                # 128 x 256: 5.28 ms, in 64 x 512 tiles 5.55
    assert plan(2, 32, 32, 8, 204, 1249)["form"] == 1                # 128 x 256: 334 us, in 64 x 128 tiles 420


def test_static_call_takes_what_the_portable_kernel_fits():
    """64 conversations x one token of 40 heads, 80 layers: 5 MB of records without the float32 kernel's padding to 32 rows, 105
    MB with it.  (The queries are misaligned: past the plan the call is refused before any GPU work.)"""
    import ctypes
    shp = kr.KrulShape(64, 80, 40, 40, 128, 1000, 1, kr.KRUL_F32, 0.0, 0)
    vp = ctypes.c_void_p
    rc = kr.lib().krul_pair_similarity_static(ctypes.byref(shp), vp(0x1008), vp(0x2000), vp(0x3000), None, None, None)
    assert rc in (kr.KRUL_EINVAL, kr.KRUL_ELAUNCH), rc   # (without a GPU the scratch area is not found)
