"""Plans of long calls: the workgroups fill the rounds they run in, within the limit on records, whatever the number of row tiles."""
import math

import pytest

import paper_2507_08045_amd as kr

# (B, L, Hq, Hkv, d, S, Tq): numbers of units and row tiles for which ceil(256 / tiles) splits are just over one round
SHAPES = [(1, 32, 32, 8, 128, 19743, 1042), (3, 32, 32, 8, 128, 12162, 128), (1, 32, 32, 8, 128, 27723, 299), (2, 32, 32, 8, 128, 15337, 175),
          (6, 32, 32, 8, 128, 2702, 700), (1, 32, 32, 8, 128, 2573, 806), (5, 32, 32, 8, 128, 971, 417), (2, 24, 16, 4, 64, 18625, 120)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[6]}-over-{s[5]}")
def test_rounds_are_full(shape):
    B, L, Hq, Hkv, d, S, Tq = shape
    sh = kr.KrulShape(*shape, kr.KRUL_BF16, 0.0, 0)
    p = kr.plan(sh)
    places = 512 if p["form"] in (5, 6) else 256   # workgroups that run side by side
    rounds = p["n_workgroups"] / places
    assert rounds / math.ceil(rounds) >= 0.85, p
    assert kr.workspace_bytes(sh) <= (520 << 20)


@pytest.mark.parametrize("shape", [(1, 32, 32, 8, 128, 6000, 1), (6, 32, 32, 8, 128, 916, 1), (3, 80, 64, 8, 128, 5535, 1), (1, 32, 32, 8, 128, 8253, 1),
                                   (1, 80, 64, 8, 128, 1494, 1)], ids=lambda s: f"{s[0]}-over-{s[5]}")
def test_no_nearly_empty_last_round_of_a_decode_step(shape):
    p = kr.plan(kr.KrulShape(*shape, kr.KRUL_BF16, 0.0, kr.KRUL_FLAG_CAUSAL))
    rounds = p["n_workgroups"] / (512 if p["form"] == 5 else 256)
    assert rounds <= 1 or rounds / math.ceil(rounds) >= 0.7, p


@pytest.mark.parametrize("shape", [(2, 24, 16, 4, 64, 11145, 1), (13, 24, 16, 4, 64, 1652, 1), (2, 24, 16, 4, 64, 10944, 5)], ids=lambda s: f"{s[0]}x{s[6]}-over-{s[5]}")
def test_small_heads_cut_the_layers_rather_than_leave_one_workgroup_a_cu(shape):
    p = kr.plan(kr.KrulShape(*shape, kr.KRUL_BF16, 0.0, kr.KRUL_FLAG_CAUSAL))
    assert p["form"] == 5 and p["n_workgroups"] > 512, p


# calls for which 256 x 256 tiles are estimated to be the fastest, though their rows fill them badly or they are small
@pytest.mark.parametrize("shape", [(2, 8, 16, 4, 128, 14839, 49), (1, 8, 32, 8, 128, 13637, 52), (5, 32, 32, 8, 128, 12524, 50), (3, 80, 64, 8, 128, 1116, 51)],
                         ids=lambda s: f"{s[0]}x{s[6]}-over-{s[5]}")
def test_no_more_calls_take_the_tiles_that_keep_exponentials_in_binary16(shape):
    B, L, Hq, Hkv, d, S, Tq = shape
    rows, tiles = Hq // Hkv * Tq, -(-S // 256)
    row_tiles = -(-rows // 256)
    assert row_tiles * 256 * 7 > rows * 8 or B * Hkv * row_tiles * tiles < 512
    assert kr.plan(kr.KrulShape(*shape, kr.KRUL_BF16, 0.0, 0))["form"] != 8


def test_forms_are_told_apart():
    """Every long 16-bit call takes a matrix-core form, whatever its number: 0 is the kernel of float32 inputs and heads above 128."""
    for d in (8, 40, 64, 72, 96, 128):
        for S, Tq in ((16384, 64), (4096, 512), (65536, 1), (906, 1179)):
            assert kr.plan(kr.KrulShape(1, 24, 16, 4, d, S, Tq, kr.KRUL_BF16, 0.0, 0))["form"] != 0, (d, S, Tq)
