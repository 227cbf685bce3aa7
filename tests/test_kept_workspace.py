"""A caller that keeps one workspace over a growing history: memory that holds the plan of whole rounds serves every length, where
the fastest plans ask for more at some."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2507_08045_amd as kr
import workloads

vp = ctypes.c_void_p


def ceil_div(a, b):
    return -(-a // b)


def records(shape, rows, n_split, ir=False):
    """Bytes of a plan of `rows`-row tiles and n_split key splits: a record of 16 per row, split and layer (four more for the layer
    test) and the head values, each on 256."""
    B, L, Hq, Hkv, d, S, Tq = shape
    n = B * Hkv * ceil_div(Hq // Hkv * Tq, rows) * rows * n_split * L

    def up(v):
        return ceil_div(v, 256) * 256
    return up(16 * n) + 2 * up(4 * B * (L - 1) * Hq) + ((up(4 * n) + up(4 * B * L * Hq)) if ir else 0)


def status(sh, ws_bytes, entry):
    """Status of a call that gets past the workspace's check only to find misaligned keys: nothing runs."""
    ws, n = vp(0x10000), ctypes.c_size_t(ws_bytes)
    if entry == "dense":
        return kr.lib().krul_pair_similarity(ctypes.byref(sh), vp(0x1000), vp(0x2008), vp(0x3000), None, None, ws, n, None)
    if entry == "strided":
        kl = kr.KrulKLayout(0x1004, 1 << 20, 1 << 20, 1 << 10)
        return kr.lib().krul_pair_similarity_strided(ctypes.byref(sh), vp(0x1000), ctypes.byref(kl), vp(0x3000), None, None, ws, n, None)
    return kr.lib().krul_pair_similarity_ir(ctypes.byref(sh), vp(0x1000), vp(0x2008), ctypes.c_float(0.2), vp(0x3000), None, None,
                                            vp(0x4000), None, ws, n, None)


HISTORIES = sorted({*range(1024, 32769, 1024), 1300, 2707, 5214, 9451, 17255, 30001})

# entry, (B, L, Hq, Hkv, d, Tq), key splits of 128-row tiles whose records are enough at any of HISTORIES
KEPT = [("dense", (8, 32, 32, 8, 128, 172), 2), ("strided", (5, 24, 16, 4, 64, 393), 1), ("ir", (5, 24, 16, 4, 64, 393), 1)]


@pytest.mark.parametrize("entry,model,n_split", KEPT, ids=[c[0] for c in KEPT])
def test_one_workspace_over_a_growing_history(entry, model, n_split):
    B, L, Hq, Hkv, d, Tq = model
    ir, sizes = entry == "ir", []
    for S in HISTORIES:
        shape = (B, L, Hq, Hkv, d, S, Tq)
        sh = kr.KrulShape(*shape, kr.KRUL_BF16, 0.0, 0)
        need = records(shape, 128, n_split, ir)
        assert status(sh, need, entry) == kr.KRUL_EINVAL, S
        sizes.append(kr.workspace_bytes_ir(sh) if ir else kr.workspace_bytes(sh))
        assert status(sh, sizes[-1], entry) == kr.KRUL_EINVAL, S
        assert status(sh, records(shape, 64, 1, ir) // 2, entry) == kr.KRUL_EWORKSPACE, S
    assert max(sizes) > need   # (the fastest plans do take more at some)


# (B, L, Hq, Hkv, d, S, Tq), flags, rows of a tile, key splits of the plan of whole rounds
PLANS = [((3, 8, 16, 8, 128, 1681, 213), 0, 64, 3), ((2, 4, 16, 4, 96, 19406, 66), kr.KRUL_FLAG_CAUSAL, 64, 19),
         ((2, 4, 16, 8, 64, 19822, 72), 0, 64, 10), ((3, 8, 16, 8, 72, 2080, 231), kr.KRUL_FLAG_CAUSAL, 64, 5)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape,flags,rows,n_split", PLANS, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else "")
def test_the_plan_that_fits_matches_the_oracle(oracle, shape, flags, rows, n_split):
    import gpu_util as G
    B, L, Hq, Hkv, d, S, Tq = shape
    w = workloads.make("kept-workspace", B=B, L=L, Hq=Hq, Hkv=Hkv, d=d, S=S, Tq=Tq, dtype="bf16", seed=S)
    q, k = G.to_device(w)
    need, size = records(shape, rows, n_split), kr.workspace_bytes(kr.make_shape(q, k, 0.0, flags))
    assert need < size
    units = [(b, l, h) for b, l, h in ((0, 0, 0), (B - 1, L - 2, Hq - 1), (B - 1, (L - 1) // 2, Hq // 2))]
    cos, _ = oracle.unit_scores(w.q, w.k, units, causal=bool(flags))
    out = [kr.pair_similarity(q, k, flags=flags, want_head_score=True, workspace=torch.empty(n, dtype=torch.uint8, device="cuda")) for n in (size, need)]
    torch.cuda.synchronize()
    for o in out:
        err = np.max(np.abs(np.array([float(o["head_score"][u]) for u in units]) - cos))
        print(f"[{shape}] {err:.2e}", flush=True)
        # exponentials known to 7e-7 (logits below 16 to 2^-20), means of rows of thousands of keys to a fraction of that
        assert err <= 1e-6
    for n in ("head_score", "pair_dist"):
        assert torch.max(torch.abs(out[0][n] - out[1][n])) <= 2e-6


# All pairs: (B, L, Hq, Hkv, d, S, Tq), bytes of up to 256 rows of a kv head with eight classes, a round of splits and the rows'
# matrices: up to 32 layers, where the plan that is fastest wants sixteen classes, and with more
ALL_PAIRS = [((1, 24, 16, 4, 64, 346, 3), 2151424), ((4, 4, 2, 1, 128, 2488, 8), 4148736), ((1, 32, 8, 1, 128, 4200, 2), 8081408),
             ((1, 48, 16, 16, 64, 600, 20), 5539840), ((2, 40, 8, 2, 72, 500, 33), 10539008)]
ids = [f"{s[0]}x{s[6]}-over-{s[5]}-{s[1]}layers" for s, _ in ALL_PAIRS]


@pytest.mark.parametrize("shape,need", ALL_PAIRS, ids=ids)
def test_all_pairs_takes_a_smaller_batch(shape, need):
    sh = kr.KrulShape(*shape, kr.KRUL_BF16, 0.0, 0)

    def status(n):
        return kr.lib().krul_all_pairs_similarity(ctypes.byref(sh), vp(0x1000), vp(0x2008), vp(0x3000), None, None, vp(0x10000),
                                                  ctypes.c_size_t(n), None)
    for n in (need, kr.all_pairs_workspace_bytes(sh, 1), kr.all_pairs_workspace_bytes(sh)):
        assert status(n) == kr.KRUL_EINVAL, n
    assert status(need - 1) == kr.KRUL_EWORKSPACE
    assert kr.all_pairs_workspace_bytes(sh, need) == need   # (a budget is kept)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,need", ALL_PAIRS, ids=ids)
def test_all_pairs_in_a_smaller_batch_matches_the_oracle(oracle, shape, need):
    import gpu_util as G
    B, L, Hq, Hkv, d, S, Tq = shape
    w = workloads.make("kept-workspace-all-pairs", B=B, L=L, Hq=Hq, Hkv=Hkv, d=d, S=S, Tq=Tq, dtype="bf16", seed=S)
    q, k = G.to_device(w)
    out = kr.all_pairs_similarity(q, k, want_head_score=True, workspace=torch.empty(need, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    G.assert_all_pairs(out, oracle.all_pairs(w.q, w.k), G.all_pairs_tolerance(q, k, False, split=128 if L > 32 else None), f"{need} bytes")
