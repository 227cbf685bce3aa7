"""GPU parity of every workgroup tile shape of the matrix-core kernel.  Which shape runs is chosen by an estimate from the rows per
kv head and the size of the problem; each case below says which one its call takes (krul_pair_similarity_plan), and together they take
all of them, at both head sizes.  (The calls with other flags on the same inputs may take others.)"""
import zlib

import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return gpu_util


FORMS = {1: "128 x 256, eight waves", 2: "64 x 512, eight waves", 4: "32 x 512, four waves, deep ring", 5: "32 x 256, four waves", 6: "64 x 128, four waves", 7: "128 x 128, eight waves"}   # as krul_pair_similarity_plan numbers them

# (name, B, L, Hq, Hkv, d, S, Tq, dtype, form)
CASES = [
    ("slim-short", 2, 4, 16, 8, 128, 1300, 1, "bf16", 5),
    ("slim-short-d64-rows", 1, 3, 32, 8, 64, 2100, 4, "bf16", 5),
    ("slim-12-conversations", 12, 3, 16, 8, 128, 1300, 1, "bf16", 5),
    ("slim-f16", 16, 3, 8, 8, 64, 1100, 2, "f16", 5),
    ("slim-24-conversations", 24, 3, 16, 8, 128, 1300, 1, "bf16", 5),
    ("slim-40-conversations-d64", 40, 3, 8, 8, 64, 700, 3, "bf16", 5),
    ("mid-short", 2, 3, 16, 4, 128, 900, 12, "bf16", 6),
    ("mid-short-d64", 1, 4, 8, 8, 64, 1500, 40, "f16", 6),
    ("mid", 12, 3, 16, 8, 64, 700, 20, "bf16", 2),
    ("mid-d128", 9, 3, 8, 8, 128, 1100, 50, "bf16", 2),
    ("wide-short", 1, 3, 8, 2, 128, 700, 70, "bf16", 7),
    ("rows-200-d64", 2, 3, 8, 4, 64, 400, 100, "bf16", 6),
    ("rows-90-d64", 6, 3, 8, 8, 64, 600, 90, "bf16", 6),
    ("rows-130", 9, 3, 4, 4, 128, 500, 130, "f16", 6),
    ("deep-d64", 24, 2, 1, 1, 64, 4904, 1, "bf16", 4),
    ("deep", 24, 2, 2, 2, 128, 2488, 1, "f16", 4),
    ("wide-d64", 12, 2, 8, 8, 64, 263, 86, "bf16", 1),
    ("wide", 24, 2, 16, 4, 128, 261, 20, "f16", 1),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_tile_shapes_match_oracle(G, oracle, case):
    import paper_2507_08045_amd as kr
    name, B, L, Hq, Hkv, d, S, Tq, dtype, form = case
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    rho = rng.uniform(0.5, 0.95, size=(B, L - 1, Hkv))
    w = workloads.make(name, B=B, L=L, Hq=Hq, Hkv=Hkv, d=d, S=S, Tq=Tq, dtype=dtype, rho_k=rho, seed=211)
    q, k = G.to_device(w)
    assert kr.plan(kr.make_shape(q, k))["form"] == form
    want = oracle.pair_similarity(w.q, w.k)
    got = G.gpu_scores(q, k)
    e1 = G.assert_close(got["head_score"], want["head_score"], G.TOL, f"{name} head_score")
    G.assert_close(got["pair_score"], want["pair_score"], G.TOL, f"{name} pair_score")
    e3 = G.assert_close(got["pair_dist"], want["pair_dist"], G.TOL, f"{name} pair_dist")
    print(f"[{name}: {FORMS[form]}] max err head={e1:.2e} dist={e3:.2e}", flush=True)
    # the Initial-Recent test and the causal reading ride in the same kernels
    ir = kr.pair_similarity_ir(q, k, 0.2)
    torch.cuda.synchronize()
    want_mass, _ = oracle.ir_mass(w.q, w.k, 0.2)
    G.assert_close(ir["ir_mass"].cpu().numpy(), want_mass, G.TOL, f"{name} ir_mass")
    if Tq > 1:
        wc = oracle.pair_similarity(w.q, w.k, causal=True)
        gc = G.gpu_scores(q, k, flags=kr.KRUL_FLAG_CAUSAL)
        G.assert_close(gc["head_score"], wc["head_score"], G.TOL, f"{name} causal head_score")
    # one workgroup walking all key tiles (running records parked in memory between tiles)
    one = G.gpu_scores(q, k, flags=kr.KRUL_FLAG_SINGLE_SPLIT)
    G.assert_close(one["head_score"], want["head_score"], G.TOL, f"{name} single split")
