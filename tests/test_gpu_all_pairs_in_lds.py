"""GPU parity of the all-pairs kernel that keeps the exponentials of up to 32 layers in LDS: numbers of layers around what its
waves share out, key counts around a key block, row blocks with and without neighbours, and logits that grow along the
history, so that the reference exponents are raised many times."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

# (name, B, L, Hq, Hkv, d, S, Tq, dtype, causal, growing logits)
CASES = [
    ("two-layers-one-key", 1, 2, 1, 1, 64, 1, 1, "bf16", False, False),
    ("eight-layers-s31", 1, 8, 4, 2, 64, 31, 5, "f16", False, False),
    ("nine-layers-s33", 2, 9, 4, 1, 128, 33, 9, "bf16", False, True),
    ("seventeen-layers-d72", 1, 17, 6, 2, 72, 97, 11, "bf16", False, False),
    ("all-layers", 1, 32, 8, 2, 128, 161, 40, "bf16", False, True),
    ("all-layers-d40-causal", 2, 32, 4, 4, 40, 130, 70, "f16", True, False),
    ("31-layers-causal-growing", 1, 31, 4, 1, 128, 300, 33, "bf16", True, True),
    ("33-layers", 1, 33, 4, 2, 64, 65, 3, "bf16", False, True),   # one too many: the form with the exponentials in memory
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_matches_oracle(oracle, case):
    import gpu_util as G
    import paper_2507_08045_amd as kr
    name, B, L, Hq, Hkv, d, S, Tq, dtype, causal, growing = case
    rng = np.random.default_rng(len(name) + L * S)
    rho = rng.uniform(0.5, 0.95, size=(B, L - 1, Hkv))
    w = workloads.make(name, B=B, L=L, Hq=Hq, Hkv=Hkv, d=d, S=S, Tq=Tq, dtype=dtype, rho_k=rho, seed=61)
    q, k = G.to_device(w)
    kb = w.k
    if growing:   # logits' spread from 1 to 24 along the keys (exact: whole factors would not change the rounding question)
        gain = torch.exp2(torch.linspace(0, 4.6, S, device="cuda")).round()[:, None]
        k = (k.float() * gain).to(k.dtype).contiguous()
        kb = k.cpu().view(torch.int16).numpy().view(w.k.dtype).reshape(w.k.shape)
    want = oracle.all_pairs(w.q, kb, causal=causal)
    out = kr.all_pairs_similarity(q, k, want_head_score=True, flags=kr.KRUL_FLAG_CAUSAL if causal else 0)
    torch.cuda.synchronize()
    G.assert_all_pairs(out, want, G.all_pairs_tolerance(q, k, causal, split=128 if L > 32 else None), name)
