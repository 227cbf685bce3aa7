"""Helpers for the GPU parity tests: run a workload through the C ABI (via the thin
binding) and through the fp64 oracle, and compare."""
import numpy as np
import torch

import paper_2507_08045_amd as kr
import workloads

TOL = 2e-3   # absolute tolerance on similarities (cosine and distance), from the benchmark spec


def to_device(w: workloads.Workload):
    if w.dtype in ("f32", "f16"):
        q = torch.from_numpy(w.q).cuda()
        k = torch.from_numpy(w.k).cuda()
    else:
        q = torch.from_numpy(w.q.view(np.int16)).cuda().view(torch.bfloat16)
        k = torch.from_numpy(w.k.view(np.int16)).cuda().view(torch.bfloat16)
    return q, k


def arrays_to_device(q: np.ndarray, k: np.ndarray):
    if q.dtype in (np.float32, np.float16):
        return torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda()
    return (torch.from_numpy(q.view(np.int16)).cuda().view(torch.bfloat16),
            torch.from_numpy(k.view(np.int16)).cuda().view(torch.bfloat16))


def gpu_scores(q, k, **kw):
    out = kr.pair_similarity(q, k, **kw)
    torch.cuda.synchronize()
    return {n: (None if out[n] is None else out[n].cpu().numpy()) for n in ("pair_score", "head_score", "pair_dist")}


def assert_close(got, want, tol=TOL, what=""):
    got = np.asarray(got, dtype=np.float64)
    assert np.all(np.isfinite(got)), f"{what}: non-finite output"
    err = np.max(np.abs(got - want))
    assert err <= tol, f"{what}: max |gpu - oracle| = {err:.3e} > {tol}"
    return err


def check_selection(oracle, gpu_pair_score, oracle_pair_score, n_select):
    """The selector run on the GPU scores must equal the oracle selector on the same
    fp32 scores bit for bit.  It must also equal the oracle's own end-to-end choice
    whenever the two score vectors are certain to sort alike: every two oracle scores of a
    conversation further apart than twice the error observed between GPU and oracle scores
    (then no two candidates can have changed places, so the scan sees the same list)."""
    ps = torch.from_numpy(np.ascontiguousarray(gpu_pair_score, dtype=np.float32)).cuda()
    pairs, count = kr.select_pairs(ps, n_select)
    torch.cuda.synchronize()
    pairs, count = pairs.cpu().numpy(), count.cpu().numpy()
    want_pairs, want_count = oracle.select_pairs(np.asarray(gpu_pair_score, dtype=np.float64), n_select)
    np.testing.assert_array_equal(pairs, want_pairs)
    np.testing.assert_array_equal(count, want_count)
    e2e_pairs, e2e_count = oracle.select_pairs(oracle_pair_score, n_select)
    margins, asserted = [], 0
    for b in range(oracle_pair_score.shape[0]):
        s = np.sort(oracle_pair_score[b])
        margins.append(np.min(np.diff(s)) if s.size > 1 else np.inf)
        err = float(np.max(np.abs(np.asarray(gpu_pair_score[b], dtype=np.float64) - oracle_pair_score[b])))
        assert err <= TOL
        if margins[-1] > 2 * err:
            np.testing.assert_array_equal(pairs[b], e2e_pairs[b])
            assert count[b] == e2e_count[b]
            asserted += 1
    check_selection.last_asserted = asserted   # conversations whose end-to-end choice was compared
    return pairs, count, min(margins)


def all_pairs_tolerance(q, k, causal, split=None):
    """What the rounding of the exponentials to binary16 can do to all-pairs results, for q [B,L,Hq,Tq,d] and k [B,L,Hkv,S,d] on
    the GPU: (head cosines [B,Hq,L,L], pair cosines [B,L,L], pair distances [B,L,L]), six standard deviations.  Every stored exponential
    is off by an independent 2^-11 of itself at most (2^-11/sqrt(3) rms); with `split` keys per key split there are two such roundings
    (of the exponential and of its product with its split's factor) and a third that a split's keys share (the factor's).  To first order, with a, b
    the normalised rows, c their cosine, d the distance of the weights p, r:  dc = sum_k (a_k b_k - c a_k^2) e_k + the same for b,
    dd = sum_k (p_k - r_k) p_k / d e_k + the same for r; the mean of N rows deviates by the root of their mean variance over N.
    On top: float32 sums (2e-6), and under the distance's root a float32 difference of squares."""
    B, L, Hq, Tq, d = q.shape
    S, g = k.shape[3], Hq // k.shape[2]
    eps2 = 2.0 ** -22 / 3
    cos_var = torch.empty(B, Hq, L, L, dtype=torch.float64, device="cuda")   # (of a row, averaged over a head's rows)
    dist_var, dist_floor = torch.empty_like(cos_var), torch.empty_like(cos_var)
    for b in range(B):
        for h in range(Hq):
            x = torch.matmul(q[b, :, h].double(), k[b, :, h // g].double().transpose(-1, -2).contiguous()) / d ** 0.5
            if causal:
                seen = torch.arange(S, device="cuda")[None, :] <= torch.arange(S - Tq, S, device="cuda")[:, None]
                x = x.masked_fill(~seen, -float("inf"))
            p = torch.softmax(x, -1).transpose(0, 1).contiguous()   # [Tq, L, S]

            def gram(u, v):
                return torch.matmul(u, v.transpose(-1, -2).contiguous())

            def both(m):   # m[i][j] + m[j][i]
                return m + m.transpose(-1, -2)
            p2 = p * p
            n2 = p2.sum(-1)                                          # |p_i|^2
            ni, nj = n2[:, :, None], n2[:, None, :]
            G = gram(p, p)
            nn = torch.sqrt(ni * nj)
            c = G / nn
            dist2 = (ni + nj - 2 * G).clamp(min=1e-30)
            g22, g31, p4 = gram(p2, p2), gram(p2 * p, p), (p2 * p2).sum(-1)
            own = g22 / nn ** 2 - 2 * c * g31 / (nn * ni) + c * c * p4[:, :, None] / ni ** 2
            var_c = (2 if split else 1) * eps2 * both(own)
            var_d = (2 if split else 1) * eps2 * both(p4[:, :, None] - 2 * g31 + g22) / dist2
            if split:
                for s in range(0, S, split):
                    ps = p[..., s:s + split].contiguous()
                    gs, ns = gram(ps, ps), (ps * ps).sum(-1)[:, :, None]
                    var_c += eps2 * both((gs / nn - c * ns / ni) ** 2)
                    var_d += eps2 * both((ns - gs) ** 2) / dist2
            root = 4 * 2.0 ** -24 * (ni + nj)
            floor_d = torch.minimum(torch.sqrt(root), root / (2 * torch.sqrt(dist2)))
            cos_var[b, h], dist_var[b, h], dist_floor[b, h] = var_c.clamp(min=0).mean(0), var_d.clamp(min=0).mean(0), floor_d.mean(0)
    head = 6 * torch.sqrt(cos_var / Tq) + 2e-6
    pair = 6 * torch.sqrt(cos_var.mean(1) / (Tq * Hq)) + 2e-6
    dist = 6 * torch.sqrt(dist_var.mean(1) / (Tq * Hq)) + dist_floor.mean(1) + 2e-6
    return head.cpu().numpy(), pair.cpu().numpy(), dist.cpu().numpy()


def assert_all_pairs(got, want, tolerances, what):
    """Results of all_pairs_similarity (a dict of GPU tensors) against the oracle's, within all_pairs_tolerance."""
    for n, tol in zip(("head_score", "pair_score", "pair_dist"), tolerances):
        x = got[n].cpu().numpy().astype(np.float64)
        assert np.isfinite(x).all(), f"{what} {n}: non-finite output"
        err = np.abs(x - want[n])
        at = np.unravel_index(np.argmax(err / tol), err.shape)
        print(f"[{what}] {n}: {err[at]:.2e} of {tol[at]:.2e} allowed", flush=True)
        assert err[at] <= tol[at], f"{what} {n} at {at}: off by {err[at]:.3e}, allowed {tol[at]:.3e}"
