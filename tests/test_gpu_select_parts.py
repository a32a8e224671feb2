"""The one-launch selection of a layer at the edges of its ranges: score rows that
end inside a 16-byte vector, around a wave's 2048 and a batch's 16384 scores,
on both sides of the lengths where the three-launch selection takes over, with
ties, whole bins, more equal keys than its LDS list holds, and infinite,
negative and zero scores.

Selections are exact: the reference is a stable sort of the same scores by
(score descending, index ascending), scores below zero ranking as zero.
"""
import math

import numpy as np
import pytest
import torch

import paper_2508_02401_amd as ckv

pytestmark = pytest.mark.gpu


def _top(scores, n):
    key = np.maximum(scores.astype(np.float32), np.float32(0))
    return np.sort(np.argsort(-key, kind="stable")[:n])


@pytest.mark.parametrize("Ls", [1, 2, 3, 5, 1007, 2047, 2049, 8190, 16383, 16385, 32767, 32768, 32769,
                                40001])
@pytest.mark.parametrize("values", ["heavy", "ties", "narrow", "signed"])
def test_select_exact(Ls, values):
    dev, n_kv, d, w = torch.device("cuda:0"), 3, 64, 8
    rng = np.random.default_rng(Ls)
    if values == "heavy":
        sc = np.exp(2.0 * rng.standard_normal((n_kv, Ls)))
        sc[:, Ls // 2] = math.inf
    elif values == "ties":  # few distinct values, one of them most of the row
        sc = rng.choice([0.0, 0.25, 0.25, 0.25, 0.5], size=(n_kv, Ls))
    elif values == "narrow":  # one first-level bin, more keys than the LDS list holds
        sc = 1.0 + rng.random((n_kv, Ls)) / 64
    else:
        sc = rng.standard_normal((n_kv, Ls))
    sc = sc.astype(np.float32)
    desc = ckv.layer_desc(n_kv, n_kv, d, w, torch.bfloat16)
    k = torch.zeros((n_kv, Ls + w, d), dtype=torch.bfloat16, device=dev)
    for n in sorted({1, Ls // 3, Ls - 1, Ls}):
        if n < 0:
            continue
        s = ckv.Seq(None, k, k, n + w)
        s.scores = torch.from_numpy(sc).to(dev)
        s.idx = torch.full((n_kv, min(n + w, Ls + w)), -1, dtype=torch.int32, device=dev)
        ws = ckv.alloc_workspace(desc, [s], dev)
        print("case", Ls, values, n, flush=True)
        ckv.ckv_select(desc, [s], ws)
        torch.cuda.synchronize()
        got = s.idx.cpu().numpy()
        for g in range(n_kv):
            want = np.concatenate([_top(sc[g], n), np.arange(Ls, Ls + w)])
            assert np.array_equal(got[g], want), (Ls, values, n, g)


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("keep_window", [True, False])
@pytest.mark.parametrize("L,budgets", [(77, (9, 76, 77)), (2100, (40, 700)), (16500, (333, 16499)),
                                       (65540, (1000,)), (65600, (1000,))])
def test_compress_layer_parts(L, budgets, keep_window, shared):
    _compress_and_check(12, 3, [(L, b) for b in budgets], keep_window, shared)


# A batch of prompts of which one or two are long, with budgets at both ends of
# their range: units whose parts differ in number (8 KV heads: one prompt keeps
# most of the batch's rows), more units than CUs (24 KV heads), and prompts past
# 65536 scored tokens, which send the whole batch through the three launches.
RAGGED = {
    "parts": (8, 8, [(30001, 14000)] + [(200 + 31 * i, 9 + 40 * i) for i in range(13)] + [(77, 77), (500, 8)]),
    "rounds": (24, 24, [(2100, 8), (2100, 9), (2100, 2099), (2100, 2100), (300, 40), (5000, 600),
                        (77, 76), (900, 1000), (1025, 8), (64, 30), (333, 333), (2047, 12)]),
    "uneven": (24, 24, [(40000, 3000)] + [(300, 20)] * 11),
    "long": (12, 3, [(65700, 8), (300, 9), (65700, 65699), (300, 8), (300, 300), (2100, 700)]),
    "long keep all": (12, 3, [(65700, 65700), (300, 299), (70001, 9), (9000, 9001), (65700, 33000)]),
}


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("keep_window", [True, False])
@pytest.mark.parametrize("batch", sorted(RAGGED))
def test_compress_layer_ragged(batch, keep_window, shared):
    H, n_kv, prompts = RAGGED[batch]
    _compress_and_check(H, n_kv, prompts, keep_window, shared)


def _compress_and_check(H, n_kv, prompts, keep_window, shared):
    """One layer call over prompts (L, budget) against a stable sort of its scores."""
    dev, d, w = torch.device("cuda:0"), 64, 8
    gen = torch.Generator(device=dev).manual_seed(prompts[0][0])
    L = max(n for n, _ in prompts)
    q = torch.randn((H, w, d), generator=gen, device=dev).to(torch.float16)
    k, v = (torch.randn((n_kv, L, d), generator=gen, device=dev).to(torch.float16) for _ in range(2))
    flags = (ckv.CKV_KEEP_WINDOW if keep_window else 0) | (ckv.CKV_SHARE_LAYER if shared else 0)
    desc = ckv.layer_desc(H, n_kv, d, w, torch.float16, 0.0, ckv.CKV_POOL_MAX, 7, flags)
    mask = np.array([1] + [0] * (H // n_kv - 2) + [1] * (H > n_kv), np.uint8)
    mask = np.tile(mask, n_kv)
    tail = w if keep_window else 0
    seqs = []
    for n, b in prompts:  # one call, so that prompts and parts mix
        s = ckv.alloc_outputs(desc, ckv.Seq(q, k[:, L - n:], v[:, L - n:], b))
        s.scores = torch.empty((1 if shared else n_kv, n - tail), device=dev)
        seqs.append(s)
    print("case", H, prompts, keep_window, shared, flush=True)
    ckv.ckv_compress_layer(desc, mask, seqs, ckv.alloc_workspace(desc, seqs, dev))
    torch.cuda.synchronize()
    for (n, b), s in zip(prompts, seqs):
        sc, idx = s.scores.cpu().numpy(), s.idx.cpu().numpy().reshape(1 if shared else n_kv, -1)
        for g in range(n_kv):
            r = 0 if shared else g
            kept = min(b, n)
            want = np.arange(n) if kept == n else np.concatenate([_top(sc[r], kept - tail),
                                                                  np.arange(n - tail, n)])
            assert np.array_equal(idx[r], want), (n, b, g)
            at = torch.from_numpy(want).to(dev)
            assert torch.equal(s.k_out[g], s.k[g, at]) and torch.equal(s.v_out[g], s.v[g, at]), (n, b, g)
