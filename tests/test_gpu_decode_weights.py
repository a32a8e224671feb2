"""The weights of decode attention where their rounding shows: maxima that move
often beside large ones that stay, and weights below the smallest normal fp32
number.

Logits are products of single entries (query row r holds one nonzero element),
so they are exact and the tolerances are those of the sums alone.
"""
import math

import numpy as np
import pytest
import torch

import paper_2508_02401_amd as ckv

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24  # half a unit in the last place of fp32
# what the high and low parts of a probability leave out of it
SPLIT = {torch.bfloat16: 2.0 ** -17, torch.float16: 2.0 ** -22, torch.float32: 0.0}


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("G", [32, 64])
def test_rows_whose_maximum_stays(dtype, G):
    """Rows of equal logits (100 to 255, natural units) beside four rows whose
    maximum moves at every tile: their result is the plain mean of V.

    All weights of such a row are one number, so what may differ is the fp32
    sums: a wave adds its 256 tiles of 32 keys one by one, to the weighted V
    and to the sum of weights, and 4 waves meet: (256 + 32 + 4) roundings each,
    and the split of the weights (16-bit types)."""
    dev, d, n, n_kv, prompts = torch.device("cuda:0"), 64, 32768, 32, 16
    tiles = n // 32
    q = torch.zeros((1, n_kv, G, d))
    k = torch.zeros((n, d))
    tile = torch.arange(n) // 32
    for r in range(G):
        if r < 4:  # climbs over its quarter of the tiles
            q[:, :, r, r] = 1.0
            k[:, r] = (tile - r * tiles // 4).clamp(0, 255).float()
        else:      # logit 8 * k / sqrt(64) = k
            q[:, :, r, r] = 8.0
            k[:, r] = float(255 - (r - 4) * 155 // (G - 4))
    at = torch.arange(1, d + 1) * n // (d + 1)
    v = (torch.arange(n)[:, None] < at[None, :]).float()  # column c: 1 up to key at[c]
    qd = q.view(1, n_kv * G, d).to(dtype).to(dev)
    kd, vd = (x.to(dtype).to(dev).unsqueeze(0).expand(n_kv, n, d) for x in (k, v))
    desc = ckv.attn_desc(n_kv * G, n_kv, d, dtype)
    outs = [torch.full((1, n_kv * G, d), math.nan, device=dev) for _ in range(prompts)]
    seqs = [ckv.decode_seq(qd, ckv.kv_cache(kd, vd), o) for o in outs]
    ws = torch.empty(ckv.ckv_decode_batch_workspace_bytes(desc, seqs), dtype=torch.uint8, device=dev)
    print("case", dtype, G, flush=True)
    ckv.ckv_decode_attention_batch(desc, seqs, ws)
    torch.cuda.synchronize()
    z = (q[0, 0].double() @ k.double().t()) / math.sqrt(d)
    ref = (z.softmax(dim=1) @ v.double()).numpy()
    got = np.stack([o.view(n_kv, G, d).cpu().double().numpy() for o in outs])
    err = np.abs(got[:, :, 4:] - ref[None, None, 4:]).max()
    tol = 2 * (256 + 32 + 4) * EPS + SPLIT[dtype]
    assert err <= tol, "max err %.3g, bound %.3g" % (err, tol)


@pytest.mark.parametrize("G", [1, 40])
@pytest.mark.parametrize("where", ["tile", "later tile"])
def test_fp32_weights_below_the_normal_range(G, where):
    """fp32 caches: a weight of 2^-130 of the largest still counts where V is large.

    32 keys weigh 2^-130, a subnormal number with 19 bits left, with V = 2^120;
    the keys of the largest weight have V = 0 and share the small ones' tile of
    32, or come up to four tiles later, when the sums so far are rescaled (512 KV
    heads keep the 160 keys in one chunk, tiles 0 and 4 with one wave)."""
    dev, d, n_kv = torch.device("cuda:0"), 64, 512
    n = 32 if where == "tile" else 160
    small = slice(1, 32) if where == "tile" else slice(0, 32)
    q = torch.zeros((1, n_kv * G, d), device=dev)
    q[:, :, 0] = 8.0
    k, v = torch.zeros((n, d), device=dev), torch.zeros((n, d), device=dev)
    k[:, 0] = 130.0 * math.log(2.0)
    k[small, 0] = 0.0
    v[small] = 2.0 ** 120
    kd, vd = (x.unsqueeze(0).expand(n_kv, n, d) for x in (k, v))
    desc = ckv.attn_desc(n_kv * G, n_kv, d, torch.float32)
    out = torch.full((1, n_kv * G, d), math.nan, device=dev)
    ws = torch.empty(ckv.ckv_decode_workspace_bytes(desc, 1, n), dtype=torch.uint8, device=dev)
    print("case", G, where, flush=True)
    ckv.ckv_decode_attention(desc, q, ckv.kv_cache(kd, vd), out, ws)
    torch.cuda.synchronize()
    ref = float(((k[:, 0].double()).softmax(dim=0) @ v.double())[0])
    # the exponent 130 is rounded to 2^-23 of itself in all (alpha, the maximum),
    # 1.1e-5 of a weight, which keeps 19 bits: 1e-6
    rel = (out.double() / ref - 1).abs().max().item()
    assert rel <= 2e-5, "relative error %.3g" % rel
