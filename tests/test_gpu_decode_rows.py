"""Decode attention at the edges of its kernels' ranges: the query rows where
the kernel changes (32 and 64 rows per KV head) or a row block is partial, and
cache lengths around a tile (32 keys), a wave round (128 keys) and several
chunks, in one ragged batch, against the fp64 oracle.

Tolerance: |gpu - oracle| <= 1e-4 * (|oracle| + 1), as for every decode test:
fp32 sums over inputs that are exact in fp32.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2508_02401_amd as ckv

pytestmark = pytest.mark.gpu

LENS = [1, 31, 32, 33, 127, 128, 129, 515, 4100]


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.float16, 64),
                                     (torch.float16, 128), (torch.float32, 128), (torch.float32, 64)])
@pytest.mark.parametrize("G,T", [(7, 1), (31, 1), (8, 4), (11, 3), (16, 4), (13, 5), (16, 8)])
def test_decode_rows_and_lengths(dtype, d, G, T):
    dev, n_kv = torch.device("cuda:0"), 2
    H = n_kv * G
    gen = torch.Generator().manual_seed(G * 100 + T)
    desc = ckv.attn_desc(H, n_kv, d, dtype)
    seqs, held = [], []
    for i, n in enumerate(LENS):
        # the cache is the middle of a buffer whose other rows hold NaN: a row
        # past the cache that counted would show
        buf = torch.full((2, n_kv, n + 40, d), math.nan)
        kv = torch.randn((2, n_kv, n, d), generator=gen)
        buf[:, :, 3:3 + n] = kv
        buf = buf.to(dtype).to(dev)
        t = T if i != 2 else 1  # prompts of one batch may differ in T
        q = (torch.randn((t, H, d), generator=gen) * 1.5).to(dtype)
        out = torch.full((t, H, d), math.nan, device=dev)
        qd = q.to(dev)
        seqs.append(ckv.decode_seq(qd, ckv.kv_cache(buf[0, :, 3:3 + n], buf[1, :, 3:3 + n]), out))
        held.append((q, kv.to(dtype), out, buf, qd))
    ws = torch.empty(ckv.ckv_decode_batch_workspace_bytes(desc, seqs), dtype=torch.uint8, device=dev)
    print("case", dtype, d, G, T, flush=True)
    ckv.ckv_decode_attention_batch(desc, seqs, ws)
    torch.cuda.synchronize()
    for n, (q, kv, out, _, _) in zip(LENS, held):
        qd, kd, vd = q.double().numpy(), kv[0].double().numpy(), kv[1].double().numpy()
        ref = np.stack([oracle.decode_attention(qd[t], kd, vd, 1.0 / math.sqrt(d))
                        for t in range(q.shape[0])])
        err = np.abs(out.cpu().numpy() - ref)
        assert np.all(err <= 1e-4 * (np.abs(ref) + 1.0)), "n %d: max err %.3g" % (n, err.max())
