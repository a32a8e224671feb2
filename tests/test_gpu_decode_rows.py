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


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_few_rows_keep_their_kernel_beside_many(dtype):
    """A batch of one-token prompts and of prompts of more than 64 query rows per KV
    head, the former with 2 * 150000 keys, enough to be launched apart: each kind is
    launched as it is without the other, so the results are the same bit for bit."""
    dev, n_kv, G, d = torch.device("cuda:0"), 2, 7, 128
    H = n_kv * G
    gen = torch.Generator(device=dev).manual_seed(3)
    desc = ckv.attn_desc(H, n_kv, d, dtype)
    prompts = []
    for n, T in [(700, 1), (3000, 16), (129, 1), (5000, 10), (150000, 1)]:
        q = (torch.randn((T, H, d), generator=gen, device=dev) * 1.5).to(dtype)
        k, v = (torch.randn((n_kv, n, d), generator=gen, device=dev).to(dtype) for _ in range(2))
        prompts.append((q, k, v))

    def run(some):
        outs = [torch.full(q.shape, math.nan, device=dev) for q, _, _ in some]
        seqs = [ckv.decode_seq(q, ckv.kv_cache(k, v), o) for (q, k, v), o in zip(some, outs)]
        ws = torch.empty(ckv.ckv_decode_batch_workspace_bytes(desc, seqs), dtype=torch.uint8, device=dev)
        ckv.ckv_decode_attention_batch(desc, seqs, ws)
        torch.cuda.synchronize()
        return outs

    print("case", dtype, flush=True)
    both = run(prompts)
    for which in ([0, 2, 4], [1, 3]):
        for i, o in zip(which, run([prompts[i] for i in which])):
            assert torch.equal(both[i], o), i
