"""ckv_set_stage_events: after a layer call or ckv_select every event of the stages it
runs has been recorded by that call, whichever launches it took."""
import numpy as np
import pytest
import torch

import paper_2508_02401_amd as ckv

pytestmark = pytest.mark.gpu

STAGES = {"layer": (0, 1, 2, 3, 4), "select": (3, 4)}


@pytest.mark.parametrize("entry", ["layer", "select"])
@pytest.mark.parametrize("L", [1000, 40000, 66000])  # on both sides of the one-launch selection's limits
def test_every_pair_is_recorded(entry, L):
    dev, H, n_kv, d, w = torch.device("cuda:0"), 4, 2, 64, 8
    gen = torch.Generator(device=dev).manual_seed(L)
    q = torch.randn((H, w, d), generator=gen, device=dev).to(torch.bfloat16)
    k, v = (torch.randn((n_kv, L, d), generator=gen, device=dev).to(torch.bfloat16) for _ in range(2))
    desc = ckv.layer_desc(H, n_kv, d, w, torch.bfloat16)
    s = ckv.alloc_outputs(desc, ckv.Seq(q, k, v, 300))
    s.scores = torch.rand((n_kv, L - w), generator=gen, device=dev)
    ws = ckv.alloc_workspace(desc, [s], dev)
    begin, end = ([torch.cuda.Event(enable_timing=True) for _ in range(ckv.CKV_NUM_STAGES)]
                  for _ in range(2))
    for e in begin + end:
        e.record()  # creates the event
    torch.cuda.synchronize()
    mark = torch.cuda.Event(enable_timing=True)
    mark.record()
    print("case", entry, L, flush=True)
    ckv.ckv_set_stage_events([e.cuda_event for e in begin], [e.cuda_event for e in end])
    try:
        if entry == "layer":
            ckv.ckv_compress_layer(desc, np.array([1, 0, 0, 1], np.uint8), [s], ws)
        else:
            ckv.ckv_select(desc, [s], ws)
    finally:
        ckv.ckv_set_stage_events(None, None)
    torch.cuda.synchronize()
    last = 0.0
    for st in STAGES[entry]:
        b, e = mark.elapsed_time(begin[st]), mark.elapsed_time(end[st])
        # not the event's first record, before the mark, and in the stages' order
        assert last <= b <= e, "stage %d: %.4f to %.4f ms, the stage before ended at %.4f" % (st, b, e, last)
        last = e
