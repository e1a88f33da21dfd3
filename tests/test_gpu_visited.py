"""The visited table where its slots collide: all ids of the graph have their home among the last slots of the table, so that
every id but a few walks past the table's end and along one run of taken slots, and every neighbour comes in several rows of
a round.  Same results as with the bitmap, which has neither, and as the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_11490_amd as ann
from workloads import random_mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,cap,E", [(1, 3, 1), (4, 3, 40), (40, 2, 300)])  # tables of 160, 576 and 6,496 slots at most
@pytest.mark.parametrize("staged", [True, False])
@pytest.mark.parametrize("Q", [3, 2100])
def test_ids_that_share_their_slots(W, cap, E, staged, Q, monkeypatch):
    N, R, L, k, d = 1 << 17, 16, 64, 30, 64
    slots = 2 * (E + cap * W * R + W * R)
    h = (torch.arange(N) * 0x9E3779B1) & 0xFFFFFFFF
    ids = torch.nonzero(h >= (1 << 32) - 3 * (1 << 32) // slots)[:, 0]
    assert len(ids) > 40
    gen = torch.Generator().manual_seed(W)
    adj = ids[torch.randint(0, len(ids), (N, R), generator=gen)].int()
    entries = ids[torch.randint(0, len(ids), (Q, E), generator=gen)].int()
    emb = torch.randn(N, d, generator=gen).bfloat16()
    users = torch.randn(Q, d, generator=gen).bfloat16()
    Ws, bs = random_mlp([2 * d, 256, 3], 5, "bf16", bias_scale=0.2)
    Ws, hw = [w.bfloat16() for w in Ws], torch.tensor([0.5, 0.3, 0.2])
    runs = []
    for form in ("hash", "bitmap"):
        monkeypatch.setenv("GMPGR_VISITED_SET", form)
        g = ann.ann_graph_load(adj.cuda(), emb.cuda())
        m = ann.ann_mlp_load(Ws, bs, hw, d, ann.ANN_BF16)
        ann.ann_profile_enable(staged)
        try:
            runs.append(ann.ann_search(g, m, users.cuda(), entries.cuda(), W, L, k, cap))
            torch.cuda.synchronize()
        finally:
            ann.ann_profile_enable(False)
    assert torch.equal(runs[0][0], runs[1][0]) and torch.equal(runs[0][1], runs[1][1])
    mlp = oracle.Mlp([w.float().numpy() for w in Ws], [b.numpy() for b in bs], hw.numpy())
    ref = oracle.search(emb.float().numpy(), adj.numpy(), users[:3].float().numpy(), mlp, entries[:3].numpy(), W, L, k, cap,
                        n_threads=4, act_round=1)
    got = runs[0][0][:3].cpu().numpy()
    assert np.mean(got == ref["ids"]) >= 0.9  # neighbours in a list change places where an activation rounds the other way
