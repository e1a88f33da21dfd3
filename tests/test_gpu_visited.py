"""The visited table where its slots collide: all ids of the graph have their home among the last slots of the table, so that
every id but a few walks past the table's end and along one run of taken slots, and every neighbour comes in several rows of
a round.  Same results as with the bitmap, which has neither, and as the oracle's.  The graph has more items than get one bit
each in the LDS of a search in one launch, whose table is there from 2,048 slots on, up to 8,192 or what the list leaves
room for; the last case outgrows that table and goes on in memory."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_11490_amd as ann
from workloads import random_mlp

pytestmark = pytest.mark.gpu


def _paths(ws):
    """Queries that a workgroup, and that waves ran (the eighth and ninth word of the counters)."""
    torch.cuda.synchronize()
    return ws[256:384].view(torch.int64)[7:9].tolist()


# tables of 192, 640, 4,480 and 9,600 slots (the last: 4,096 in LDS beside a list of 5,500; moved with 2,000 ids in it)
@pytest.mark.parametrize("W,cap,E,L,homes", [(1, 3, 1, 64, 3), (4, 3, 40, 64, 3), (40, 2, 300, 64, 3), (40, 2, 300, 64, 100),
                                             (40, 6, 300, 5500, 275)])
@pytest.mark.parametrize("staged", [True, False])
@pytest.mark.parametrize("Q", [3, 2100])
def test_ids_that_share_their_slots(W, cap, E, L, homes, staged, Q, monkeypatch):
    N, R, k, d = 140_001, 16, 30, 64
    slots = -(-2 * (E + cap * W * R + W * R) // 64) * 64
    h = (torch.arange(N) * 0x9E3779B1) & 0xFFFFFFFF
    ids = torch.nonzero(h >= (1 << 32) - homes * (1 << 32) // slots)[:, 0]
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
            ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, E, W, L, k, cap), dtype=torch.uint8, device="cuda")
            runs.append(ann.ann_search(g, m, users.cuda(), entries.cuda(), W, L, k, cap, workspace=ws))
            by_groups, by_waves = _paths(ws)
            assert by_groups == (Q if Q == 3 and not staged else 0)
            assert by_waves == (Q if Q > 3 and L == 64 and not staged else 0)
        finally:
            ann.ann_profile_enable(False)
    assert torch.equal(runs[0][0], runs[1][0]) and torch.equal(runs[0][1], runs[1][1])
    mlp = oracle.Mlp([w.float().numpy() for w in Ws], [b.numpy() for b in bs], hw.numpy())
    ref = oracle.search(emb.float().numpy(), adj.numpy(), users[:3].float().numpy(), mlp, entries[:3].numpy(), W, L, k, cap,
                        n_threads=4, act_round=1)
    got = runs[0][0][:3].cpu().numpy()
    assert np.mean(got == ref["ids"]) >= 0.9  # neighbours in a list change places where an activation rounds the other way
