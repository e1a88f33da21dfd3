"""Searches in one launch of a batch that gives every query a CU: weights in registers or LDS, visited set in LDS.  A table of
200,000 items, too large for one bit per item there, so a hash table begins there and a bitmap, by id or by rank, is in
memory; the same searches run stage by stage are the reference (id for id, relevance for relevance, counter for
counter)."""
import pytest
import torch

import paper_2502_11490_amd as ann
from test_gpu_fused_search import _both, _handles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("visited", ["hash", "bitmap", "rank"])
@pytest.mark.parametrize("dtype,du,d,hidden,J", [
    ("bf16", 64, 64, (256, 128), 3), ("f16", 7, 64, (256, 128), 8), ("bf16", 64, 64, (256,), 1), ("f16", 64, 64, (256,), 4),
    ("bf16", 128, 128, (512, 256), 4), ("bf16", 80, 96, (192, 96), 2), ("f16", 30, 26, (40,), 3), ("f32", 32, 32, (64,), 3)])
@pytest.mark.parametrize("Q,R,E,W,L,k,cap", [
    (2, 32, 4, 4, 700, 50, 0),    # some 15,000 ids a query: the visited set moves from LDS to memory
    (3, 31, 1, 1, 40, 7, 0),      # fewer pairs than a column block of 32
    (1, 33, 4, 4, 300, 9, 0),     # 132 candidates a round: up to a pass of 128 pairs, and a few in a second one
    (256, 32, 2, 2, 30, 40, 0),   # the most queries; up to two column blocks
    (5, 32, 70, 3, 90, 10, 0),    # three column blocks
    (3, 32, 270, 1, 400, 9, 0),   # one and two parents a round among more entries than a wave has lanes
    (2, 33, 4, 2, 300, 9, 0),
    (4, 48, 200, 5, 120, 30, 25)])
def test_one_launch_close_to_its_data(dtype, du, d, hidden, J, Q, R, E, W, L, k, cap, visited, monkeypatch):
    monkeypatch.setenv("GMPGR_VISITED_SET", "hash" if visited == "hash" else "bitmap")
    g, m, users, entries = _handles(dtype, du, d, hidden, J, 200_000, R, Q, E)
    if visited == "rank":
        ann.ann_graph_set_locality(g, torch.randperm(200_000, generator=torch.Generator().manual_seed(1)).to(torch.int32).cuda())
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, E, W, L, k, cap), dtype=torch.uint8, device="cuda")
    _both(g, m, lambda: ann.ann_search(g, m, users, entries, W, L, k, cap, workspace=ws), ws, "one")
