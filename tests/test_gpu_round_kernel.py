"""Which build of the round kernel a batch runs (workgroup, visited set, list in LDS, visited filter: its template arguments, read
from a captured call) on either side of the lines, and that the builds agree."""
import re

import pytest
import torch

import paper_2502_11490_amd as ann
from gpu_util import captured_kernels
from workloads import random_mlp

pytestmark = pytest.mark.gpu
WALKERS = 2


def _handles(N, R, Q, E, f8=False):
    gen = torch.Generator().manual_seed(N + R)
    dims = [128, 512, 256, 2] if f8 else [64, 32, 2]
    d = dims[0] // 2
    Ws, bs = random_mlp(dims, 5, "bf16", bias_scale=0.2)
    emb = torch.randn(N, d, generator=gen).bfloat16().cuda()
    adj = torch.randint(-1, N, (N, R), generator=gen, dtype=torch.int32)
    adj[::5, R - 1] = adj[::5, R // 2]
    m = ann.ann_mlp_load([w.bfloat16() for w in Ws], bs, torch.rand(2, generator=gen), d, ann.ANN_F8 if f8 else ann.ANN_BF16)
    g = ann.ann_graph_load(adj.cuda(), ann.ann_quantize_e4m3(emb) if f8 else emb)
    users = torch.randn(Q, d, generator=gen).bfloat16().cuda()
    return g, m, users, torch.randint(0, N, (Q, E), generator=gen, dtype=torch.int32).cuda()


def _round_kernel(call):
    """(threads, bitmap, list resident, filter)"""
    found = {tuple(int(x) for x in t.groups()) for name, _, _ in captured_kernels(call)
             if (t := re.search(r"round_kernelILi(\d+)ELb([01])ELb([01])ELi(\d)E", name))}
    assert len(found) == 1, found
    return found.pop()


@pytest.mark.parametrize("visited", ["hash", "bitmap"])
@pytest.mark.parametrize("Q,R,E,k,threads", [(8192, 32, 4, 100, 128), (8191, 32, 4, 100, 256), (8192, 32, 4, 768, 128),
                                             (8192, 32, 4, 769, 256), (8192, 33, 4, 100, 256), (8192, 1, 1, 5, 128)])
def test_walkers_of_a_large_batch(Q, R, E, k, threads, visited, monkeypatch):
    monkeypatch.setenv("GMPGR_VISITED_SET", visited)
    g, m, users, entries = _handles(3001, R, Q, E)
    ws = torch.empty(ann.ann_search_walkers_workspace_bytes(g, m, Q, E, 6, k), dtype=torch.uint8, device="cuda")
    out = dict(out_ids=torch.empty(Q, k, dtype=torch.int32, device="cuda"), out_scores=torch.empty(Q, k, device="cuda"))
    call = lambda: ann.ann_search_walkers(g, m, users, entries, 6, k, workspace=ws, **out)
    call()
    ids, sc = out["out_ids"].clone(), out["out_scores"].clone()
    assert _round_kernel(call) == (threads, int(visited == "bitmap"), 1, WALKERS)
    few = ann.ann_search_walkers(g, m, users[:64].contiguous(), entries[:64].contiguous(), 6, k)
    assert torch.equal(ids[:64], few[0]) and torch.equal(sc[:64], few[1])
