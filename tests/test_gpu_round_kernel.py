"""Which build of the round kernel a batch runs (workgroup, visited set, list in LDS, visited filter: its template arguments, read
from a captured call) on either side of the lines, and that the builds agree."""
import re

import pytest
import torch

import paper_2502_11490_amd as ann
from gpu_util import captured_kernels
from workloads import random_mlp

pytestmark = pytest.mark.gpu
ATOMIC, ORDERED, WALKERS = 0, 1, 2


def _handles(N, R, Q, E, f8=False):
    gen = torch.Generator().manual_seed(N + R)
    dims = [256, 512, 256, 2] if f8 else [64, 32, 2]
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
    found = {tuple(int(x) for x in t.groups()) for name, *_ in captured_kernels(call)
             if (t := re.search(r"round_kernelILi(\d+)ELb([01])ELb([01])ELi(\d)E", name))}
    assert len(found) == 1, found
    return found.pop()


def _seeds_by_eight_waves(call):
    """The seeding kernel leaves room for eight waves a SIMD (64 registers a lane) and keeps nothing in scratch memory."""
    (registers, scratch), = {k[3:] for k in captured_kernels(call) if "init_kernel" in k[0]}
    assert 0 < registers <= 64 and scratch == 0


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
    _seeds_by_eight_waves(call)
    few = ann.ann_search_walkers(g, m, users[:64].contiguous(), entries[:64].contiguous(), 6, k)
    assert torch.equal(ids[:64], few[0]) and torch.equal(sc[:64], few[1])


@pytest.mark.parametrize("Q,R,W,L,ranked,threads,which", [
    (4096, 32, 4, 100, False, 256, ATOMIC), (4096, 43, 3, 100, False, 256, ORDERED), (1024, 32, 11, 100, True, 256, ATOMIC),
    (1024, 32, 12, 100, True, 256, ORDERED), (256, 32, 64, 300, False, 512, ATOMIC), (257, 32, 64, 300, False, 512, ORDERED),
    (1024, 32, 16, 1024, False, 256, ORDERED), (1024, 32, 16, 1024, True, 256, ORDERED), (1024, 32, 16, 1500, True, 256, ATOMIC),
    (1024, 32, 16, 1500, False, 256, ORDERED), (1024, 32, 17, 300, True, 512, ORDERED), (1024, 32, 32, 1500, False, 512, ORDERED),
    (1024, 32, 33, 300, True, 512, ORDERED), (8192, 32, 2, 60, False, 128, ATOMIC), (8192, 13, 5, 60, True, 128, ORDERED)])
def test_visited_filter_on_a_bitmap(Q, R, W, L, ranked, threads, which, monkeypatch):
    """On either side of the lines; the searches with the hash table, which always takes the atomics, are the reference."""
    N, E, k, cap = 4001, 5, 50, 12
    g, m, users, entries = _handles(N, R, Q, E, f8=True)
    out = dict(out_ids=torch.empty(Q, k, dtype=torch.int32, device="cuda"), out_scores=torch.empty(Q, k, device="cuda"))
    found = []
    for form in ("hash", "bitmap"):
        monkeypatch.setenv("GMPGR_VISITED_SET", form)
        if ranked and form == "bitmap":
            ann.ann_graph_set_locality(g, torch.randperm(N, generator=torch.Generator().manual_seed(1)).to(torch.int32).cuda())
        ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, E, W, L, k, cap), dtype=torch.uint8, device="cuda")
        call = lambda: ann.ann_search(g, m, users, entries, W, L, k, cap, workspace=ws, **out)
        call()
        found.append((out["out_ids"].clone(), out["out_scores"].clone()))
        _seeds_by_eight_waves(call)
        t, bitmap, _, picked = _round_kernel(call)
        assert (t, bitmap, picked) == (threads, int(form == "bitmap"), which if form == "bitmap" else ATOMIC)
    assert torch.equal(found[0][0], found[1][0]) and torch.equal(found[0][1], found[1][1])
