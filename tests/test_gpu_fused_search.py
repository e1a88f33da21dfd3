"""Searches that run as one launch (small batches) against the same searches run stage by stage: id for id, relevance for
relevance, counter for counter.  Enabling the stage timing selects the separate kernels, whose parity with the oracle
the other tests hold.  Every case also says which path it takes: the queries that a workgroup runs to their end
are counted in the eighth word of the workspace's counters (at byte 256), those that waves are given in the ninth."""
import time

import pytest
import torch

import paper_2502_11490_amd as ann
from workloads import random_mlp

pytestmark = pytest.mark.gpu
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
ANN = {"f32": ann.ANN_F32, "bf16": ann.ANN_BF16, "f16": ann.ANN_F16}


def _handles(dtype, du, d, hidden, J, N, R, Q, E, seed=3):
    gen = torch.Generator().manual_seed(seed)
    Ws, bs = random_mlp([du + d, *hidden, J], 5, "bf16" if dtype == "bf16" else "f32", bias_scale=0.2)
    emb = torch.randn(N, d, generator=gen).to(TORCH[dtype])
    adj = torch.randint(0, N, (N, R), generator=gen, dtype=torch.int32)
    adj[::7, 0] = -1                      # padding, a repeated neighbour
    adj[::5, R - 1] = adj[::5, R // 2]
    users = torch.randn(Q, du, generator=gen).to(TORCH[dtype]).cuda()
    entries = torch.randint(0, N, (Q, E), generator=gen, dtype=torch.int32)
    entries[0, 0], entries[-1, E - 1] = -1, N
    entries[Q // 2, E - 1] = entries[Q // 2, 0]
    m = ann.ann_mlp_load([w.to(TORCH[dtype]) for w in Ws], bs, torch.rand(J, generator=gen), du, ANN[dtype])
    g = ann.ann_graph_load(adj.cuda(), emb.cuda())
    return g, m, users, entries.cuda()


def _ended_in_one_launch(ws):
    torch.cuda.synchronize()
    return int(ws[256:320].view(torch.int64)[7])


def _given_to_waves(ws):
    torch.cuda.synchronize()
    return int(ws[256:384].view(torch.int64)[8])


def _both(g, m, call, ws, path, overflow=None):
    """path: "one" = the whole batch in one launch, a workgroup a query, "staged" = no query, "tail" = the last ones, "waves" = the
    batch by waves (test_gpu_wave_search.py), the last ones of it perhaps by workgroups.  overflow: the arrays
    that a call writes which ends with ANN_EWORKSPACE (-5)."""
    runs = []
    for staged in (True, False):
        ann.ann_profile_enable(staged)
        try:
            if overflow is None:
                ids, sc = call()
            else:
                ids, sc = overflow
                ids.fill_(-7)
                with pytest.raises(ann.AnnError) as e:
                    call()
                assert e.value.code == -5 and "visited table" in str(e.value)
        finally:
            ann.ann_profile_enable(False)
        st = ann.ann_search_stats(ws)
        runs.append((ids.clone(), sc.clone(), (st.pairs_scored, st.nodes_expanded, st.max_query_iters, st.visited_overflow, st.queries)))
        ended = _ended_in_one_launch(ws)
        assert _given_to_waves(ws) == (st.queries if path == "waves" and not staged else 0)
        if staged or path == "staged":
            assert ended == 0
        elif path == "waves":
            assert ended <= 256
        else:
            assert ended == st.queries if path == "one" else 0 < ended < st.queries
    assert torch.equal(runs[0][0], runs[1][0])
    assert torch.equal(runs[0][1].view(torch.int32), runs[1][1].view(torch.int32))  # NaN too
    assert runs[0][2] == runs[1][2]
    return runs[0]


SHAPES = [("bf16", 64, 64, (256, 128), 3), ("f16", 128, 128, (512, 256), 4), ("bf16", 64, 64, (256,), 3),
          ("f32", 32, 32, (64,), 3), ("bf16", 13, 20, (48, 24, 16), 2), ("f32", 5, 7, (), 8)]
# candidates per round (of at most 256 queries) up to which one launch serves them: 110 million operations a CU over the
# metric's weights without the user's share of layer 1 in its built-in shapes, fp32 counted 32 times
MOST = {SHAPES[0]: 1110, SHAPES[1]: 278, SHAPES[2]: 3206, SHAPES[3]: 400, SHAPES[4]: 17449, SHAPES[5]: 17903}


@pytest.mark.parametrize("visited", ["hash", "bitmap", "rank"])
@pytest.mark.parametrize("dtype,du,d,hidden,J", SHAPES)
def test_one_launch_is_the_staged_search(dtype, du, d, hidden, J, visited, monkeypatch):
    """One query and a few; one candidate a round up to several pieces of the filter; more seeds than a piece; odd
    lists, k above and below L, lists longer than a workgroup; with and without a cap.  (So few items have a bit each in LDS whatever
    the form; test_gpu_fused_close.py and test_gpu_visited.py have larger tables.)  The widest metric and the fp32
    one take the staged path at 600 candidates and more, and one launch at the sizes just below their lines."""
    monkeypatch.setenv("GMPGR_VISITED_SET", "hash" if visited == "hash" else "bitmap")
    for Q, R, E, W, L, k, cap in [(1, 16, 1, 1, 1, 5, 0), (3, 1, 2, 1, 33, 7, 0), (65, 32, 3, 4, 257, 30, 0),
                                  (5, 24, 600, 2, 65, 100, 0), (2, 32, 1024, 9, 1500, 11, 0), (17, 17, 4, 37, 300, 20, 6),
                                  (5, 24, 278, 2, 65, 100, 0), (2, 32, 277, 8, 1500, 11, 0), (17, 17, 4, 16, 300, 20, 6)]:
        g, m, users, entries = _handles(dtype, du, d, hidden, J, 3001, R, Q, E)
        if visited == "rank":
            rank = torch.randperm(3001, generator=torch.Generator().manual_seed(1)).to(torch.int32).cuda()
            ann.ann_graph_set_locality(g, rank)
        ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, E, W, L, k, cap), dtype=torch.uint8, device="cuda")
        path = "one" if max(W * R, E) <= MOST[dtype, du, d, hidden, J] else "staged"
        _both(g, m, lambda: ann.ann_search(g, m, users, entries, W, L, k, cap, workspace=ws), ws, path)


@pytest.mark.parametrize("Q", [256, 257, 512, 513, 1024, 1025])
@pytest.mark.parametrize("dtype,du,d,hidden,J", [SHAPES[0], SHAPES[3]])
def test_batch_sizes_around_the_lines(dtype, du, d, hidden, J, Q):
    """Per-query widths, lists and caps, at the batch sizes where tile and workgroup change."""
    g, m, users, entries = _handles(dtype, du, d, hidden, J, 5000, 16, Q, 4)
    gen = torch.Generator().manual_seed(Q)
    own = [torch.randint(lo, hi, (Q,), generator=gen, dtype=torch.int32).cuda() for lo, hi in ((0, 10), (0, 140), (0, 30))]
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, 4, 8, 128, 20, 24), dtype=torch.uint8, device="cuda")
    _both(g, m, lambda: ann.ann_search_ragged(g, m, users, entries, *own, 8, 128, 20, 24, workspace=ws), ws,
          ("one" if Q == 256 else "waves") if dtype == "bf16" else "one" if Q <= 768 else "staged")


@pytest.mark.parametrize("dtype,du,d,hidden,J,Q,R,W", [
    (*SHAPES[0], 257, 16, 16), (*SHAPES[0], 512, 16, 16), (*SHAPES[0], 600, 20, 16), ("f16", *SHAPES[0][1:], 512, 31, 9),
    (*SHAPES[2], 512, 16, 16), (*SHAPES[2], 768, 16, 24), (*SHAPES[2], 1024, 16, 33), (*SHAPES[2], 1025, 16, 33)])
def test_wide_rounds_of_middle_batches(dtype, du, d, hidden, J, Q, R, W):
    """The metrics of 64-wide items beyond 256 queries, where rounds that are wide for the number of queries stay with a workgroup
    a query (tiles of one, two and four column blocks) instead of a wave."""
    g, m, users, entries = _handles(dtype, du, d, hidden, J, 5000, R, Q, 4)
    gen = torch.Generator().manual_seed(Q)
    own = [torch.randint(lo, hi, (Q,), generator=gen, dtype=torch.int32).cuda() for lo, hi in ((0, W + 3), (0, 140), (0, 30))]
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, 4, W, 128, 20, 24), dtype=torch.uint8, device="cuda")
    _both(g, m, lambda: ann.ann_search_ragged(g, m, users, entries, *own, W, 128, 20, 24, workspace=ws), ws,
          "one" if Q <= 1024 else "waves")


@pytest.mark.parametrize("dtype,du,d,hidden,J", SHAPES[:4])
def test_items_that_are_not_finite(dtype, du, d, hidden, J):
    """Infinities and NaN in the item table reach the same relevances on both paths."""
    g, m, users, entries = _handles(dtype, du, d, hidden, J, 400, 16, 9, 8)
    emb = torch.randn(400, d).to(TORCH[dtype])
    emb[::9, 1], emb[3::11, 0], emb[5::13, 2] = float("inf"), float("-inf"), float("nan")
    g = ann.ann_graph_load(torch.randint(0, 400, (400, 16), dtype=torch.int32).cuda(), emb.cuda())
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, 9, 8, 4, 64, 200, 0), dtype=torch.uint8, device="cuda")
    _both(g, m, lambda: ann.ann_search(g, m, users, entries, 4, 64, 200, 0, workspace=ws), ws, "one")


@pytest.mark.parametrize("visited", ["hash", "bitmap"])
@pytest.mark.parametrize("dtype,du,d,hidden,J", SHAPES[:4])
def test_last_queries_of_a_large_batch(dtype, du, d, hidden, J, visited, monkeypatch):
    """A batch too large for one launch ends in one: the list, the state and the survivors move over in the middle of
    the search.  Lists of very different lengths, so that a few queries run long after the others (the enqueuing thread
    is at most four rounds ahead of the device and sees that few are left); also through slots, where six of seven
    queries have no valid seed and end at once."""
    monkeypatch.setenv("GMPGR_VISITED_SET", visited)
    Q, R, E, W, L, k = 1400, 16, 3, 4, 301, 40
    g, m, users, entries = _handles(dtype, du, d, hidden, J, 4001, R, Q, E)
    own = [torch.full((Q,), W, dtype=torch.int32), torch.full((Q,), 9, dtype=torch.int32), torch.zeros(Q, dtype=torch.int32)]
    own[1][::11] = L
    own = [o.cuda() for o in own]
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, E, W, L, k, 0), dtype=torch.uint8, device="cuda")
    _both(g, m, lambda: ann.ann_search_ragged(g, m, users, entries, *own, W, L, k, 0, workspace=ws), ws,
          "waves" if d == 64 else "tail")
    few = entries.clone()
    few[torch.arange(Q, device="cuda") % 7 != 0] = -1
    for seeds in (entries, few):
        want = ann.ann_search(g, m, users, seeds, W, 60, k, 0)
        for slots in (1100, 70):
            ws = torch.empty(ann.ann_search_stream_workspace_bytes(g, m, Q, slots, E, W, 60, k, 0), dtype=torch.uint8, device="cuda")
            ids, sc = ann.ann_search_stream(g, m, users, seeds, slots, W, 60, k, workspace=ws)
            assert torch.equal(ids, want[0]) and torch.equal(sc, want[1])
            if seeds is few or slots == 70:
                assert 0 < _ended_in_one_launch(ws) < Q


def slow_rounds():
    """A search of one query with slow rounds: 64 nodes a layer, each joined to one of the next layer and to 63 items of its own,
    so that every round brings 4,096 new pairs; an fp32 metric of eight layers, whose passes over 64 pairs wait for each other
    at every layer.  Relevance grows from layer to layer, the other items have the least."""
    R, W, layers = 64, 64, 60
    N = layers * W * R
    i = torch.arange(N, device="cuda").view(layers, W, R)
    adj = torch.full((layers, W, R, R), -1, dtype=torch.int32, device="cuda")
    adj[:-1, :, 0, 0] = i[1:, :, 0]
    adj[:, :, 0, 1:] = i[:, :, 1:]
    emb = torch.zeros(layers, W, R, 1, device="cuda")
    emb[:, :, 0, 0] = torch.linspace(0.5, 3, layers * W, device="cuda").view(layers, W)
    first = torch.zeros(7, 2)
    first[0, 1] = 1
    between = torch.eye(7)
    Ws = [first] + [between.clone() for _ in range(6)] + [between[:1].clone()]
    m = ann.ann_mlp_load(Ws, [torch.zeros(7) for _ in range(7)] + [torch.zeros(1)], torch.ones(1), 1, ann.ANN_F32)
    return ann.ann_graph_load(adj.view(N, R), emb.view(N, 1)), m, torch.zeros(1, 1, device="cuda"), i[:1, :, 0].int().contiguous(), W, layers


def test_a_search_in_one_launch_reports_its_progress():
    """60 rounds of one query, 0.5 ms each, under a limit far below the 20 ms after which the waiting thread asks: the kernel
    reports often enough (every eighth round) for the call to see that it goes on.  One report in 64 rounds would not do."""
    g, m, users, entries, W, layers = slow_rounds()
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, 1, W, W, W, W, 0), dtype=torch.uint8, device="cuda")
    want = ann.ann_search(g, m, users, entries, W, W, W, 0, workspace=ws)
    assert ann.ann_search_stats(ws).max_query_iters == layers and _ended_in_one_launch(ws) == 1
    start = time.perf_counter()
    ann.ann_search(g, m, users, entries, W, W, W, 0, workspace=ws)
    torch.cuda.synchronize()
    assert time.perf_counter() - start > 0.025
    ann.ann_set_progress_timeout(1e-3)
    try:
        got = ann.ann_search(g, m, users, entries, W, W, W, 0, workspace=ws)
    finally:
        ann.ann_set_progress_timeout(600.0)
        torch.cuda.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def _rising(dtype, N, R, Q):
    """Items whose relevance rises with their id, every item joined to the next R: a search with a list of one entry goes
    on to the last item and scores all of them.  id / 64 and id % 64 are the item's two coordinates (exact in 16 bits)."""
    i = torch.arange(N, device="cuda")
    emb = torch.stack([(i // 64).float(), (i % 64).float()], 1).to(TORCH[dtype])
    adj = i[:, None] + 1 + torch.arange(R, device="cuda")
    adj = torch.where(adj < N, adj, -1).int()
    w = torch.tensor([[0.0, 2.0 ** -4, 2.0 ** -10]]).to(TORCH[dtype])
    m = ann.ann_mlp_load([w], [torch.tensor([-4.0])], torch.ones(1), 1, ANN[dtype])
    return ann.ann_graph_load(adj, emb), m, torch.zeros(Q, 1, device="cuda").to(TORCH[dtype])


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("Q", [5, 1400])
def test_visited_table_that_fills_up(dtype, Q, monkeypatch):
    """A table of 2,048 slots (34 assumed rounds of 16 ids) takes 1,024 ids: queries that start far from the last item stop
    when it is full, in the one launch of a small batch, in the one that ends a large batch, and in a slot that the next
    query takes.  Same error, results and counters as stage by stage."""
    monkeypatch.setenv("GMPGR_VISITED_SET", "hash")
    N, R, k = 8000, 16, 3
    g, m, users = _rising(dtype, N, R, Q)
    start = torch.full((Q,), N - 30, dtype=torch.int32)        # two rounds to the last item ...
    if Q == 5:
        start[:4] = torch.tensor([0, N - 1010, N - 1009, N - 1008])
    else:
        start[::10] = torch.linspace(0, N - 100, Q // 10).int()
    entries = start[:, None].contiguous().cuda()
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, 1, 1, 1, k, 0), dtype=torch.uint8, device="cuda")
    out = torch.empty(Q, k, dtype=torch.int32, device="cuda"), torch.empty(Q, k, device="cuda")
    call = lambda: ann.ann_search(g, m, users, entries, 1, 1, k, 0, workspace=ws, out_ids=out[0], out_scores=out[1])
    ids, sc, counters = _both(g, m, call, ws, "one" if Q == 5 else "tail", overflow=out)
    # 16 ids a round: 1 + 16 * 63 fit, 16 more do not
    assert torch.equal(ids[:, 0].cpu(), (start + 16 * 63).clamp(max=N - 1))
    assert counters[3] == int((start + 16 * 63 <= N - 1).sum()) > 0
    if Q > 5:
        ws = torch.empty(ann.ann_search_stream_workspace_bytes(g, m, Q, 300, 1, 1, 1, k, 0), dtype=torch.uint8, device="cuda")
        call = lambda: ann.ann_search_stream(g, m, users, entries, 300, 1, 1, k, workspace=ws, out_ids=out[0], out_scores=out[1])
        streamed = _both(g, m, call, ws, "tail", overflow=out)
        assert torch.equal(streamed[0], ids) and torch.equal(streamed[1], sc) and streamed[2] == counters
