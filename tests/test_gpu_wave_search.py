"""Searches run by waves that take one query after the other (metrics with items of 64 and 256 hidden units, batches
beyond what a workgroup per query is best at) against the same searches run stage by stage: id for id, relevance for
relevance, counter for counter.  Enabling the stage timing selects the separate kernels.  The ninth word of the workspace's
counters (at byte 256) says how many queries such a launch was given."""
import time

import pytest
import torch

import paper_2502_11490_amd as ann
from test_gpu_fused_search import _handles

pytestmark = pytest.mark.gpu
TWO, ONE = (64, 64, (256, 128), 3), (64, 64, (256,), 4)


def _both(call, ws, waves=True):
    runs = []
    for staged in (True, False):
        ann.ann_profile_enable(staged)
        try:
            ids, sc = call()
        finally:
            ann.ann_profile_enable(False)
        st = ann.ann_search_stats(ws)
        runs.append((ids.clone(), sc.clone(), (st.pairs_scored, st.nodes_expanded, st.max_query_iters, st.visited_overflow, st.queries)))
        ended, given = ws[256:384].view(torch.int64)[7:9].tolist()
        assert given == (st.queries if waves and not staged else 0)
        assert not waves or ended <= (0 if staged else 256)  # by workgroups: at most those that were handed over
    assert torch.equal(runs[0][0], runs[1][0])
    assert torch.equal(runs[0][1].view(torch.int32), runs[1][1].view(torch.int32))  # NaN too
    assert runs[0][2] == runs[1][2]
    return runs[1]


@pytest.mark.parametrize("visited", ["hash", "bitmap", "rank"])
@pytest.mark.parametrize("dtype,shape", [("bf16", TWO), ("f16", TWO), ("bf16", ONE), ("f16", ONE)])
def test_search_by_waves_is_the_staged_search(dtype, shape, visited, monkeypatch):
    """Fewer and more queries than waves of the launch, one more than a multiple of a CU's; one neighbour an item; rounds of
    one candidate, of a number that is no multiple of a wave, of one and several pieces of 128 and 256; lists of one entry
    and lists that leave room for one to sixteen waves a CU; k above and below L; more seeds than candidates; with
    and without a cap."""
    monkeypatch.setenv("GMPGR_VISITED_SET", "hash" if visited == "hash" else "bitmap")
    for Q, R, E, W, L, k, cap in [(2048, 32, 4, 4, 64, 100, 0), (2049, 16, 1, 1, 1, 5, 0), (2100, 1, 2, 3, 33, 7, 0),
                                  (4097, 24, 3, 5, 100, 20, 0), (2050, 32, 300, 9, 200, 11, 0), (2048, 32, 2, 12, 250, 40, 9),
                                  (9000, 17, 4, 2, 40, 10, 7), (2048, 16, 4, 4, 900, 30, 0), (2040, 16, 1024, 4, 2500, 30, 0),
                                  (300, 16, 1024, 1, 6690, 30, 0),
                                  (1025, 32, 4, 4, 64, 100, 0), (1300, 16, 4, 16, 500, 30, 6), (300, 32, 4, 4, 64, 100, 0), (777, 8, 5, 7, 131, 9, 0), (1024, 32, 4, 16, 300, 50, 5)]:
        g, m, users, entries = _handles(dtype, *shape, 3001, R, Q, E)
        if visited == "rank":
            rank = torch.randperm(3001, generator=torch.Generator().manual_seed(1)).to(torch.int32).cuda()
            ann.ann_graph_set_locality(g, rank)
        ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, E, W, L, k, cap), dtype=torch.uint8, device="cuda")
        _both(lambda: ann.ann_search(g, m, users, entries, W, L, k, cap, workspace=ws), ws)


@pytest.mark.parametrize("shape,Q,W,L,cap,waves", [
    (TWO, 8192, 4, 1024, 0, True), (TWO, 8192, 4, 1500, 0, False), (TWO, 2048, 4, 2000, 0, True), (TWO, 2048, 8, 2000, 0, False),
    (TWO, 4096, 2, 1500, 0, True), (TWO, 4096, 4, 1500, 0, False), (TWO, 1024, 4, 3000, 0, True), (TWO, 1024, 8, 3000, 0, False),
    (TWO, 768, 4, 3000, 0, False), (TWO, 8192, 8, 5000, 0, False), (TWO, 4096, 16, 1000, 0, True), (TWO, 4096, 16, 1000, 60, False),
    (TWO, 1024, 8, 2000, 1000, True), (TWO, 1024, 8, 2000, 250, False), (ONE, 1024, 4, 6000, 0, True), (ONE, 2048, 4, 6000, 0, False),
    (ONE, 768, 8, 6000, 0, True), (ONE, 8192, 2, 4000, 0, True), (ONE, 8192, 16, 4096, 0, False), (ONE, 512, 4, 9000, 0, True),
    (ONE, 768, 4, 9000, 0, False)])
def test_long_lists_that_leave_room_for_few_waves(shape, Q, W, L, cap, waves):
    """Both sides of the lines from which on a wave per query falls behind: a batch of many queries whose lists leave room for
    one to four waves a CU goes to the other paths (8,192 queries, W = 8, L = 5,000 took three times as long by waves)."""
    g, m, users, entries = _handles("bf16", *shape, 3001, 32, Q, 4)
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, 4, W, L, 100, cap), dtype=torch.uint8, device="cuda")
    _both(lambda: ann.ann_search(g, m, users, entries, W, L, 100, cap, workspace=ws), ws, waves)


@pytest.mark.parametrize("waves,Q,W,L", [(True, 4096, 8, 2000), (False, 8192, 16, 2000), (False, 600, 4, 5000)])
def test_long_lists_of_their_own(waves, Q, W, L):
    """Without a cap and with lists of every length the batch path runs all rounds at the pace of the longest query."""
    g, m, users, entries = _handles("bf16", *TWO, 3001, 32, Q, 4)
    gen = torch.Generator().manual_seed(Q)
    own = [torch.randint(1, hi + 1, (Q,), generator=gen, dtype=torch.int32).cuda() for hi in (W, L)] + [torch.zeros(Q, dtype=torch.int32).cuda()]
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, 4, W, L, 100, 0), dtype=torch.uint8, device="cuda")
    _both(lambda: ann.ann_search_ragged(g, m, users, entries, *own, W, L, 100, 0, workspace=ws), ws, waves)


@pytest.mark.parametrize("cap", [0, 24])
@pytest.mark.parametrize("dtype,shape", [("bf16", TWO), ("f16", ONE)])
def test_queries_with_their_own_parameters(dtype, shape, cap):
    """Widths, lists and caps per query, some of them outside their range (they are taken to its ends)."""
    Q = 3000
    g, m, users, entries = _handles(dtype, *shape, 5000, 16, Q, 4)
    gen = torch.Generator().manual_seed(Q)
    own = [torch.randint(lo, hi, (Q,), generator=gen, dtype=torch.int32).cuda() for lo, hi in ((0, 14), (0, 190), (0, 30))]
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, 4, 12, 170, 20, cap), dtype=torch.uint8, device="cuda")
    _both(lambda: ann.ann_search_ragged(g, m, users, entries, *own, 12, 170, 20, cap, workspace=ws), ws)


@pytest.mark.parametrize("shape,Q", [(TWO, 3000), (TWO, 2000), (ONE, 5000)])
def test_the_longest_query_is_handed_over(shape, Q):
    """The only query that has a seed: with more queries than waves it is taken first, among the last it would not be seen."""
    g, m, users, entries = _handles("bf16", *shape, 5000, 16, Q, 4)
    entries[torch.arange(Q) != 7] = -1
    own = [torch.full((Q,), v, dtype=torch.int32, device="cuda") for v in (1, 20, 0)]
    own[1][7] = 170
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, 4, 4, 170, 20, 0), dtype=torch.uint8, device="cuda")
    _, _, counters = _both(lambda: ann.ann_search_ragged(g, m, users, entries, *own, 4, 170, 20, 0, workspace=ws), ws)
    assert counters[2] > 100 and int(ws[256:384].view(torch.int64)[7]) == 1


@pytest.mark.parametrize("shape", [TWO, ONE])
def test_items_that_are_not_finite(shape):
    Q = 2200
    g, m, users, entries = _handles("bf16", *shape, 400, 16, Q, 8)
    emb = torch.randn(400, 64).bfloat16()
    emb[::9, 1], emb[3::11, 0], emb[5::13, 2] = float("inf"), float("-inf"), float("nan")
    g = ann.ann_graph_load(torch.randint(0, 400, (400, 16), dtype=torch.int32).cuda(), emb.cuda())
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, 8, 4, 64, 200, 0), dtype=torch.uint8, device="cuda")
    _both(lambda: ann.ann_search(g, m, users, entries, 4, 64, 200, 0, workspace=ws), ws)


def _under_a_limit(call, ws, Q, at_least):
    """The call by waves, again under a limit far below the 20 ms after which the waiting thread asks; it has to take longer than
    that for the reports to be needed."""
    call()
    torch.cuda.synchronize()
    start = time.perf_counter()
    ids, sc = [t.clone() for t in call()]
    torch.cuda.synchronize()
    assert time.perf_counter() - start > at_least
    assert int(ws[256:384].view(torch.int64)[8]) == Q
    ann.ann_set_progress_timeout(1e-3)
    try:
        got = call()
    finally:
        ann.ann_set_progress_timeout(600.0)
        torch.cuda.synchronize()
    assert torch.equal(got[0], ids) and torch.equal(got[1], sc)


def test_a_batch_by_waves_reports_its_progress():
    Q = 16384
    g, m, users, entries = _handles("bf16", *TWO, 200_000, 32, Q, 4)
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, 4, 4, 512, 10, 0), dtype=torch.uint8, device="cuda")
    _under_a_limit(lambda: ann.ann_search(g, m, users, entries, 4, 512, 10, 0, workspace=ws), ws, Q, 0.025)


def test_many_short_searches_report_their_progress():
    """Every query ends within seven rounds."""
    Q = 2_500_000
    g, m, users, entries = _handles("bf16", *TWO, 16, 16, Q, 4)
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, 4, 4, 16, 8, 0), dtype=torch.uint8, device="cuda")
    _under_a_limit(lambda: ann.ann_search(g, m, users, entries, 4, 16, 8, 0, workspace=ws), ws, Q, 0.03)
    assert ann.ann_search_stats(ws).max_query_iters < 7


def _rising_metric(hidden):
    """Relevance rises with the items' first two coordinates, 2 ** -4 and 2 ** -10 of them (small whole numbers: exact)."""
    d = 64
    dims = [2 * d, *hidden, 1]
    Ws = [torch.zeros(o, n) for n, o in zip(dims, dims[1:])]
    Ws[0][0, d], Ws[0][1, d + 1] = 1, 1
    for w in Ws[1:-1]:
        w[0, 0], w[1, 1] = 1, 1
    Ws[-1][0, 0], Ws[-1][0, 1] = 2.0 ** -4, 2.0 ** -10
    bs = [torch.zeros(o) for o in dims[1:-1]] + [torch.tensor([-4.0])]
    return ann.ann_mlp_load([w.bfloat16() for w in Ws], bs, torch.ones(1), d, ann.ANN_BF16)


def test_a_long_search_of_wide_rounds_reports_its_progress(monkeypatch):
    """One query that runs 500 rounds of 1,152 new items while the others end at once; rounds that wide are not handed over, so
    its wave scores them alone, some 40 ms in 256 rounds.  18 nodes a layer, each joined to one of the next and to 63 of its own."""
    monkeypatch.setenv("GMPGR_VISITED_SET", "bitmap")
    R, W, layers, Q, q = 64, 18, 500, 1100, 5
    N = layers * W * R
    i = torch.arange(N, device="cuda").view(layers, W, R)
    adj = torch.full((layers, W, R, R), -1, dtype=torch.int32, device="cuda")
    adj[:-1, :, 0, 0] = i[1:, :, 0]
    adj[:, :, 0, 1:] = i[:, :, 1:]
    emb = torch.zeros(layers, W, R, 64, device="cuda")
    rank = torch.arange(1, layers + 1, device="cuda")[:, None]
    emb[:, :, 0, 0], emb[:, :, 0, 1] = (rank // 64).float(), (rank % 64).float()
    g, m = ann.ann_graph_load(adj.view(N, R), emb.view(N, 64).bfloat16()), _rising_metric((256, 128))
    entries = torch.full((Q, W), -1, dtype=torch.int32, device="cuda")
    entries[q] = i[0, :, 0]
    users = torch.zeros(Q, 64, device="cuda").bfloat16()
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, W, W, W, W, 0), dtype=torch.uint8, device="cuda")
    _under_a_limit(lambda: ann.ann_search(g, m, users, entries, W, W, W, 0, workspace=ws), ws, Q, 0.04)
    assert ann.ann_search_stats(ws).max_query_iters == layers


@pytest.mark.parametrize("far", [100, 900])
@pytest.mark.parametrize("hidden", [(256, 128), (256,)])
def test_visited_table_that_fills_up(hidden, far, monkeypatch):
    """Items whose relevance rises with their id (id / 64 and id % 64 are two exact coordinates), each joined to the next 16: a
    table of 2,048 slots takes 1,024 ids, and queries that start far from the last item stop when it is full.  100 of them
    are all that run when the waves hand the last 256 queries over, of 900 many end before."""
    monkeypatch.setenv("GMPGR_VISITED_SET", "hash")
    N, R, k, Q, d = 8000, 16, 3, 2100, 64
    i = torch.arange(N, device="cuda")
    emb = torch.zeros(N, d, device="cuda")
    emb[:, 0], emb[:, 1] = (i // 64).float(), (i % 64).float()
    adj = i[:, None] + 1 + torch.arange(R, device="cuda")
    adj = torch.where(adj < N, adj, -1).int()
    g = ann.ann_graph_load(adj, emb.bfloat16())
    m = _rising_metric(hidden)
    start = torch.full((Q,), N - 30, dtype=torch.int32)
    start[torch.arange(far) * Q // far] = torch.linspace(0, N - 1100, far).int()
    entries, users = start[:, None].contiguous().cuda(), torch.zeros(Q, d, device="cuda").bfloat16()
    ws = torch.empty(ann.ann_search_workspace_bytes(g, m, Q, 1, 1, 1, k, 0), dtype=torch.uint8, device="cuda")
    out = torch.empty(Q, k, dtype=torch.int32, device="cuda"), torch.empty(Q, k, device="cuda")

    def call():
        with pytest.raises(ann.AnnError) as e:
            ann.ann_search(g, m, users, entries, 1, 1, k, 0, workspace=ws, out_ids=out[0].fill_(-7), out_scores=out[1])
        assert e.value.code == -5 and "visited table" in str(e.value)
        return out
    ids, _, counters = _both(call, ws)
    assert torch.equal(ids[:, 0].cpu(), (start + 16 * 63).clamp(max=N - 1))  # 1 + 16 * 63 ids fit, 16 more do not
    assert counters[3] == far
