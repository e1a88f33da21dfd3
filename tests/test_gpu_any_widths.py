"""Relevance on the matrix cores for layer widths of the caller's own, against the oracle: widths on either side of
the instruction's 32 (fp32: 16), item and user widths with and without whole 16-byte pieces, tables that are only
4-byte aligned, no hidden layer, widths beyond the LDS (vector-ALU kernel), lists of one pair up to several batches.

Bounds: fp32 relevances are sums in fp64, rounded once (2^-24 relative, 1e-6 asserted); 16-bit ones meet the bars of
the 16-bit modes (2e-3 against the oracle at the kernel's precision, median 2e-5; 1e-2 against the exact one)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import captured_launches
from workloads import random_mlp, to_host

pytestmark = pytest.mark.gpu

ann = pytest.importorskip("paper_2502_11490_amd")
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
ANN = {"f32": ann.ANN_F32, "bf16": ann.ANN_BF16, "f16": ann.ANN_F16}


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("d_user,d,hidden,J,M", [
    (32, 32, (64,), 3, 4097), (13, 20, (48, 24, 16), 1, 65), (80, 96, (192, 96), 2, 40001), (1, 2, (), 4, 33),
    (24, 40, (31, 33), 8, 1), (160, 160, (320, 313, 296), 4, 997), (8, 8, (33,) * 7, 5, 129),
    (7, 1000, (600, 40), 2, 70), (40, 24, (1200, 1100), 2, 50)])
def test_relevance_own_widths(dtype, d_user, d, hidden, J, M):
    rng = np.random.default_rng(d_user * 1000 + d)
    N, Q = 500, 37
    dims = [d_user + d, *hidden, J]
    Ws, bs = random_mlp(dims, 5, "bf16" if dtype == "bf16" else "f32", bias_scale=0.2)
    Ws = [w.to(TORCH[dtype]) for w in Ws]
    gen = torch.Generator().manual_seed(3)
    emb = torch.randn(N, d, generator=gen).to(TORCH[dtype])
    users = torch.randn(Q, d_user, generator=gen).to(TORCH[dtype])
    wl = {"emb": emb, "users": users, "W": Ws, "b": bs, "head_w": torch.rand(J, generator=gen)}
    q, it = rng.integers(0, Q, M).astype(np.int32), rng.integers(0, N, M).astype(np.int32)
    h = to_host(wl)
    mlp = oracle.Mlp(h["W"], h["b"], h["head_w"])
    exact = oracle.score_pairs(h["emb"], h["users"], mlp, q, it, n_threads=8)
    adj = torch.zeros(N, 1, dtype=torch.int32, device="cuda")
    qd, itd = torch.from_numpy(q).cuda(), torch.from_numpy(it).cuda()
    m = ann.ann_mlp_load(Ws, bs, wl["head_w"], d_user, ANN[dtype])
    results = []
    for shift in (0, 4 // emb.element_size()):  # base addresses 256-byte aligned, then only 4-byte aligned
        flat = torch.zeros(N * d + shift, dtype=emb.dtype, device="cuda")
        table = flat[shift:].view(N, d)
        table.copy_(emb)
        g = ann.ann_graph_load(adj, table)
        results.append(ann.ann_score_pairs(g, m, users.cuda(), qd, itd).cpu().numpy())
    assert np.array_equal(results[0], results[1])
    got = results[0]
    if dtype == "f32":
        np.testing.assert_allclose(got, exact, rtol=1e-6, atol=0)
        return
    assert np.max(np.abs(got - exact)) <= 1e-2 * max(1.0, float(np.sum(h["head_w"])))
    kern = oracle.score_pairs(h["emb"], h["users"], mlp, q, it, act_round=1 if dtype == "bf16" else 3, n_threads=8)
    err = np.abs(got - kern)
    assert np.max(err) <= 2e-3 * max(1.0, float(np.sum(h["head_w"]))) and np.median(err) <= 2e-5


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_own_widths_pairs_out_of_range_and_infinities(dtype):
    """Pairs out of range give NaN; an infinite input reaches only the pairs that hold it, and a hidden unit of
    minus infinity is zero after the ReLU whatever the rounded-up units around it hold."""
    Ws, bs = random_mlp([20, 33, 2], 9, dtype, bias_scale=0.2)
    emb = torch.randn(50, 12).to(TORCH[dtype])
    emb[7, 3] = float("inf")
    g = ann.ann_graph_load(torch.zeros(50, 1, dtype=torch.int32, device="cuda"), emb.cuda())
    m = ann.ann_mlp_load(Ws, bs, torch.tensor([0.5, 0.5]), 8, ANN[dtype])
    generic = ann.ann_mlp_load(Ws, bs, torch.tensor([0.5, 0.5]), 8, ANN[dtype], ann.ANN_MLP_GENERIC)
    users = torch.randn(4, 8).to(TORCH[dtype]).cuda()
    q = torch.tensor([0, 4, 1, -1, 2, 3, 3], dtype=torch.int32).cuda()
    it = torch.tensor([5, 5, 50, 3, 7, 6, -2], dtype=torch.int32).cuda()
    got = ann.ann_score_pairs(g, m, users, q, it).cpu().numpy()
    want = ann.ann_score_pairs(g, generic, users, q, it).cpu().numpy()
    assert list(np.isnan(got)) == list(np.isnan(want)) and np.isnan(got[[1, 2, 3, 6]]).all()
    keep = ~np.isnan(want)
    np.testing.assert_allclose(got[keep], want[keep], atol=1e-6 if dtype == "f32" else 2e-3)


@pytest.mark.parametrize("dtype,d_user,d,hidden", [("f32", 32, 32, (64,)), ("f32", 13, 20, (48, 24, 16)),
                                                   ("bf16", 13, 20, (48, 24, 16)), ("f16", 80, 96, (192, 96))])
def test_batches_of_every_size_give_a_pair_the_same_bits(dtype, d_user, d, hidden):
    """tile_rows is the most pairs a batch holds (one workgroup each), down to one block of columns; a pair's relevance
    is the same bit for bit whichever batch it lies in, a list too short for large batches by itself included."""
    gen = torch.Generator().manual_seed(7)
    N, Q, M, J = 700, 41, 40_003, 3
    Ws, bs = random_mlp([d_user + d, *hidden, J], 5, "bf16" if dtype == "bf16" else "f32", bias_scale=0.2)
    emb, users = (torch.randn(n, w, generator=gen).to(TORCH[dtype]).cuda() for n, w in ((N, d), (Q, d_user)))
    g = ann.ann_graph_load(torch.zeros(N, 1, dtype=torch.int32, device="cuda"), emb)
    m = ann.ann_mlp_load([w.to(TORCH[dtype]) for w in Ws], bs, torch.rand(J, generator=gen), d_user, ANN[dtype])
    q, it = (torch.randint(0, n, (M,), generator=gen, dtype=torch.int32).cuda() for n in (Q, N))
    base = ann.ann_score_pairs(g, m, users, q, it)  # long enough for the largest batches
    short, least = 1234, 16 if dtype == "f32" else 32
    for tile_rows in (0, 1, 16, 31, 32, 63, 64, 1000):
        out = torch.empty(short, device="cuda")
        call = lambda: ann.ann_score_pairs(g, m, users, q[:short], it[:short], out=out, tile_rows=tile_rows)
        call()
        assert torch.equal(out, base[:short]), tile_rows
        pairs = max(least, 64 if tile_rows >= 64 else 32 if tile_rows >= 32 else 16)
        if tile_rows > 0:
            assert captured_launches(call) == [(-(-short // pairs), 256)], tile_rows
        assert torch.equal(ann.ann_score_pairs(g, m, users, q, it, tile_rows=tile_rows), base), tile_rows
