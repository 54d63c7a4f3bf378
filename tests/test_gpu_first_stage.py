"""First stages of few tiles, which run in quarter tiles: datastores of one stage whose last tile ends in each of its quarters,
in every width of the query tile and every type of row.  Whole numbers, so that ids and scores must be the oracle's."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("Q", [33, 64, 65, 128, 129, 300])
@pytest.mark.parametrize("N,d", [(1, 8), (63, 64), (16 * 256 + 1, 136), (16 * 256 + 65, 768), (16 * 256 + 192, 64),
                                 (16 * 256 + 255, 1032)])
def test_partial_last_tiles(oracle, N, d, Q, dtype):
    from paper_2401_14021_amd import binding as B
    g = torch.Generator().manual_seed(N + Q)
    X = torch.randint(-3, 4, (N, d), generator=g).float()
    q = torch.randint(-3, 4, (Q, d), generator=g).float()
    k = min(10, N)
    Xd = X.cuda()
    ds = B.Datastore(Xd) if dtype == "f32" else B.Datastore.from_fp32(Xd, torch.bfloat16 if dtype == "bf16" else torch.float16)
    assert B.ralm_scan_routes(Q, ds, k)[0] == "all_quarters"
    ws = B.alloc_workspace(Q, ds, k)
    ids, sc = B.ralm_retrieve_topk_ex(q.cuda(), ds, k, workspace=ws)
    c = B.ralm_workspace_counters(ws)
    assert c["exact_pass"] == 0 and c["ladder_overflows"] == 0, c
    wi, wsc = oracle.retrieve_topk(q.numpy(), X.numpy(), k)
    np.testing.assert_array_equal(ids.cpu().numpy(), wi)
    np.testing.assert_array_equal(sc.cpu().numpy(), wsc)


def _check(oracle, X, q, dtype, metric, k, tail):
    """ids and scores of all queries; the first stage leaves scores and ends in a tile of `tail` rows"""
    from paper_2401_14021_amd import binding as B
    (N, d), Q = X.shape, q.shape[0]
    Xd = X.cuda()
    half = torch.bfloat16 if dtype == "bf16" else torch.float16
    ds = B.Datastore.for_l2(Xd, half) if metric == "l2" else (B.Datastore(Xd) if dtype == "f32" else B.Datastore.from_fp32(Xd, half))
    assert B.ralm_first_stage_scores(Q, ds, k)
    ws = B.alloc_workspace(Q, ds, k)
    ids, sc = B.ralm_retrieve_topk_ex(q.cuda(), ds, k, workspace=ws)
    c = B.ralm_workspace_counters(ws)
    assert c["ladder_overflows"] == 0 and c["unanswered"] == 0 and c["exact_pass"] == 0, c
    assert B.ralm_workspace_stage_entries(ws)[0] == Q * (63 * 256 + tail)
    full = 2.0 * Xd.double() @ q.double().cuda().T - (Xd.double() ** 2).sum(dim=1)[:, None] if metric == "l2" else Xd.double() @ q.double().cuda().T
    key = full * 2 ** 19 + (N - torch.arange(N, device="cuda", dtype=torch.float64))[:, None]   # equal scores by lower id
    assert torch.equal(ids.long(), key.topk(k, dim=0).indices.T)
    picked = list(range(0, Q, max(1, Q // 12)))
    wi, wsc = oracle.retrieve_topk(q[picked].numpy(), X.numpy(), k, metric=metric)
    np.testing.assert_array_equal(ids.cpu().numpy()[picked], wi)
    np.testing.assert_array_equal(sc.cpu().numpy()[picked], wsc)


@pytest.mark.parametrize("tail", [1, 31, 32, 33, 255, 256])      # rows of the first stage's last tile
@pytest.mark.parametrize("Q", [3, 32, 33, 64, 100, 200, 300, 600])
@pytest.mark.parametrize("dtype,metric", [("f32", "ip"), ("bf16", "ip"), ("f16", "ip"), ("f16", "l2")])
def test_scores_of_a_first_stage(oracle, dtype, metric, Q, tail):
    """Every second tile, 64 of them, and the last one ends anywhere in its blocks of 32: whole numbers, so that many blocks have
    the same best.  A third of the queries has its best rows among the last, a third has one of few scores for all rows."""
    N, d, k = 126 * 256 + tail, 72, 20
    g = torch.Generator().manual_seed(tail)
    X = torch.randint(-2, 3, (N, d), generator=g).float()
    X[:, 0] = torch.arange(N).remainder(3).float()
    X[:, 1] = 0.0
    X[-min(tail, 40):, 1] = 1.0
    q = torch.randint(-2, 3, (Q, d), generator=g).float()
    q[:, 1] = 0.0
    q[1::3] = 0.0
    q[1::3, 0] = 1.0                                             # scores 0, 1 and 2
    q[2::3, 1] = 64.0
    _check(oracle, X, q, dtype, metric, k, tail)


@pytest.mark.parametrize("tail", [1, 33, 256])
@pytest.mark.parametrize("Q", [16, 64, 128, 256])
def test_scores_of_a_first_stage_of_distant_tiles(oracle, Q, tail):
    """Every 13th tile: rows' numbers follow from their places in the stage."""
    N, d = 819 * 256 + tail, 16
    g = torch.Generator().manual_seed(tail)
    X = torch.randint(-2, 3, (N, d), generator=g).float()
    X[-1] = 3.0
    q = torch.randint(-2, 3, (Q, d), generator=g).float()
    q[::2] = q[::2].abs() + 1
    _check(oracle, X, q, "bf16", "ip", 32, tail)
