"""Stages scan with an admission key of a better rank than k' of the rows scanned so far.  Stores whose first sample holds a
query's best rows all together: rows between that rank and k' are then not admitted, the check has to take the
admission key for the best row that may be missing, and rows that belong in the first k have to be found all the same.
Whole numbers: ids and scores must be the oracle's."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
N, d = 200_001, 64


def _rows(levels):
    """Column c of four is query c's: tile 0, which every stage's sample has visited, holds 64 rows of the best scores in it, another
    tile, which only the last stage visits (a prime number of tiles from the first), 59 rows with scores of ranks 40 to 60, and
    five of the best."""
    g = torch.Generator().manual_seed(3)
    X = torch.randint(-1, 2, (N, d), generator=g).float()
    X[:, :4] = torch.randint(0, 40, (N, 4), generator=g).float()
    for c in range(4):
        X[c * 64:c * 64 + 64, c] = 230 - (torch.arange(64) // levels).float()
        t = 701 * 256 + c * 64
        X[t:t + 59, c] = 230 - ((40 + torch.arange(59) % 20) // levels).float()
        X[t + 59:t + 64, c] = 240.0
    return X


@pytest.mark.parametrize("levels", [1, 4, 32])   # rows of the same score among the best
@pytest.mark.parametrize("Q", [3, 70, 200, 600])
@pytest.mark.parametrize("dtype,metric", [("bf16", "ip"), ("f16", "ip"), ("f16", "l2"), ("f32", "ip")])
def test_best_rows_in_the_first_sample(oracle, dtype, metric, Q, levels):
    from paper_2401_14021_amd import binding as B
    X = _rows(levels)
    q = torch.zeros(Q, d)
    q[torch.arange(Q), torch.arange(Q) % 4] = 1.0 + (torch.arange(Q) // 4 % 3).float()
    if metric == "l2":   # rows of one norm in the columns that count rank by distance as by product
        q[torch.arange(Q), torch.arange(Q) % 4] = 255.0
    Xd = X.cuda()
    if metric == "l2":
        ds = B.Datastore.for_l2(Xd, torch.float16)
    elif dtype == "f32":
        ds = B.Datastore(Xd)
    else:
        ds = B.Datastore.from_fp32(Xd, torch.bfloat16 if dtype == "bf16" else torch.float16)
    picked = list(range(min(Q, 24)))
    for k in (5, 20, 60):
        ws = B.alloc_workspace(Q, ds, k)
        ids, sc = B.ralm_retrieve_topk_ex(q.cuda(), ds, k, workspace=ws)
        c = B.ralm_workspace_counters(ws)
        assert c["unanswered"] == 0 and c["ladder_overflows"] == 0, c
        wi, wsc = oracle.retrieve_topk(q[picked].numpy(), X.numpy(), k, metric=metric)
        np.testing.assert_array_equal(ids.cpu().numpy()[picked], wi)
        np.testing.assert_array_equal(sc.cpu().numpy()[picked], wsc)
        full = Xd.double() @ q.double().cuda().T
        if metric == "ip" and Q > 24:   # all queries: whole numbers, equal scores by lower id
            key = full * 2 ** 18 + (N - torch.arange(N, device="cuda", dtype=torch.float64))[:, None]
            assert torch.equal(ids.long(), key.topk(k, dim=0).indices.T)


def test_the_check_knows_what_was_not_admitted():
    """The margin is taken from the admission key where it lies above the worst kept candidate."""
    from paper_2401_14021_amd import binding as B
    X, k = _rows(1), 20
    q = torch.zeros(4, d)
    q[torch.arange(4), torch.arange(4)] = 1.0
    ds = B.Datastore.from_fp32(X.cuda())
    ws, margin = B.alloc_workspace(4, ds, k), torch.empty(4, device="cuda")
    ids, sc = B.ralm_retrieve_topk_ex(q.cuda(), ds, k, workspace=ws, out_margin=margin)
    c = B.ralm_workspace_counters(ws)
    assert c["exact_pass"] == 0 and c["soft_certified"] == 4, c
    # The best: five of 240, then 230, 229, ..: rank 20 scores 216.  The admission key of the last stages is the first sample's rank 31
    # (score 200) or a few ranks worse, above the other tile's 59 rows; the worst kept of 64 candidates scores 172.
    assert sc[:, -1].cpu().tolist() == [216.0] * 4
    m = margin.cpu()
    assert ((m >= 216 - 200) & (m <= 216 - 191)).all(), m


@pytest.mark.parametrize("Q", [16, 100, 200, 600])
@pytest.mark.parametrize("k", [10, 20])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_copies_that_lie_together(dtype, k, Q):
    """Every row 40 times in a row: the first sample holds a query's best k rows and as many of the same score again.  An admission key among
    those would leave the check no margin; one of rank k' does, and no query may need the exact pass."""
    from paper_2401_14021_amd import binding as B, inputs
    copies = 40
    X, _ = inputs.clustered_datastore(5000, 128, 1000, seed=7, device="cuda")
    near = torch.arange(Q, device="cuda") % 4 + 1                # their copies lie in tile 0
    q = inputs.queries_near_rows(X, near, seed=Q, sigma=0.005)
    ds = B.Datastore.from_fp32(X.repeat_interleave(copies, 0).contiguous(), dtype)
    ws = B.alloc_workspace(Q, ds, k)
    ids, _ = B.ralm_retrieve_topk_ex(q, ds, k, workspace=ws)
    c = B.ralm_workspace_counters(ws)
    assert c["exact_pass"] == 0 and c["soft_certified"] == Q, c
    best = (q.double() @ X.double().T).argmax(dim=1)             # its first k copies
    assert torch.equal(ids.long(), best[:, None] * copies + torch.arange(k, device="cuda"))


@pytest.mark.parametrize("Q", [3, 70, 200, 600])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_equal_scores_around_the_admission_key(oracle, dtype, Q):
    """Whole numbers, which every type scores exactly: ranks 1 to 40 of the first sample have one score.  Rows of that score that come
    later have higher ids, so nothing is in doubt and no query may need the exact pass."""
    from paper_2401_14021_amd import binding as B
    k = 20
    X = torch.zeros(N, d)
    for c in range(4):
        X[c * 64:c * 64 + 40, c] = 230.0
        X[c * 64 + 40:c * 64 + 64, c] = 200.0 - torch.arange(24).float()
        X[701 * 256 + c * 64:701 * 256 + c * 64 + 8, c] = 230.0
    q = torch.zeros(Q, d)
    q[torch.arange(Q), torch.arange(Q) % 4] = 1.0
    ds = B.Datastore(X.cuda()) if dtype == "f32" else B.Datastore.from_fp32(X.cuda(), torch.bfloat16 if dtype == "bf16" else torch.float16)
    ws = B.alloc_workspace(Q, ds, k)
    ids, sc = B.ralm_retrieve_topk_ex(q.cuda(), ds, k, workspace=ws)
    c = B.ralm_workspace_counters(ws)
    assert c["exact_pass"] == 0 and c["ladder_overflows"] == 0, c
    wi, wsc = oracle.retrieve_topk(q[:4].numpy(), X.numpy(), k)
    want = np.arange(Q) % 4
    np.testing.assert_array_equal(ids.cpu().numpy(), wi[want])
    np.testing.assert_array_equal(sc.cpu().numpy(), wsc[want])


@pytest.mark.parametrize("Q", [3, 70, 200, 300])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_a_row_that_rounding_puts_below_the_admission_key(oracle, dtype, Q):
    """The check has to queue a query whose rank-k score lies within the rounding of the admission key.  Values near 480 (2270 for fp16), where the scan's
    type counts by two.  Tile 0, 64 rows per query: scan scores 484 (19 rows), 480, 474 (ranks 21 to 31) and 462 (up to rank 64),
    every one 0.99 off the exact score, which rounding can be 8 times of in the check's eyes: 7.9.  The admission key is 474, 5 below the exact rank-20 score, the
    worst kept score 462, 17 below it.  Another tile holds a row of the exact score 479.92, before rank 20, whose eight values are each rounded down by 0.99: its
    scan score 472 is not admitted."""
    from paper_2401_14021_amd import binding as B
    k, width = 20, 128
    base, n = (1792, 3000) if dtype == "f16" else (0, 300)
    X = torch.zeros(N, width)
    v = torch.tensor([484.0] * 19 + [480.0] + [474.0] * 11 + [462.0] * 33)
    off = torch.where(torch.arange(64) % 2 == 0, 0.99, -0.99)     # (rank 20: -0.99)
    total = 472 + base + 3 * n                                    # of the other tile's row's five positive values, as scanned
    low = total // 10 * 2
    five = [low + 2] * ((total - 5 * low) // 2) + [low] * (5 - (total - 5 * low) // 2)
    for c in range(4):
        X[c * 64:c * 64 + 64, 8 * c] = v + base + off
        X[701 * 256 + c, 8 * c:8 * c + 8] = torch.tensor([x + 0.99 for x in five] + [-(n - 0.99)] * 3)
    q = torch.zeros(Q, width)
    for i in range(Q):
        q[i, i % 4 * 8:i % 4 * 8 + 8] = 2.0 ** (i // 4 % 3)
    ds = B.Datastore(X.cuda()) if dtype == "f32" else B.Datastore.from_fp32(X.cuda(), torch.bfloat16 if dtype == "bf16" else torch.float16)
    ws, margin = B.alloc_workspace(Q, ds, k), torch.empty(Q, device="cuda")
    ids, sc = B.ralm_retrieve_topk_ex(q.cuda(), ds, k, workspace=ws, out_margin=margin)
    c = B.ralm_workspace_counters(ws)
    assert c["exact_pass"] == Q and c["ladder_overflows"] == 0 and c["unanswered"] == 0, c
    scale = 2.0 ** (torch.arange(Q) // 4 % 3)
    assert torch.allclose(margin.cpu(), 5.01 * scale, rtol=0, atol=0.01)   # 479.01 - 474
    picked = list(range(min(Q, 12)))
    wi, wsc = oracle.retrieve_topk(q[picked].numpy(), X.numpy(), k)
    assert (wi[:, -1] == 701 * 256 + np.arange(len(picked)) % 4).all()
    np.testing.assert_array_equal(ids.cpu().numpy(), wi[np.arange(Q) % 4])
    np.testing.assert_array_equal(sc.cpu().numpy()[picked], wsc)
