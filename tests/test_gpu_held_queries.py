"""The scan that holds its queries in registers, at the edges of what it takes: every count of 64-element strips that it is
built for (an odd count keeps its operands differently), rows that end inside a strip, rows that are no whole lines, batches
that fill a tile and batches that do not, several query tiles, a last tile of rows that is nearly empty.

Whole numbers of at most 3 in magnitude: sums of up to 1088 products are exact in every type on the way, so ids and scores
must be the oracle's, and no query may need the exact pass."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
N = 150_001


@pytest.fixture(scope="module")
def rows():
    g = torch.Generator().manual_seed(11)
    X = torch.randint(-3, 4, (N, 1088), generator=g, dtype=torch.int8)
    # a run of equal rows that beat all others, in tiles that only the last stage visits: more scores of a tile are
    # admitted than a wave puts aside and than a workgroup parks
    X[391 * 256 + 7:391 * 256 + 200] = 3
    return X


def _best_two(Xd64, q64, l2):
    """Ids and scores of every query's two best rows, equal scores by lower id; whole numbers, exact in double."""
    ids, sc = [], []
    for i in range(0, len(q64), 64):
        full = Xd64 @ q64[i:i + 64].T
        if l2:
            full = 2 * full - (Xd64 ** 2).sum(1)[:, None] - (q64[i:i + 64] ** 2).sum(1)
        key = full * 2 ** 18 + (2 ** 18 - 1 - torch.arange(len(Xd64), device="cuda", dtype=torch.float64))[:, None]
        top = key.topk(2, dim=0).indices.T
        ids.append(top)
        sc.append(full.T.gather(1, top))
    return torch.cat(ids), torch.cat(sc)


def _check(rows, oracle, d, Q, dtype, metric_l2=False, last="held", ds=None):
    from paper_2401_14021_amd import binding as B
    k = 2
    X = rows[:, :d].float().contiguous()
    g = torch.Generator().manual_seed(d + Q)
    q = torch.randint(-3, 4, (Q, d), generator=g).float()
    q[::3] = q[::3].abs()   # these queries' best rows are the run of equal ones
    Xd = X.cuda()
    if ds is None:
        ds = B.Datastore.for_l2(Xd, dtype) if metric_l2 else B.Datastore.from_fp32(Xd, dtype)
    # the kernel that is meant is the one that runs: it takes the last stage, which holds most rows
    assert B.ralm_scan_routes(Q, ds, k, 4)[-1] == last
    ws = B.alloc_workspace(Q, ds, k, 4)
    ids, sc = B.ralm_retrieve_topk_ex(q.cuda(), ds, k, 4, workspace=ws)
    c = B.ralm_workspace_counters(ws)
    assert c["exact_pass"] == 0 and c["unanswered"] == 0 and c["ladder_overflows"] == 0, c
    wi, wsc = _best_two(Xd.double(), q.double().cuda(), metric_l2)
    np.testing.assert_array_equal(ids.cpu().numpy(), wi.cpu().numpy())
    np.testing.assert_array_equal(sc.cpu().numpy(), wsc.float().cpu().numpy())
    picked = sorted({0, min(31, Q - 1), min(32, Q - 1), Q // 2, Q - 1})
    wi, ws_ = oracle.retrieve_topk(q[picked].numpy(), X.numpy(), k, metric="l2" if metric_l2 else "ip")
    np.testing.assert_array_equal(ids.cpu().numpy()[picked], wi)
    np.testing.assert_array_equal(sc.cpu().numpy()[picked], ws_)


@pytest.mark.parametrize("strips", range(5, 18))
@pytest.mark.parametrize("full", [True, False])
def test_one_column_block_per_wave(rows, oracle, strips, full):
    d = strips * 64 if full else strips * 64 - 56
    _check(rows, oracle, d, 128 if full else 65, torch.bfloat16 if full else torch.float16)


@pytest.mark.parametrize("strips", range(5, 13))
@pytest.mark.parametrize("full", [True, False])
def test_two_column_blocks_per_wave(rows, oracle, strips, full):
    d = strips * 64 if full else strips * 64 - 56
    _check(rows, oracle, d, 256 if full else 129, torch.float16 if full else torch.bfloat16)


@pytest.mark.parametrize("d,Q", [(392, 1), (904, 40), (1032, 64), (328, 33)])
def test_few_queries_over_rows_that_are_no_whole_lines(rows, oracle, d, Q):
    _check(rows, oracle, d, Q, torch.float16)


@pytest.mark.parametrize("d,Q,last", [(768, 512, "held"), (712, 1000, "held"), (392, 512, "held"), (576, 1024, "held"),
                                      (904, 129, "held"), (1000, 256, "held"), (1080, 512, "held"), (840, 1000, "held"),
                                      (1080, 384, "parked")])   # three tiles on 30 of an XCD's 32 compute units
def test_several_query_tiles(rows, oracle, d, Q, last):
    _check(rows, oracle, d, Q, torch.bfloat16, last=last)


@pytest.mark.parametrize("d,Q", [(392, 1700), (768, 1792), (520, 2304), (520, 8448)])
def test_more_workgroups_than_compute_units(d, Q):
    """Seven and nine query tiles do not share out over an XCD's 32 compute units, and 33 are more than it has: the launch has a
    second round of workgroups or more, which begin as the first ones end, in the LDS that those leave."""
    from paper_2401_14021_amd import binding as B
    n = 2 ** 19 - 1
    g = torch.Generator().manual_seed(d)
    X = torch.randint(-3, 4, (n, d), generator=g, dtype=torch.int8).float().cuda()
    q = torch.randint(-3, 4, (Q, d), generator=g).float().cuda()
    X[391 * 256 + 7:391 * 256 + 200] = 3
    q[::3] = q[::3].abs()   # these queries' best rows are the run of equal ones
    ds = B.Datastore.from_fp32(X, torch.bfloat16)
    assert B.ralm_scan_routes(Q, ds, 2, 4)[-1] == "held"
    ws = B.alloc_workspace(Q, ds, 2, 4)
    ids, sc = B.ralm_retrieve_topk_ex(q, ds, 2, 4, workspace=ws)
    c = B.ralm_workspace_counters(ws)
    assert c["exact_pass"] == 0 and c["unanswered"] == 0 and c["ladder_overflows"] == 0, c
    Xd, order = X.double(), (n - torch.arange(n, device="cuda", dtype=torch.float64))[:, None]
    for i in range(0, Q, 64):   # whole numbers: exact in double, also with the order of equal scores behind them
        full = Xd @ q[i:i + 64].double().T
        want = (full * 2 ** 19 + order).topk(2, dim=0).indices.T
        assert torch.equal(ids[i:i + 64].long(), want)
        assert torch.equal(sc[i:i + 64], full.T.gather(1, want).float())


@pytest.mark.parametrize("d,Q", [(1024, 100), (632, 200)])
def test_squared_distance(rows, oracle, d, Q):
    _check(rows, oracle, d, Q, torch.float16, metric_l2=True)


@pytest.mark.parametrize("reserve", [8, 240, 300])
def test_compute_units_reserved(rows, oracle, reserve):
    from paper_2401_14021_amd import binding as B
    B.ralm_scan_reserve_cus(reserve)
    try:
        # with one unit per XCD left two query tiles find no place; up to 32 queries stay in tiles under any reserve
        _check(rows, oracle, 904, 129, torch.bfloat16, last="parked" if reserve == 300 else "held")
        _check(rows, oracle, 768, 100, torch.bfloat16)
        _check(rows, oracle, 392, 40, torch.float16)
        _check(rows, oracle, 392, 20, torch.float16, last="parked")
    finally:
        B.ralm_scan_reserve_cus(0)


@pytest.mark.parametrize("d,Q", [(768, 100), (392, 40), (768, 200), (904, 250)])
def test_products_that_cancel_in_order(oracle, d, Q):
    """A score is one chain of sums over its elements in their order.  Products of one sign in every other group of 16
    elements and of the other sign between them: in order they cancel, added by even and odd groups they overflow fp32 to
    both infinities, the score is no number and the row is lost."""
    from paper_2401_14021_amd import binding as B
    N, r = 150_001, 391 * 256 + 77   # a row that only the last stage visits
    g = torch.Generator().manual_seed(d)
    X = torch.randint(-3, 4, (N, d), generator=g).float()
    q = torch.randint(1, 4, (Q, d), generator=g).float()
    q[:, :64] = 1.0
    X[r] = 0.0
    X[r, [0, 32]] = -2.0 ** 127
    X[r, [16, 48]] = 2.0 ** 127
    X[r, 64] = 2.0 ** 100            # the score, in double and in fp32 alike
    ds = B.Datastore.from_fp32(X.cuda(), torch.bfloat16)
    assert B.ralm_scan_routes(Q, ds, 2, 4)[-1] == "held"
    ids, sc = B.ralm_retrieve_topk_ex(q.cuda(), ds, 2, 4)
    ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
    np.testing.assert_array_equal(ids[:, 0], np.full(Q, r))
    np.testing.assert_array_equal(sc[:, 0], q[:, 64].numpy() * 2.0 ** 100)
    wi, ws = oracle.retrieve_topk(q[:4].numpy(), X.numpy(), 2)
    np.testing.assert_array_equal(ids[:4], wi)
    np.testing.assert_array_equal(sc[:4], ws)


@pytest.mark.parametrize("d,pitch,Q", [(392, 448, 100), (392, 400, 30), (392, 400, 200), (456, 512, 200), (712, 768, 65),
                                       (712, 768, 256), (904, 960, 128), (904, 912, 1), (904, 912, 200), (1032, 1088, 100)])
def test_spare_columns_are_never_used(rows, oracle, d, pitch, Q):
    """Rows that end inside a strip, NaN behind them: pitches of whole and of broken lines, counts of strips odd and even, one
    and two column blocks."""
    from paper_2401_14021_amd import binding as B
    X = rows[:, :d].float().contiguous().cuda()
    store = torch.full((N, pitch), float("nan"), dtype=torch.bfloat16, device="cuda")
    B.ralm_build_scan_copy(X, store[:, :d])
    assert torch.isnan(store[:, d:]).all()
    _check(rows, oracle, d, Q, torch.bfloat16, ds=B.Datastore(X, store[:, :d]))


@pytest.mark.parametrize("d,Q", [(320, 100), (392, 20), (320, 200), (904, 200)])
def test_infinite_scores(rows, oracle, d, Q):
    """Rows whose scores overflow fp32, in tiles that only the last stage visits: three to +inf, which rank by id, one to -inf, and
    one whose products overflow to both: that score is no number in the scan, and small in double."""
    from paper_2401_14021_amd import binding as B
    X = rows[:, :d].float().contiguous()
    t = 391 * 256
    X[t:t + 256] = rows[:256, :d].float()   # (without the run of equal rows)
    X[[t + 40, t + 9, N - 1], 0] = 3e38
    X[t + 8, 0] = -3e38
    X[t + 77, :64] = 0
    X[t + 77, 0], X[t + 77, 16] = 3e38, -3e38
    g = torch.Generator().manual_seed(Q)
    q = torch.randint(-3, 4, (Q, d), generator=g).float()
    q[:, [0, 16]] = 4
    ds = B.Datastore.from_fp32(X.cuda(), torch.bfloat16)
    assert B.ralm_scan_routes(Q, ds, 5, 8)[-1] == "held"
    ids, sc = B.ralm_retrieve_topk_ex(q.cuda(), ds, 5, 8)
    ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
    np.testing.assert_array_equal(ids[:, :3], np.tile([t + 9, t + 40, N - 1], (Q, 1)))
    assert (sc[:, :3] == np.inf).all() and np.isfinite(sc[:, 3:]).all()
    assert not np.isin(ids, [t + 8, t + 77]).any()
    picked = [0, 31 % Q, Q // 2, Q - 1]
    wi, wsc = oracle.retrieve_topk(q[picked].numpy(), X.numpy(), 5)
    np.testing.assert_array_equal(ids[picked], wi)
    np.testing.assert_array_equal(sc[picked], wsc)
