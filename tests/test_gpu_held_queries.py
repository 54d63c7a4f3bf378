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


def _check(rows, oracle, d, Q, dtype, metric_l2=False):
    from paper_2401_14021_amd import binding as B
    k = 2
    X = rows[:, :d].float().contiguous()
    g = torch.Generator().manual_seed(d + Q)
    q = torch.randint(-3, 4, (Q, d), generator=g).float()
    q[::3] = q[::3].abs()   # these queries' best rows are the run of equal ones
    Xd = X.cuda()
    ds = B.Datastore.for_l2(Xd, dtype) if metric_l2 else B.Datastore.from_fp32(Xd, dtype)
    ws = B.alloc_workspace(Q, ds, k, 4)
    ids, sc = B.ralm_retrieve_topk_ex(q.cuda(), ds, k, 4, workspace=ws)
    c = B.ralm_workspace_counters(ws)
    assert c["exact_pass"] == 0 and c["unanswered"] == 0 and c["ladder_overflows"] == 0, c
    ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
    # queries at the borders of the waves' column blocks, and one in each block
    pick = sorted({i for b in range(0, Q, 32) for i in (b, min(b + 31, Q - 1))} | {0, Q - 1, Q // 2})[:24]
    Xd64 = Xd.double()
    for i in pick:
        qi = q[i].double().cuda()
        full = -((Xd64 - qi) ** 2).sum(1) if metric_l2 else Xd64 @ qi
        best = full.max()
        assert sc[i, 0] == best.item()
    picked = pick[:4] + pick[-4:]
    if metric_l2:
        wi, ws_ = oracle.retrieve_topk(q[picked].numpy(), X.numpy(), k, metric="l2")
    else:
        wi, ws_ = oracle.retrieve_topk(q[picked].numpy(), X.numpy(), k)
    np.testing.assert_array_equal(ids[picked], wi)
    np.testing.assert_array_equal(sc[picked], ws_)


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


@pytest.mark.parametrize("d,Q", [(768, 512), (712, 1000), (392, 512), (576, 1024), (904, 129), (1000, 256), (1080, 384), (840, 1000)])
def test_several_query_tiles(rows, oracle, d, Q):
    _check(rows, oracle, d, Q, torch.bfloat16)


@pytest.mark.parametrize("d,Q", [(1024, 100), (632, 200)])
def test_squared_distance(rows, oracle, d, Q):
    _check(rows, oracle, d, Q, torch.float16, metric_l2=True)


@pytest.mark.parametrize("reserve", [8, 240, 300])
def test_compute_units_reserved(rows, oracle, reserve):
    from paper_2401_14021_amd import binding as B
    B.ralm_scan_reserve_cus(reserve)
    try:
        _check(rows, oracle, 904, 129, torch.bfloat16)
        _check(rows, oracle, 768, 100, torch.bfloat16)
        _check(rows, oracle, 392, 20, torch.float16)
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
    ids, sc = B.ralm_retrieve_topk_ex(q.cuda(), ds, 2, 4)
    ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
    np.testing.assert_array_equal(ids[:, 0], np.full(Q, r))
    np.testing.assert_array_equal(sc[:, 0], q[:, 64].numpy() * 2.0 ** 100)
    wi, ws = oracle.retrieve_topk(q[:4].numpy(), X.numpy(), 2)
    np.testing.assert_array_equal(ids[:4], wi)
    np.testing.assert_array_equal(sc[:4], ws)
