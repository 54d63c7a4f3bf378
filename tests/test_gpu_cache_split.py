"""The cache lookup around the sizes at which a request's cache is split over several workgroups, and where the queries that no
request owns are answered: both forms of the kernel (rows that the fp64 matrix cores take and rows that they do not)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
N = 20_000


@pytest.fixture(scope="module", params=[64, 72, 776])
def store(request):
    from paper_2401_14021_amd import binding as B, inputs
    X, _ = inputs.clustered_datastore(N, request.param, 60, seed=5, device="cuda")
    return X, B.Datastore(X)


def _case(X, strides, C, seed):
    from paper_2401_14021_amd import inputs
    off = inputs.stride_offsets(strides)
    Q = int(off[-1])
    src = inputs.pick_rows(N, max(Q, 1), seed)
    q = inputs.queries_near_rows(X, src, seed + 1)[:Q]
    cids, clen = inputs.speculation_caches(N, len(strides), C, off, src[:Q], None, seed + 2)
    return cids.cuda(), clen.cuda(), q, off.cuda()


def _want(oracle, case, X):
    return oracle.cache_lookup(*(t.cpu().numpy() for t in case), X.cpu().numpy())


@pytest.mark.parametrize("R,C", [(1, 64), (1, 65), (1, 128), (1, 129), (3, 1024), (33, 700), (100, 300), (128, 257), (129, 1024),
                                 (257, 640), (300, 1024), (512, 200), (513, 129)])
def test_split_requests(store, oracle, R, C):
    from paper_2401_14021_amd import binding as B
    X, ds = store
    rng = np.random.default_rng(R + C)
    case = _case(X, rng.integers(0, 7, size=R).tolist(), C, R)
    Q = case[2].shape[0]
    wi, wsc = _want(oracle, case, X)
    ws = torch.empty(max(Q, 1), dtype=torch.int64, device="cuda").random_()
    for _ in range(3):   # the slots and the counts of one call are no concern of the next
        ids, sc = B.ralm_cache_lookup(*case, ds, workspace=ws)
        np.testing.assert_array_equal(ids.cpu().numpy(), wi)
        np.testing.assert_array_equal(sc.cpu().numpy(), wsc)


@pytest.mark.parametrize("R,C,use_workspace", [(5, 600, True), (5, 600, False), (200, 100, True), (600, 40, True), (5000, 8, True)])
def test_queries_outside_all_ranges(store, oracle, R, C, use_workspace):
    """Three queries in front of the first range and four behind the last: answered where the outputs are the call's own, left alone
    in the caller's."""
    from paper_2401_14021_amd import binding as B
    X, ds = store
    cids, clen, q, off = _case(X, [i % 3 for i in range(R)], C, R)
    wi, wsc = _want(oracle, (cids, clen, q, off), X)
    Q = q.shape[0]
    q = torch.cat([q[:3], q, q[:4]])
    off = off + 3
    ids, sc = B.ralm_cache_lookup(cids, clen, q, off, ds, use_workspace=use_workspace)
    np.testing.assert_array_equal(ids.cpu().numpy(), np.concatenate([[-1] * 3, wi, [-1] * 4]))
    np.testing.assert_array_equal(sc.cpu().numpy(), np.concatenate([[-np.inf] * 3, wsc, [-np.inf] * 4]).astype(np.float32))
    ids, sc = torch.full((Q + 7,), -9, dtype=torch.int32, device="cuda"), torch.full((Q + 7,), 9.0, device="cuda")
    B.ralm_cache_lookup(cids, clen, q, off, ds, spec_ids=ids, spec_scores=sc, use_workspace=use_workspace)
    np.testing.assert_array_equal(ids.cpu().numpy(), np.concatenate([[-9] * 3, wi, [-9] * 4]))
    np.testing.assert_array_equal(sc.cpu().numpy(), np.concatenate([[9.0] * 3, wsc, [9.0] * 4]).astype(np.float32))


@pytest.mark.parametrize("C", [64, 700])
def test_ranges_that_are_not_in_order(store, oracle, C):
    """A decreasing pair is an empty range; what a single request owns is answered, also outside the first and the last offset."""
    from paper_2401_14021_amd import binding as B
    X, ds = store
    cids, clen, q, _ = _case(X, [2] * 5, C, 3)
    off = torch.tensor([4, 6, 2, 4, 9, 7], device="cuda")   # [4, 6), none, [2, 4), [4, 9), none; 4 and 5 have two owners
    owner = {2: 2, 3: 2, 6: 3, 7: 3, 8: 3}
    ids, sc = B.ralm_cache_lookup(cids, clen, q, off, ds)
    ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
    for i, r in owner.items():
        one = torch.tensor([0, 1])
        wi, wsc = oracle.cache_lookup(cids[r:r + 1].cpu().numpy(), clen[r:r + 1].cpu().numpy(), q[i:i + 1].cpu().numpy(),
                                      one.numpy(), X.cpu().numpy())
        assert ids[i] == wi[0] and sc[i] == wsc[0]
    for i in (0, 1, 9):
        assert ids[i] == -1 and sc[i] == -np.inf
    for i in (4, 5):
        assert ids[i] in cids[0].tolist() + cids[3].tolist()
