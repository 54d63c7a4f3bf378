"""The cache lookup where a request's cache is split over several workgroups and where it is not, and where the queries that no
request owns are answered: both forms of the kernel (rows that the fp64 matrix cores take and rows that they do not), both row
types and metrics.  The tests of a route state it."""
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


def _whole_numbers(dtype, d, metric, R, C, smax):
    """Rows and queries of whole numbers (sums are exact, equal scores go to the lower id), ragged caches, requests without queries."""
    from paper_2401_14021_amd import binding as B, inputs
    rng = np.random.default_rng(d + 7 * R + C)
    n = 5000
    X = torch.from_numpy(rng.integers(-3, 4, size=(n, d)).astype(np.float32)).to(torch.float16 if dtype == "f16" else torch.float32)
    strides = rng.integers(0, smax + 1, size=R)
    strides[0] = smax
    off = inputs.stride_offsets(strides.tolist())
    q = torch.from_numpy(rng.integers(-3, 4, size=(int(off[-1]), d)).astype(np.float32))
    cids = torch.from_numpy(rng.integers(0, n, size=(R, C)).astype(np.int32))
    clen = torch.from_numpy(rng.choice([0, 1, C // 3, C - 1, C], size=R).astype(np.int32))
    clen[0] = C
    ds = B.Datastore(X.cuda()) if metric == "ip" else B.Datastore.for_l2(X.cuda())
    return X, ds, cids, clen, q, off


ROUTES = [   # dtype, d, metric, R, C, most queries of a request, (workgroups per request, pieces in flight; 0: vector units)
    ("f32", 768, "ip", 64, 1024, 3, (4, 4)), ("f32", 768, "ip", 3, 1024, 20, (16, 8)), ("f32", 768, "ip", 33, 1024, 2, (7, 8)),
    ("f32", 768, "ip", 300, 1024, 2, (3, 4)), ("f32", 192, "ip", 33, 300, 5, (5, 6)), ("f32", 192, "ip", 64, 300, 5, (4, 4)),
    ("f16", 1024, "ip", 16, 300, 18, (5, 8)), ("f16", 1024, "ip", 64, 4096, 1, (4, 8)), ("f16", 128, "ip", 100, 1000, 2, (2, 4)),
    ("f16", 392, "ip", 8, 256, 17, (4, 0)), ("f32", 768, "l2", 100, 300, 8, (2, 0)), ("f16", 1000, "l2", 8, 129, 9, (3, 0)),
    ("f32", 392, "ip", 300, 1024, 2, (3, 0)), ("f32", 768, "ip", 400, 300, 2, (1, 4)), ("f16", 1024, "ip", 400, 700, 1, (1, 8)),
]


@pytest.mark.parametrize("dtype,d,metric,R,C,smax,route", ROUTES)
def test_routes(oracle, dtype, d, metric, R, C, smax, route):
    """Outputs of the call's own and of the caller's, each with queries that nobody owns, in a workspace that holds anything."""
    from paper_2401_14021_amd import binding as B
    X, ds, cids, clen, q, off = _whole_numbers(dtype, d, metric, R, C, smax)
    wi, wsc = oracle.cache_lookup(cids.numpy(), clen.numpy(), q.numpy(), off.numpy(), X.numpy(), metric)
    q, off = torch.cat([q[:1], q, q[:2]]).cuda(), off.cuda() + 1
    Q = q.shape[0]
    assert B.ralm_lookup_route(R, Q, C, ds)[:2] == route
    args = (cids.cuda(), clen.cuda(), q, off, ds)
    ws = torch.empty(Q, dtype=torch.int64, device="cuda").random_()
    for _ in range(2):   # the slots and the counts of one call are no concern of the next
        ids, sc = B.ralm_cache_lookup(*args, workspace=ws)
        np.testing.assert_array_equal(ids.cpu().numpy(), np.concatenate([[-1], wi, [-1] * 2]))
        np.testing.assert_array_equal(sc.cpu().numpy(), np.concatenate([[-np.inf], wsc, [-np.inf] * 2]).astype(np.float32))
        ids, sc = torch.full((Q,), -9, dtype=torch.int32, device="cuda"), torch.full((Q,), 9.0, device="cuda")
        B.ralm_cache_lookup(*args, spec_ids=ids, spec_scores=sc, workspace=ws)
        np.testing.assert_array_equal(ids.cpu().numpy(), np.concatenate([[-9], wi, [-9] * 2]))
        np.testing.assert_array_equal(sc.cpu().numpy(), np.concatenate([[9.0], wsc, [9.0] * 2]).astype(np.float32))


@pytest.mark.parametrize("dtype,d,metric", [("f32", 768, "ip"), ("f16", 1024, "ip"), ("f16", 392, "ip"), ("f32", 768, "l2")])
@pytest.mark.parametrize("own_outputs", [True, False])
def test_ranges_that_are_not_in_order_of_split_requests(oracle, dtype, d, metric, own_outputs):
    from paper_2401_14021_amd import binding as B
    X, ds, cids, clen, q, _ = _whole_numbers(dtype, d, metric, 5, 700, 3)
    q = torch.cat([q] * 10)[:10]
    off = torch.tensor([4, 6, 2, 4, 9, 7])   # [4, 6), none, [2, 4), [4, 9), none; 4 and 5 have two owners
    owner = {2: 2, 3: 2, 6: 3, 7: 3, 8: 3}
    clen[:] = 700
    assert B.ralm_lookup_route(5, 10, 700, ds)[0] == 11
    ids, sc = torch.full((10,), -9, dtype=torch.int32, device="cuda"), torch.full((10,), 9.0, device="cuda")
    ids, sc = B.ralm_cache_lookup(cids.cuda(), clen.cuda(), q.cuda(), off.cuda(), ds, **({} if own_outputs else dict(spec_ids=ids, spec_scores=sc)))
    ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
    for i, r in owner.items():
        wi, wsc = oracle.cache_lookup(cids[r:r + 1].numpy(), clen[r:r + 1].numpy(), q[i:i + 1].numpy(), np.array([0, 1]), X.numpy(), metric)
        assert ids[i] == wi[0] and sc[i] == wsc[0]
    for i in (0, 1, 9):
        assert (ids[i], sc[i]) == ((-1, -np.inf) if own_outputs else (-9, 9.0))
    for i in (4, 5):
        assert ids[i] in cids[0].tolist() + cids[3].tolist()


@pytest.mark.parametrize("dtype,d,metric,R,C,smax,route", [ROUTES[i] for i in (0, 1, 3, 7, 9)])
def test_split_lookups_replay_from_a_hip_graph(dtype, d, metric, R, C, smax, route):
    """Every replay equals the eager call on the same queries, with other work and waits between the replays."""
    from paper_2401_14021_amd import binding as B
    X, ds, cids, clen, q, off = _whole_numbers(dtype, d, metric, R, C, smax)
    cids, clen, q, off = cids.cuda(), clen.cuda(), q.cuda(), off.cuda()
    Q = q.shape[0]
    ws = torch.empty(Q, dtype=torch.int64, device="cuda")
    B.ralm_cache_lookup(cids, clen, q, off, ds, workspace=ws)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            ids, sc = B.ralm_cache_lookup(cids, clen, q, off, ds, workspace=ws)
    torch.cuda.synchronize()
    g = torch.Generator().manual_seed(1)
    for _ in range(4):
        q.copy_(torch.randint(-3, 4, (Q, d), generator=g).float())
        graph.replay()
        torch.cuda.synchronize()
        want = B.ralm_cache_lookup(cids, clen, q, off, ds)
        torch.cuda.synchronize()
        assert torch.equal(ids, want[0]) and torch.equal(sc, want[1])


@pytest.mark.parametrize("Qt", [200, 4096, 4097])
@pytest.mark.parametrize("d", [64, 72])
def test_unowned_queries_around_and_between_ranges(oracle, d, Qt):
    """Ranges of every alignment to the words of a bit map, some of them empty or out of order; what lies between two of them
    belongs to somebody unless a decreasing pair of offsets skips it."""
    from paper_2401_14021_amd import binding as B
    rng = np.random.default_rng(Qt + d)
    R, C, n = 40, 20, 500
    X = torch.from_numpy(rng.integers(-3, 4, size=(n, d)).astype(np.float32))
    q = torch.from_numpy(rng.integers(-3, 4, size=(Qt, d)).astype(np.float32))
    cids = torch.from_numpy(rng.integers(0, n, size=(R, C)).astype(np.int32))
    clen = torch.full((R,), C, dtype=torch.int32)
    ds = B.Datastore(X.cuda())
    lo = np.sort(rng.integers(3, 190, size=R - 1))
    for off in (np.concatenate([[3], lo, [190]]), np.concatenate([[160], np.sort(rng.integers(160, 180, size=R - 1)), [7]]),
                np.concatenate([[64, 96, 32], [32] * (R - 3), [63]])):
        owner = np.full(Qt, -1)
        for r in range(R):
            owner[off[r]:max(off[r], off[r + 1])] = r
        ids, sc = B.ralm_cache_lookup(cids.cuda(), clen.cuda(), q.cuda(), torch.from_numpy(off).cuda(), ds)
        assert B.ralm_lookup_route(R, Qt, C, ds) == (1, 4 if d == 64 else 0, Qt > 4096)
        ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
        assert (ids[owner < 0] == -1).all() and (sc[owner < 0] == -np.inf).all()
        mine = np.nonzero(owner >= 0)[0]
        wi, wsc = oracle.cache_lookup(cids.numpy()[owner[mine]], clen.numpy()[owner[mine]], q.numpy()[mine],
                                      np.arange(len(mine) + 1), X.numpy())
        np.testing.assert_array_equal(ids[mine], wi)
        np.testing.assert_array_equal(sc[mine], wsc)


@pytest.mark.parametrize("dtype,d,R,C,route", [
    ("f16", 1024, 171, 300, (3, 4)), ("f32", 768, 300, 600, (2, 8)), ("f32", 768, 300, 64, (1, 4)), ("f32", 192, 200, 1024, (3, 6)),
    ("f32", 192, 33, 700, (11, 4)), ("f32", 392, 171, 300, (3, 0)), ("f32", 1544, 100, 300, (2, 0)), ("f32", 392, 300, 300, (2, 0)),
])
def test_routes_of_the_k_best(oracle, dtype, d, R, C, route):
    from paper_2401_14021_amd import binding as B
    k = 9
    X, ds, cids, clen, q, off = _whole_numbers(dtype, d, "ip", R, C, 1)
    rng = np.random.default_rng(C)
    cids = torch.from_numpy(np.stack([rng.choice(len(X), size=C, replace=False) for _ in range(R)]).astype(np.int32))   # distinct
    assert B.ralm_lookup_route(R, q.shape[0], C, ds, k)[:2] == route
    ids, sc = B.ralm_cache_lookup_topk(cids.cuda(), clen.cuda(), q.cuda(), off.cuda(), ds, k)
    wi, wsc = oracle.cache_lookup_topk(cids.numpy(), clen.numpy(), q.numpy(), off.numpy(), X.numpy(), k)
    np.testing.assert_array_equal(ids.cpu().numpy(), wi)
    np.testing.assert_array_equal(sc.cpu().numpy(), wsc)
