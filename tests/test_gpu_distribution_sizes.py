"""Neighbour distributions around the lines between their kernels: 512 entries, 1024 queries."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Q", [1, 1024, 1025])
@pytest.mark.parametrize("k", [511, 512, 513, 1023, 1024])
def test_sizes(oracle, k, Q):
    from paper_2401_14021_amd import binding as B
    rng = np.random.default_rng(Q + k)
    N, V = 20000, 700
    values = rng.integers(0, V, size=N).astype(np.int32)
    ids = rng.integers(0, N, size=(Q, k)).astype(np.int32)
    sc = np.sort((rng.standard_normal((Q, k)) * 4 - 900).astype(np.float32), axis=1)[:, ::-1].copy()
    ids[:, -2:] = np.where(np.arange(Q)[:, None] % 3 == 0, -1, ids[:, -2:])
    sc[Q // 2] = sc[Q // 2, 0]
    tok, w, top, p = oracle.knnlm_probs(ids, sc, values, 1.0)
    got = [t.cpu().numpy() for t in B.ralm_knnlm_probs(torch.from_numpy(ids).cuda(), torch.from_numpy(sc).cuda(), torch.from_numpy(values).cuda(), 1.0)]
    np.testing.assert_array_equal(got[0], tok)
    np.testing.assert_array_equal(got[2], top)
    np.testing.assert_allclose(got[1], w, rtol=1e-6, atol=1e-30)     # double sums in another order, rounded to fp32 once
    np.testing.assert_allclose(got[3], p, rtol=1e-6)


def test_time_of_many_queries_follows_the_entries():
    """2048 queries with 513 entries, which are sorted as 1024, against 512: 1.6 times the time.  Workgroups of which a CU holds two
    instead of eight take 3.6 times as long."""
    from paper_2401_14021_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(1)
    values = torch.randint(0, 30000, (100_000,), generator=g, device="cuda", dtype=torch.int32)

    def calls(k):
        ids = torch.randint(0, 100_000, (2048, k), generator=g, device="cuda", dtype=torch.int32)
        sc = torch.randn(2048, k, generator=g, device="cuda")
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        times = []
        for _ in range(9):
            a.record()
            for _ in range(40):
                B.ralm_knnlm_probs(ids, sc, values, 1.0)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    assert calls(513) < 2.5 * calls(512)
