"""Cache updates whose new ids go into the ring all at once: hardly any of them waits in the slots to be overwritten.  Up to 12 new ids
of 64 are settled in order, more together; caches with fewer free slots than new ids, rings of up to 64 slots that are gone
round, repeats inside a batch.  Whole numbers: every slot must be the oracle's."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_new", [1, 12, 13, 40, 63, 64])       # different ids among 64 candidates
@pytest.mark.parametrize("C", [5, 40, 63, 64, 65, 100, 300, 2048])
def test_new_ids_together(oracle, C, n_new):
    from paper_2401_14021_amd import binding as B
    rng = np.random.default_rng(C * 100 + n_new)
    R, k, steps, N = 20, 32, 5, 1_000_000                        # 160 candidates: two batches of 64 and a half
    off = (np.arange(R + 1) * steps).astype(np.int64)
    truth = np.empty((R, steps * k), np.int32)
    for r in range(R):
        for b in range(0, steps * k, 64):
            m = min(64, steps * k - b)
            ids = rng.choice(N, size=min(n_new, m), replace=False)
            truth[r, b:b + m] = rng.permutation(np.concatenate([ids, rng.choice(ids, size=m - len(ids))]))
    truth = truth.reshape(R * steps, k)
    truth[rng.random(truth.shape) < 0.02] = -1
    lens = np.array([max(0, C - x) for x in rng.choice([0, 3, 20, 70, C], size=R)], dtype=np.int32)
    heads = np.array([rng.integers(0, C) if n == C else 0 for n in lens], dtype=np.int32)
    cache = np.full((R, C), -1, dtype=np.int32)
    for r in range(R):
        cache[r, :lens[r]] = rng.choice(N, size=lens[r], replace=False)
        known = rng.integers(0, steps * k, size=6)               # some candidates are cached already
        cache[r, :min(6, lens[r])] = np.maximum(truth[r * steps:(r + 1) * steps].reshape(-1)[known], 0)[:min(6, lens[r])]
    for p, n_next in ((k, 0), (3, 10)):
        wi, wl, wh = oracle.cache_insert(cache, lens, heads, truth, off, N=N, p=p, n_next=n_next)
        dc, dl, dh = (torch.from_numpy(x.copy()).cuda() for x in (cache, lens, heads))
        B.ralm_cache_insert(dc, dl, dh, torch.from_numpy(truth).cuda(), torch.from_numpy(off).cuda(), N, p=p, n_next=n_next)
        assert np.array_equal(dl.cpu().numpy(), wl) and np.array_equal(dh.cpu().numpy(), wh)
        got = dc.cpu().numpy()
        for r in range(R):
            assert np.array_equal(got[r, :wl[r]], wi[r, :wl[r]]), r


@pytest.mark.parametrize("at", [(0,), (7,), (8,), (31, 40), (63,), (120,), tuple(range(0, 160, 3))])   # places of ids that wait to be evicted
@pytest.mark.parametrize("C", [16, 40, 63, 64, 65, 100, 500])
def test_new_ids_and_ids_that_wait_to_be_evicted(oracle, C, at):
    """Full rings: what is in one of the next 64 slots is a member or not by what was put in before it is asked for."""
    from paper_2401_14021_amd import binding as B
    rng = np.random.default_rng(C + len(at) + at[0])
    R, k, N = 12, 160, 1_000_000
    off = np.arange(R + 1).astype(np.int64)
    cache = np.stack([rng.choice(N // 2, size=C, replace=False) for _ in range(R)]).astype(np.int32)
    heads = rng.integers(0, C, size=R).astype(np.int32)
    lens = np.full(R, C, dtype=np.int32)
    truth = np.stack([N // 2 + rng.choice(N // 2, size=k, replace=False) for _ in range(R)]).astype(np.int32)
    for r in range(R):
        truth[r, list(at)] = cache[r, (heads[r] + rng.integers(0, min(C, 64), size=len(at))) % C]
        if r % 3 == 0:
            truth[r, 70:] = truth[r, rng.integers(0, 70, size=90)]       # few different ones
    wi, wl, wh = oracle.cache_insert(cache, lens, heads, truth, off, N=N, p=k, n_next=0)
    dc, dl, dh = (torch.from_numpy(x.copy()).cuda() for x in (cache, lens, heads))
    B.ralm_cache_insert(dc, dl, dh, torch.from_numpy(truth).cuda(), torch.from_numpy(off).cuda(), N, p=k)
    np.testing.assert_array_equal(dl.cpu().numpy(), wl)
    np.testing.assert_array_equal(dh.cpu().numpy(), wh)
    np.testing.assert_array_equal(dc.cpu().numpy(), wi)
