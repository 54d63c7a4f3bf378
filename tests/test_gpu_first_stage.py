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
