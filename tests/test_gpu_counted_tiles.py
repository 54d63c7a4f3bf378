"""Launches that count a tile's admitted scores, in every width of the query tile and every type of row.  Whole numbers: many scores equal
the admission key's, and ids and scores are the exact ones, equal scores by lower id."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("Q", [1, 32, 33, 64, 65, 128, 129])
@pytest.mark.parametrize("N,d,k", [(130_001, 64, 200), (130_049, 136, 500)])
def test_counted(oracle, N, d, k, Q, dtype):
    from paper_2401_14021_amd import binding as B
    g = torch.Generator().manual_seed(N + Q)
    X = torch.randint(-3, 4, (N, d), generator=g).float()
    q = torch.randint(-3, 4, (Q, d), generator=g).float()
    Xd = X.cuda()
    ds = B.Datastore(Xd) if dtype == "f32" else B.Datastore.from_fp32(Xd, torch.bfloat16 if dtype == "bf16" else torch.float16)
    assert "counted" in B.ralm_scan_routes(Q, ds, k)
    ws = B.alloc_workspace(Q, ds, k)
    ids, sc = B.ralm_retrieve_topk_ex(q.cuda(), ds, k, workspace=ws)
    c = B.ralm_workspace_counters(ws)
    assert c["ladder_overflows"] == 0 and c["unanswered"] == 0 and c["exact_pass"] == 0, c
    full = Xd.double() @ q.double().cuda().T
    key = full * 2 ** 19 + (N - torch.arange(N, device="cuda", dtype=torch.float64))[:, None]
    assert torch.equal(ids.long(), key.topk(k, dim=0).indices.T)
    picked = list(range(0, Q, max(1, Q // 4)))
    wi, wsc = oracle.retrieve_topk(q[picked].numpy(), X.numpy(), k)
    np.testing.assert_array_equal(ids.cpu().numpy()[picked], wi)
    np.testing.assert_array_equal(sc.cpu().numpy()[picked], wsc)
