"""The exact pass on both sides of the number of queries up to which its scan ranks them itself: both forms of the scan, k' = k, which
leaves no margin, so that most queries take the pass; k up to the longest sort, and an answer that is the whole datastore."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Q", [1, 7, 8, 9])
@pytest.mark.parametrize("N,d,dtype,metric,k", [(30_000, 768, "f32", "ip", 20), (30_000, 72, "f32", "ip", 1024), (70_001, 128, "f16", "ip", 100),
                                                (9_000, 136, "f16", "ip", 3), (20_000, 64, "f32", "l2", 64), (300, 64, "f32", "ip", 300)])
def test_exact_pass(oracle, Q, N, d, dtype, metric, k):
    from paper_2401_14021_amd import binding as B
    g = torch.Generator().manual_seed(N + Q)
    X = torch.randn(N, d, generator=g).to(torch.float16 if dtype == "f16" else torch.float32)
    q = torch.randn(Q, d, generator=g)
    ds = B.Datastore.for_l2(X.cuda(), torch.bfloat16) if metric == "l2" else (
        B.Datastore(X.cuda()) if dtype == "f16" else B.Datastore.from_fp32(X.cuda(), torch.bfloat16))
    ws = B.alloc_workspace(Q, ds, k, k)
    wi, wsc = oracle.retrieve_topk(q.numpy(), X.float().numpy(), k, metric=metric)
    passes = 0
    for _ in range(2):   # the second call finds the counters of the first in its workspace
        ids, sc = B.ralm_retrieve_topk_ex(q.cuda(), ds, k, k, workspace=ws)
        c = B.ralm_workspace_counters(ws)
        passes += c["exact_pass"]
        assert c["unanswered"] == 0
        np.testing.assert_array_equal(ids.cpu().numpy(), wi)
        np.testing.assert_array_equal(sc.cpu().numpy(), wsc)
    assert passes > 0 or k == N
