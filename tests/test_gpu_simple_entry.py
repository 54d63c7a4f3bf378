"""The simple entry point learns from a word in host memory that a query was left unanswered, and redoes the call block by block."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Q", [1, 9, 800])
def test_more_equal_rows_than_a_list_holds(Q):
    from paper_2401_14021_amd import binding as B
    g = torch.Generator().manual_seed(Q)
    X = torch.randint(-3, 4, (60_000, 64), generator=g).float().cuda()
    q = torch.randint(1, 4, (Q, 64), generator=g).float().cuda()

    def check(rows):
        ids, sc = B.ralm_retrieve_topk(q, rows, 5)
        full = rows.double() @ q.double().T
        want = (full * 2 ** 16 + (2 ** 16 - 1 - torch.arange(len(rows), device="cuda", dtype=torch.float64))[:, None]).topk(5, dim=0).indices.T
        np.testing.assert_array_equal(ids.cpu().numpy(), want.cpu().numpy())
        np.testing.assert_array_equal(sc.cpu().numpy(), full.T.gather(1, want).float().cpu().numpy())

    check(X)
    equal = X.clone()
    equal[7:50_007] = 3.0            # every query's best rows, 50000 of them
    check(equal)
    check(X)                         # the word is clear again
    B.lib().ralm_release_buffers()
    check(equal)                     # ... and is there again
    check(X)
