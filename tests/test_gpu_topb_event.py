"""The lambda = 0 event with scores from queries (one launch where the logits fit) and with scores handed in, at the edges of the
instances: picks against a stable sort of the returned scores, kept rows bit for bit, ties across the budget's edge."""
import numpy as np
import pytest
import torch

from paper_2605_14292_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,b,G", [(257, 1, 7), (300, 64, 8), (512, 65, 1), (513, 512, 7), (1024, 128, 7), (1025, 64, 4), (1950, 33, 7),
                                   (1951, 33, 7), (2049, 1000, 4), (3413, 64, 4), (3414, 64, 4), (1024, 1024, 3), (700, 20, 9)])
@pytest.mark.parametrize("tied", [False, True])
def test_top_b(n, b, G, tied):
    heads = 3
    g = torch.Generator().manual_seed(n + b)
    K = torch.randn((heads, n, 128), generator=g)
    if tied:                                       # every row eight times: equal scores in every stretch of the order
        K = K[:, torch.arange(n) // 8]
    K = K.to(torch.bfloat16).to(DEV)
    V = torch.randn((heads, n, 128), generator=g).to(torch.bfloat16).to(DEV)
    Q = torch.randn((heads, G, 128), generator=g).to(torch.bfloat16).to(DEV)
    out = B.kvr_retain(K, V, b, 0.0, 1e-6, Q=Q)
    s = B.kvr_score(K, Q)
    again = B.kvr_retain(K, V, b, 0.0, 1e-6, s=s)
    torch.cuda.synchronize()
    assert torch.equal(out.s_out, s)
    for o in (out, again):
        for h in range(heads):
            sc = s[h].cpu().numpy()
            want = np.argsort(-sc, kind="stable")[:b]
            np.testing.assert_array_equal(o.pick_order[h].cpu().numpy(), want)
            np.testing.assert_array_equal(o.pick_gain[h].cpu().numpy(), sc[want])
            idx = np.sort(want)
            np.testing.assert_array_equal(o.idx_sorted[h].cpu().numpy(), idx)
            sel = torch.from_numpy(idx).to(DEV)
            assert torch.equal(o.K_out[h], K[h][sel]) and torch.equal(o.V_out[h], V[h][sel])
