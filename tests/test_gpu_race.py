"""The race over a triangle of cosines at the edges of its slots: gains that are exact in fp32 (one-hot value rows,
scores that are multiples of 1/64), so that every pick is decided by equality or by the tie rule, and the order must be
the oracle's pick by pick."""
import numpy as np
import pytest
import torch

from oracle import alpha_oracle as O

pytestmark = pytest.mark.gpu


# heads <= CUs: sixteen waves per head; 300 heads: the persistent kernels; n > 256: against the bound of the outside tokens
@pytest.mark.parametrize("heads,n,b", [
    (2, 33, 33), (2, 64, 50), (2, 65, 64), (2, 128, 65), (2, 129, 100), (2, 192, 128), (2, 193, 193), (2, 256, 256),
    (300, 64, 64), (300, 130, 64), (300, 192, 65), (300, 256, 128), (3, 257, 64), (3, 513, 128), (3, 1025, 65), (2, 700, 200)])
@pytest.mark.parametrize("levels", [3, 40])
def test_exact_gains_and_ties_give_the_oracles_order(heads, n, b, levels):
    from paper_2605_14292_amd import binding as B
    g = torch.Generator().manual_seed(1000 * n + b + levels)
    s = torch.randint(0, levels, (heads, n), generator=g).float() / 64
    V = torch.zeros((heads, n, 128))
    V.scatter_(2, torch.randint(0, 100, (heads, n, 1), generator=g), 1.0)
    V = V.to(torch.bfloat16)
    idx, order, gain = B.kvr_select_greedy(V.cuda(), s.cuda(), b, 0.25, 0.0)
    torch.cuda.synchronize()
    for h in range(heads) if heads < 10 else range(0, heads, 60):
        want = O.alpha_select(s[h].double().numpy(), V[h].double().numpy(), b, 0.25, 0.0)
        np.testing.assert_array_equal(order[h].cpu().numpy(), want["order"])
        np.testing.assert_array_equal(gain[h].cpu().numpy().astype(np.float64), want["gain"])
        np.testing.assert_array_equal(idx[h].cpu().numpy(), np.sort(want["order"]))


# long fp32 heads, either side of every step in the number of token slots a wave holds
@pytest.mark.parametrize("n", [257, 512, 513, 1024, 1025, 1536, 1537])
@pytest.mark.parametrize("b", [65, 128])
def test_long_fp32_heads_at_the_edges_of_the_slots(n, b):
    from paper_2605_14292_amd import binding as B
    g = torch.Generator().manual_seed(n + b)
    s = torch.randint(0, 12, (3, n), generator=g).float() / 64
    V = torch.zeros((3, n, 128))
    V.scatter_(2, torch.randint(0, 100, (3, n, 1), generator=g), 1.0)
    idx, order, gain = B.kvr_select_greedy(V.cuda(), s.cuda(), b, 0.25, 0.0)
    torch.cuda.synchronize()
    for h in range(3):
        want = O.alpha_select(s[h].double().numpy(), V[h].double().numpy(), b, 0.25, 0.0)
        np.testing.assert_array_equal(order[h].cpu().numpy(), want["order"])
        np.testing.assert_array_equal(gain[h].cpu().numpy().astype(np.float64), want["gain"])
        np.testing.assert_array_equal(idx[h].cpu().numpy(), np.sort(want["order"]))
