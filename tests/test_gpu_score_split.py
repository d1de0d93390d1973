"""Wide-window scores at the edges of the split over workgroups: whole and ragged last tiles, the shortest head that is
split, one query block and eight, and few heads against many (which take both passes in one launch)."""
import numpy as np
import pytest
import torch

from oracle import alpha_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,n,G", [(1, 1505, 33), (2, 1536, 256), (3, 1537, 64), (2, 2047, 224), (1, 8192, 256), (2, 4000, 97),
                                       (128, 1601, 40), (129, 1601, 40), (2, 1504, 33)])
def test_wide_scores_match_the_oracle_on_either_side_of_the_split(heads, n, G):
    from paper_2605_14292_amd import binding as B
    g = torch.Generator().manual_seed(n + G)
    K = torch.randn((heads, n, 128), generator=g).to(torch.bfloat16)
    Q = torch.randn((heads, G, 128), generator=g).to(torch.bfloat16)
    s_out = torch.full((heads, n), float("nan"), device="cuda")
    B.kvr_score(K.cuda(), Q.cuda(), s_out=s_out)
    torch.cuda.synchronize()
    for h in {0, heads - 1}:
        want = O.score_softmax_mean(K[h].double().numpy(), Q[h].double().numpy())
        # exact products, fp32 sums of 128 terms of order one: logits good to 1e-6, so scores to a few 1e-6 relative
        np.testing.assert_allclose(s_out[h].cpu().numpy(), want, rtol=2e-5)


# a whole number of query blocks, and ones filled up with other rows; split over workgroups, and in one launch
@pytest.mark.parametrize("heads", [2, 140])
@pytest.mark.parametrize("G", [33, 64, 97, 224])
def test_a_split_without_a_finite_logit_counts_for_nothing(heads, G):
    from paper_2605_14292_amd import binding as B
    n = 4000
    g = torch.Generator().manual_seed(5)
    K = torch.randn((heads, n, 128), generator=g).to(torch.bfloat16)
    Q = torch.randn((heads, G, 128), generator=g).to(torch.bfloat16)
    Q[:, :, 0] = 1.0
    K[:, :2500, 0] = -float("inf")                       # logits of -inf: these tokens score zero
    s_out = B.kvr_score(K.cuda(), Q.cuda())
    torch.cuda.synchronize()
    for h in {0, heads - 1}:
        want = O.score_softmax_mean(K[h].double().numpy(), Q[h].double().numpy())
        assert np.all(want[:2500] == 0) and abs(want.sum() - 1) < 1e-12
        np.testing.assert_allclose(s_out[h].cpu().numpy(), want, rtol=2e-5)


# heads above 4096 tokens whose logits fill a CU's LDS: the fewest heads that take one workgroup of sixteen waves, the most
# logits it holds, and one head and one token more or less (which score_wide_kernel takes)
@pytest.mark.parametrize("heads,n,G", [(103, 8192, 4), (102, 8192, 4), (103, 5814, 7), (103, 5815, 7), (104, 6145, 4), (104, 5057, 8)])
def test_scores_of_one_pass_match_the_oracle(heads, n, G):
    from paper_2605_14292_amd import binding as B
    g = torch.Generator().manual_seed(n + G)
    K = torch.randn((heads, n, 128), generator=g).to(torch.bfloat16)
    Q = torch.randn((heads, G, 128), generator=g).to(torch.bfloat16)
    s_out = torch.full((heads, n), float("nan"), device="cuda")
    B.kvr_score(K.cuda(), Q.cuda(), s_out=s_out)
    torch.cuda.synchronize()
    for h in {0, heads - 1}:
        want = O.score_softmax_mean(K[h].double().numpy(), Q[h].double().numpy())
        np.testing.assert_allclose(s_out[h].cpu().numpy(), want, rtol=2e-5)   # (the bound above)
