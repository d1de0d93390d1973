"""Flat signatures for group sizes whose eight slices end in every kind of load batch (1, 2, 3, 8, 9, 14, 16, 17, 25 heads a slice,
and slices left without heads), against the mean in fp64."""
import pytest
import torch

from paper_2605_14292_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("group", [1, 7, 9, 16, 23, 64, 71, 112, 127, 130, 193])
def test_mean_over_the_group(group, dtype):
    seqs, n = 2, 5
    g = torch.Generator().manual_seed(group)
    V = torch.randn((seqs * group, n, 128), generator=g).to(dtype).cuda()
    u = B.kvr_signature_flat(V, group)
    torch.cuda.synchronize()
    want = V.double().view(seqs, group, n, 128).mean(1)
    # group - 1 fp32 additions and one product: at most group roundings of 2^-24 on sums of at most the sum of magnitudes
    bound = (group + 1) * 2**-24 * V.double().abs().view(seqs, group, n, 128).mean(1)
    assert bool(((u.double() - want).abs() <= bound + 1e-12).all())
