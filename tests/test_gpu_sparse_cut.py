"""retain_sparse_kernel's search for s_(b) by a histogram of the leading 16 key bits, where it can go wrong: keys over more values than
it has bins, all in one bin and a low score, crowds of equal scores over the threshold, exactly as many survivors as places (which fit) and
one more (which are handed on); at the edges of the 4-, 8-, 12- and 16-slot instances.  Every pick against Eq. 2 in fp64 on the path's own prefix.
Heads that are cut at the capacity, and which heads the kernel finishes by itself: test_gpu_sparse_search.py."""
import pytest
import torch

import parity_util as P
from paper_2605_14292_amd import binding as B
from paper_2605_14292_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,b", [(257, 2), (1024, 64), (1025, 65), (2048, 128), (2049, 64), (3072, 128), (3073, 100), (4096, 128)])
def test_threshold_and_cut(n, b):
    g = torch.Generator().manual_seed(n + b)
    cap = 128 if b <= 64 else 192
    s = torch.zeros((6, n))
    s[0] = torch.exp(100 * torch.rand((n,), generator=g) - 50) * torch.sign(torch.randn((n,), generator=g))   # nearly all keys
    s[1] = 1.5 + 0.001 * torch.rand((n,), generator=g); s[1, n // 2] = -3.0                                   # one bin and a low score
    s[2] = torch.floor(4 * torch.rand((n,), generator=g))                                                     # crowds of equal scores
    for h, k in ((3, cap), (4, cap + 1)):                                                                     # survivors
        s[h, torch.randperm(n, generator=g)[:k]] = 10 + 0.3 * torch.rand((k,), generator=g)
    s[5] = torch.randn((n,), generator=g).exp()
    V = torch.randn((6, n, 128), generator=g)
    V[:, n // 2:n // 2 + n // 4] = V[:, :n // 4] + 0.05 * V[:, n // 2:n // 2 + n // 4]
    K = torch.randn((6, n, 128), generator=g).to(torch.bfloat16).to(DEV)
    V, s = V.to(torch.bfloat16).to(DEV), s.to(DEV)
    out = B.kvr_retain(K, V, b, .5, 1e-6, s=s)
    torch.cuda.synchronize()
    with B.bounds_checked_library():
        B.kvr_debug_bounds_violation()
        dbg = B.kvr_retain(K, V, b, .5, 1e-6, s=s)
        torch.cuda.synchronize()
        assert B.kvr_debug_bounds_violation() == 0
    assert torch.equal(out.pick_order, dbg.pick_order) and torch.equal(out.pick_gain, dbg.pick_gain)
    for h in range(6):
        idx = out.idx_sorted[h].long()
        P.check_head(W.to_f64(s[h]), W.to_f64(V[h]), b, .5, 1e-6, out.pick_order[h].cpu().numpy(), out.pick_gain[h].cpu().numpy(),
                     idx.cpu().numpy())
        assert torch.equal(out.V_out[h], V[h][idx]) and torch.equal(out.K_out[h], K[h][idx])
