"""select_dense_f32_kernel at the edges of its 16x16 Gram tiles, whole and after the score bound has shortened the head (the tiles are
those of the tokens that are left): every pick against Eq. 2 in fp64 on the path's own prefix."""
import pytest
import torch

import parity_util as P
from paper_2605_14292_amd import binding as B
from paper_2605_14292_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,b,left", [(1, 1, 1), (2, 2, 2), (15, 7, 15), (16, 16, 16), (17, 5, 17), (33, 33, 33), (48, 10, 48), (65, 64, 65),
                                      (128, 60, 128), (129, 128, 129), (192, 64, 192), (193, 100, 193), (255, 128, 255), (256, 256, 256),
                                      (256, 16, 16), (256, 16, 17), (200, 40, 49), (193, 100, 112), (64, 2, 3)])
def test_tile_edges(n, b, left):
    g = torch.Generator().manual_seed(1000 * n + b + left)
    V = torch.randn((3, n, 128), generator=g)
    V[:, n // 2:] = V[:, :n - n // 2] + 0.05 * V[:, n // 2:]
    K = torch.randn((3, n, 128), generator=g).to(DEV)
    s = torch.full((3, n), -4.0)
    for h in range(3):                                   # `left` tokens within lambda of the best
        s[h, torch.randperm(n, generator=g)[:left]] = 0.2 * torch.rand((left,), generator=g)
    V, s = V.to(DEV), s.to(DEV)
    out = B.kvr_retain(K, V, b, .5, 1e-6, s=s)
    torch.cuda.synchronize()
    for h in range(3):
        idx = out.idx_sorted[h].long()
        P.check_head(W.to_f64(s[h]), W.to_f64(V[h]), b, .5, 1e-6, out.pick_order[h].cpu().numpy(), out.pick_gain[h].cpu().numpy(),
                     idx.cpu().numpy())
        assert torch.equal(out.V_out[h], V[h][idx]) and torch.equal(out.K_out[h], K[h][idx])
