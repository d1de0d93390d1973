"""Batched short heads, several per workgroup, at the edges of the tile counts: the pipeline over a workgroup's heads
(first head, middle, last, a round that not every workgroup takes part in) against the oracle pick by pick."""
import numpy as np
import pytest
import torch

from oracle import alpha_oracle as O
import parity_util as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,b,G,lam", [(1, 1, 2, 0.5), (31, 9, 8, 0.5), (64, 64, 1, 0.25), (65, 20, 0, 0.5), (128, 128, 3, 0.5),
                                       (129, 64, 7, 1.0), (192, 190, 0, 0.5), (193, 50, 8, 0.5), (256, 256, 2, 0.5), (256, 40, 5, 0.0)])
def test_batched_short_heads_at_tile_edges(n, b, G, lam):
    from paper_2605_14292_amd import binding as B
    heads = 2100                                         # more than four per CU
    g = torch.Generator(device="cuda").manual_seed(n * 7 + b)
    K = torch.randn((heads, n, 128), generator=g, device="cuda").to(torch.bfloat16)
    V = torch.randn((heads, n, 128), generator=g, device="cuda").to(torch.bfloat16)
    V[:, n // 2:n // 2 + n // 3] = V[:, : n // 3]
    Q = torch.randn((heads, G, 128), generator=g, device="cuda").to(torch.bfloat16) if G else None
    s = None if G else torch.rand((heads, n), generator=g, device="cuda") * 0.01       # far below lambda: nothing to drop
    out = B.kvr_retain(K, V, b, lam, 1e-6, Q=Q, s=s)
    torch.cuda.synchronize()
    idx = out.idx_sorted.cpu().numpy()
    assert idx.min() >= 0 and idx.max() < n and np.all(np.diff(idx, axis=1) > 0)
    assert torch.equal(out.K_out, torch.gather(K, 1, out.idx_sorted.long().unsqueeze(-1).expand(-1, -1, 128)))
    assert torch.equal(out.V_out, torch.gather(V, 1, out.idx_sorted.long().unsqueeze(-1).expand(-1, -1, 128)))
    for h in (0, 255, 256, 767, 768, 1024, 2048, 2099):
        K64, V64 = K[h].double().cpu().numpy(), V[h].double().cpu().numpy()
        if G:
            s64 = O.score_softmax_mean(K64, Q[h].double().cpu().numpy())
            P.check_scores(out.s_out[h].cpu().numpy(), s64)
        else:
            s64 = s[h].double().cpu().numpy()
        P.check_head(s64, V64, b, lam, 1e-6, out.pick_order[h].cpu().numpy(), out.pick_gain[h].cpu().numpy(), idx[h])
