"""Heads of 193-256 tokens: the next head's Gram beside the pick chain or between two chains.  The rule that chooses, at measured shapes,
and both kernels on the same heads at the rule's edges: the same bits."""
import ctypes

import pytest
import torch

from paper_2605_14292_amd import binding as B

DEV = "cuda:0"


# (heads, n, b, queries): which of the two was faster on 256 CUs
@pytest.mark.parametrize("heads,n,b,queries,ahead", [
    (2688, 256, 2, False, False), (2688, 200, 48, False, False), (2688, 256, 56, False, False), (2688, 200, 64, False, True), (700, 224, 128, False, True),
    (257, 200, 64, False, False), (512, 240, 128, False, False),
    (257, 256, 48, True, False), (257, 200, 56, True, True), (400, 256, 64, True, True), (700, 200, 24, True, False), (700, 256, 56, True, False),
    (1024, 224, 48, True, False), (1024, 193, 64, True, True), (1536, 256, 24, True, False), (2688, 251, 101, True, True),
    (3072, 256, 2, True, True), (3072, 240, 40, True, True), (4096, 193, 24, True, True), (4096, 193, 40, True, False), (6144, 224, 56, True, False)])
def test_the_faster_one_is_chosen(heads, n, b, queries, ahead):
    rule = getattr(B.lib(), "_ZN3kvr15gram_ahead_paysEiiibi")      # kvr::gram_ahead_pays
    rule.restype = ctypes.c_bool
    assert rule(ctypes.c_int(heads), ctypes.c_int(n), ctypes.c_int(b), ctypes.c_bool(queries), ctypes.c_int(256)) == ahead


@pytest.mark.gpu
@pytest.mark.parametrize("n,G", [(193, 7), (224, 1), (240, 8), (256, 3), (255, 0)])
def test_both_give_the_same_bits(n, G):
    heads = 1000 if G else 700                                   # more than two heads per CU on either side of b = 64
    g = torch.Generator(device=DEV).manual_seed(n)
    K = torch.randn((heads, n, 128), generator=g, device=DEV).to(torch.bfloat16)
    V = torch.randn((heads, n, 128), generator=g, device=DEV).to(torch.bfloat16)
    V[:, n // 2:n // 2 + n // 3] = V[:, :n // 3]
    Q = torch.randn((heads, G, 128), generator=g, device=DEV).to(torch.bfloat16) if G else None
    s = None if G else torch.rand((heads, n), generator=g, device=DEV) * 0.01       # far below lambda: nothing to drop
    outs = {b: B.kvr_retain(K, V, b, .5, 1e-6, Q=Q, s=s) for b in (63, 64, 150)}
    torch.cuda.synchronize()
    for b in (63, 64):                                           # a pick depends on the earlier ones only
        assert torch.equal(outs[b].pick_order, outs[150].pick_order[:, :b])
        assert torch.equal(outs[b].pick_gain.view(torch.int32), outs[150].pick_gain[:, :b].contiguous().view(torch.int32))
        assert torch.equal(outs[b].idx_sorted, torch.sort(outs[b].pick_order, dim=1).values)
        if G:
            assert torch.equal(outs[b].s_out.view(torch.int32), outs[150].s_out.view(torch.int32))
    for h in (0, 256, heads - 1):
        assert torch.equal(outs[63].V_out[h], V[h][outs[63].idx_sorted[h].long()])


@pytest.mark.gpu
def test_both_give_the_same_bits_on_either_side_of_two_heads_per_cu():
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    heads, n, b = 2 * cus + 1, 230, 96
    g = torch.Generator(device=DEV).manual_seed(5)
    K = torch.randn((heads, n, 128), generator=g, device=DEV).to(torch.bfloat16)
    V = torch.randn((heads, n, 128), generator=g, device=DEV).to(torch.bfloat16)
    s = torch.rand((heads, n), generator=g, device=DEV) * 0.01
    many = B.kvr_retain(K, V, b, .5, 1e-6, s=s)
    few = B.kvr_retain(K[:-1], V[:-1], b, .5, 1e-6, s=s[:-1])
    torch.cuda.synchronize()
    assert torch.equal(many.pick_order[:-1], few.pick_order) and torch.equal(many.pick_gain[:-1].contiguous().view(torch.int32), few.pick_gain.view(torch.int32))
    assert torch.equal(many.V_out[:-1], few.V_out) and torch.equal(many.K_out[:-1], few.K_out)
