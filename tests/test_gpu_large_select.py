"""select_large_kernel (bf16 heads of 4097 to 8192 tokens) at the edges of its instances, chunks and
lists, every pick against Eq. 2 in fp64 on the path's own prefix, and the bounds-checked build's outputs bit for bit."""
import numpy as np
import pytest
import torch

import parity_util as P
from paper_2605_14292_amd import binding as B
from paper_2605_14292_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _inputs(heads, n, kind, seed, pad=0):
    g = torch.Generator().manual_seed(seed)
    V = torch.randn((heads, n, 128), generator=g)
    V[:, n // 2:n // 2 + n // 4] = V[:, :n // 4] + 0.05 * V[:, n // 2:n // 2 + n // 4]
    s = torch.softmax(torch.randn((heads, n), generator=g), 1)               # far below lambda: nothing to drop
    if kind == "wide":                                                       # the score bound drops most of the head
        s = torch.randn((heads, n), generator=g).exp()
    elif kind == "tied":                                                     # a crowd of equal bounds: lists of two turns
        s = torch.full((heads, n), 0.25)
        s[:, ::7] = 0.2500001
        V[:, : n // 3] = V[:, :1]
    full = torch.zeros((heads, n, 128 + pad), dtype=torch.bfloat16)
    full[:, :, :128] = V.to(torch.bfloat16)
    K = torch.randn((heads, n, 128), generator=g).to(torch.bfloat16)
    return K.to(DEV), full.to(DEV)[:, :, :128], s.to(DEV)


@pytest.mark.parametrize("n,b,kind,lam", [
    (4097, 129, "tight", .5), (4160, 64 * 4, "tight", 1.), (6000, 1024, "tight", .5), (4097, 1, "tight", .5), (4097, 2, "wide", .5),
    (5000, 65, "tight", .25), (8192, 1024, "tight", .5), (8191, 1023, "wide", .5), (4609, 640, "tied", 3.), (8192, 200, "tied", 1.)])
def test_picks_and_rows(n, b, kind, lam):
    K, V, s = _inputs(2, n, kind, n + b)
    out = B.kvr_retain(K, V, b, lam, 1e-6, s=s)
    torch.cuda.synchronize()
    with B.bounds_checked_library():
        B.kvr_debug_bounds_violation()
        dbg = B.kvr_retain(K, V, b, lam, 1e-6, s=s)
        torch.cuda.synchronize()
        assert B.kvr_debug_bounds_violation() == 0
    for f in ("idx_sorted", "pick_order", "pick_gain", "K_out", "V_out"):
        assert torch.equal(getattr(out, f), getattr(dbg, f)), f
    for h in range(2):
        idx = out.idx_sorted[h].long()
        P.check_head(W.to_f64(s[h]), W.to_f64(V[h]), b, lam, 1e-6, out.pick_order[h].cpu().numpy(),
                     out.pick_gain[h].cpu().numpy(), idx.cpu().numpy())
        assert torch.equal(out.V_out[h], V[h][idx]) and torch.equal(out.K_out[h], K[h][idx])


@pytest.mark.parametrize("n,b", [(5000, 300), (8192, 700)])
def test_per_head_budgets_are_prefixes(n, b):
    K, V, s = _inputs(6, n, "tight", n)
    b_h = torch.tensor([0, 1, 64, 65, b - 1, b], dtype=torch.int32, device=DEV)
    full = B.kvr_retain(K, V, b, .5, 1e-6, s=s)
    cut = B.kvr_retain_budgeted(K, V, b, .5, 1e-6, s=s, b_h=b_h)
    torch.cuda.synchronize()
    for h, k in enumerate(b_h.tolist()):
        assert torch.equal(cut.pick_order[h, :k], full.pick_order[h, :k]) and bool((cut.pick_order[h, k:] == -1).all())
        idx = cut.idx_sorted[h, :k].long()
        np.testing.assert_array_equal(idx.cpu().numpy(), np.sort(full.pick_order[h, :k].cpu().numpy()))
        assert torch.equal(cut.V_out[h, :k], V[h][idx])


@pytest.mark.parametrize("n,b,every", [(5000, 300, 5), (8192, 1024, 1), (4097, 260, 20), (8192, 700, 12)])
def test_many_infinite_scores(n, b, every):
    """More scores of +inf than a wave has places in the pool: they are picked first, in token order, and Eq. 2 goes on from there."""
    K, V, s = _inputs(2, n, "tight", n + every)
    s[0, ::every] = float("inf")
    out = B.kvr_retain(K, V, b, .5, 1e-6, s=s)
    torch.cuda.synchronize()
    P.check_infinite_first(W.to_f64(s[0]), W.to_f64(V[0]), b, .5, 1e-6, out.pick_order[0].cpu().numpy(), out.pick_gain[0].cpu().numpy())
    P.check_head(W.to_f64(s[1]), W.to_f64(V[1]), b, .5, 1e-6, out.pick_order[1].cpu().numpy(), out.pick_gain[1].cpu().numpy(),
                 out.idx_sorted[1].cpu().numpy())


@pytest.mark.parametrize("n,b,kind", [(8192, 1024, "tight"), (5000, 400, "tied")])
def test_runs_repeat_bit_for_bit(n, b, kind):
    """The order of a refresh list decides which products a token meets, and with them its last bits: the same heads again, on
    another stream, and each head at another place of the call."""
    heads = 8
    K, V, s = (x.repeat((heads // 2,) + (1,) * (x.dim() - 1)) for x in _inputs(2, n, kind, n - b))
    a = B.kvr_retain(K, V, b, .5, 1e-6, s=s)
    torch.cuda.synchronize()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        c = B.kvr_retain(K, V, b, .5, 1e-6, s=s, stream=st)
    st.synchronize()
    for f in ("idx_sorted", "pick_order", "pick_gain", "K_out", "V_out"):
        x, y = getattr(a, f), getattr(c, f)
        assert torch.equal(x, y) and torch.equal(x, x[:2].repeat((heads // 2,) + (1,) * (x.dim() - 1))), f


def test_rows_apart_in_memory():
    """Token strides: a little more than a row, and so much that a head spans 2 GiB (offsets of 64 bits)."""
    n, b = 4100, 130
    K, V, s = _inputs(1, n, "tight", 5)
    ref = B.kvr_select_greedy(V.contiguous(), s, b, .5)
    _, V8, _ = _inputs(1, n, "tight", 5, pad=8)
    far = torch.empty((n * 262144,), dtype=torch.bfloat16, device=DEV).view(1, n, 262144)[:, :, :128]
    far.copy_(V)
    for rows in (V8, far):
        got = B.kvr_select_greedy(rows, s, b, .5)
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(ref, got))
