"""Which heads retain_sparse_kernel finishes by itself: its search for s_(b) and for the cut must know the leading 16 key bits of both
wherever the scores lie (positive, of both signs, with zeros, with an outlier far above the rest), or heads that it could finish go to the
kernel for long heads.  The same decisions from sorted scores on the CPU; a head that is cut is finished when the best score left out stays
below the last gain of the oracle's run on what is kept."""
import ctypes
import dataclasses

import numpy as np
import pytest
import torch

import parity_util as P
from oracle import alpha_oracle as O
from paper_2605_14292_amd import binding as B
from paper_2605_14292_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LAM, EPS = 0.5, 1e-6
LAUNCH = "_ZN3kvr20launch_retain_sparseEPKvS1_PKfRKNS_6LayoutEiffPiS7_PfPvS9_P12ihipStream_tPKi"   # kvr::launch_retain_sparse


def _key16(s):
    u = np.asarray(s, dtype=np.float32).view(np.uint32)
    return (np.where(u >> 31, ~u, u | np.uint32(0x80000000)) >> np.uint32(16)).astype(np.int64)


def _score_of(key16):
    k = np.uint32(key16 << 16)
    return np.array([k & np.uint32(0x7fffffff) if k >> 31 else ~k], dtype=np.uint32).view(np.float32)[0]


def decide(s, b, cap):
    """'fits', 'handed on', or 'cut' with the tokens kept and the best score left out."""
    s = np.asarray(s, dtype=np.float32)
    if not s.max() - s.min() > LAM:
        return "handed on", None, None
    key = _key16(s + np.float32(0))
    down = np.sort(key)[::-1]
    sb = _score_of(int(down[b - 1]))
    if (s >= sb - np.float32(LAM * 1.00001) - np.float32(1e-5) * abs(sb)).sum() <= cap:
        return "fits", None, None
    kept = key > down[cap]
    left = s[~kept].max()
    if kept.sum() < b or not left < sb - 0.25 * LAM:
        return "handed on", None, None
    return "cut", np.flatnonzero(kept), left


def finishes(s, V, b, cap):
    what, kept, left = decide(s, b, cap)
    if what != "cut":
        return what, what == "fits"
    last = O.alpha_select(s.astype(np.float64)[kept], V[kept], b, LAM, EPS)["gain"][-1]
    margin = 1e-5 * (abs(last) + LAM)
    assert abs(left - (last - margin)) > margin / 2          # (the case is not a borderline one)
    return what, bool(left < last - margin)


def _scores(n, b, g):
    z = torch.randn((10, n), generator=g)
    s = z.exp()                                       # 0: log-normal
    s[1] = z[1]                                       # of both signs
    s[2] = z[2].clamp_min(0)                          # half of them zero
    s[3, n // 3] = 0.                                 # log-normal and one zero
    s[4] = 4 * z[4]
    s[5] = z[5]; s[5, n // 2] = 1e9                   # an outlier
    s[6] = (3 * z[6]).exp()                           # b-th and best more than eight binades apart, or not
    s[7] = -s[7]
    s[8] = 4 * z[8]; s[8, 5:5 + b // 2] = 1e5         # s_(b) more than eight binades below the best
    s[9] = 0.9 * z[9]                                 # (its value rows are alike: every gain falls by lambda)
    return s


def _run_alone(K, V, s, b):
    out = B.RetainBuffers(K.shape[0], K.shape[1], b, 128, torch.bfloat16, DEV, computed_scores=False)
    launch = getattr(B.lib(), LAUNCH)
    launch.restype = ctypes.c_int
    p = [ctypes.c_void_p(t.data_ptr()) for t in (K, V, s, out.idx_sorted, out.pick_order, out.pick_gain, out.K_out, out.V_out)]
    lay = B.layout_of(K)
    rc = launch(p[0], p[1], p[2], ctypes.byref(lay), ctypes.c_int(b), ctypes.c_float(LAM), ctypes.c_float(EPS), *p[3:],
                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), None)
    assert rc == 0
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("n,b", [(257, 40), (257, 128), (600, 128), (1024, 64), (1024, 128), (1025, 16), (2048, 128), (2049, 64), (3001, 128),
                                 (3073, 33), (4096, 64), (4096, 128)])
def test_heads_finished(n, b):
    cap = 128 if b <= 64 else 192
    g = torch.Generator().manual_seed(31 * n + b)
    s = _scores(n, b, g)
    V = torch.randn((10, n, 128), generator=g)
    V[:, n // 2:n // 2 + n // 4] = V[:, :n // 4] + 0.05 * V[:, n // 2:n // 2 + n // 4]
    V[9] = V[9, :1] + 0.01 * V[9]
    V = V.to(torch.bfloat16)
    want = [finishes(s[h].numpy(), W.to_f64(V[h]), b, cap) for h in range(10)]
    K = torch.randn((10, n, 128), generator=g).to(torch.bfloat16).to(DEV)
    Vd, sd = V.to(DEV), s.to(DEV)
    out = _run_alone(K, Vd, sd, b)
    done = (out.idx_sorted[:, 0] != -1).tolist()
    assert done == [f for _, f in want], want
    if n >= 1024 and b >= 64:                         # both ways out of a cut are among them, and what was lost with bins of half a binade
        assert {w for w, _ in want} == {"fits", "cut", "handed on"} and want[1] == ("cut", True) and want[9] == ("cut", False)
    whole = B.kvr_retain(K, Vd, b, LAM, EPS, s=sd)
    torch.cuda.synchronize()
    for h in range(10):
        P.check_head(W.to_f64(s[h]), W.to_f64(V[h]), b, LAM, EPS, whole.pick_order[h].cpu().numpy(), whole.pick_gain[h].cpu().numpy(),
                     whole.idx_sorted[h].cpu().numpy())
        if done[h]:
            assert torch.equal(out.pick_order[h], whole.pick_order[h]) and torch.equal(out.V_out[h], whole.V_out[h])


@pytest.mark.parametrize("b", [64, 128])
def test_heads_of_one_workgroup(b):
    """More heads than workgroups: kinds that need one histogram, three or five, and heads handed on, one after the other."""
    heads, n, cap = 1300, 600, 128 if b <= 64 else 192
    g = torch.Generator().manual_seed(b)
    s = torch.cat([_scores(n, b, g) for _ in range(heads // 10)])
    V = torch.randn((heads, n, 128), generator=g).to(torch.bfloat16)
    K = torch.randn((heads, n, 128), generator=g).to(torch.bfloat16).to(DEV)
    out = _run_alone(K, V.to(DEV), s.to(DEV), b)
    done = (out.idx_sorted[:, 0] != -1).tolist()
    assert done == [finishes(s[h].numpy(), W.to_f64(V[h]), b, cap)[1] for h in range(heads)]
    alone = [_run_alone(K[h:h + 1], V[h:h + 1].to(DEV), s[h:h + 1].to(DEV), b) for h in range(heads - 20, heads)]
    for h, one in zip(range(heads - 20, heads), alone):
        assert torch.equal(out.idx_sorted[h], one.idx_sorted[0]) and (not done[h] or torch.equal(out.pick_order[h], one.pick_order[0]))


def test_a_full_size_event_with_scores_of_both_signs():
    """7168 heads of 1024 tokens, b = 128, all of them cut: whether sampled heads are finished, their picks one by one, kept rows of all."""
    w = dataclasses.replace(W.WORKLOADS["c5"], scores="given", G=1)
    data = W.generate(w, seed=11, device=DEV)
    K, V, s = data["K"], data["V"], data["s"].log()              # (the generator's scores are log-normal)
    alone = _run_alone(K, V, s, 128)
    done = (alone.idx_sorted[:, 0] != -1)
    out = B.kvr_retain(K, V, 128, LAM, EPS, s=s)
    torch.cuda.synchronize()
    assert torch.equal(out.pick_order[done], alone.pick_order[done])
    rows = out.idx_sorted.long().unsqueeze(-1).expand(-1, -1, 128)
    assert torch.equal(out.V_out, torch.gather(V, 1, rows)) and torch.equal(out.K_out, torch.gather(K, 1, rows))
    for h in range(0, w.heads, 241):
        assert finishes(s[h].cpu().numpy(), W.to_f64(V[h]), 128, 192) == ("cut", bool(done[h]))
        P.check_head(W.to_f64(s[h]), W.to_f64(V[h]), 128, LAM, EPS, out.pick_order[h].cpu().numpy(), out.pick_gain[h].cpu().numpy(),
                     out.idx_sorted[h].cpu().numpy())
