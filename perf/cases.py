"""What a user of this library has it do, as cases that can be timed and compared: compression events of the
shapes of the benchmark configurations (`paper_2605_14292_amd.workloads`), of the sizes between them, and the three
frames around an event (observation-window scores, flat signature, budget allocator).

    listed()            the cases by name
    draw(rng)           one more case of the same ranges
    prepare(case, seed) the inputs and the output buffers a serving loop holds before the call
    run(state)          one event through the public entry points, and everything it returns
    work(case)          bytes and operations of one event that no implementation avoids
    tolerance(case)     how far another correct implementation of the same precision may be off
"""
import dataclasses
import math

import torch

from paper_2605_14292_amd import binding as B
from paper_2605_14292_amd import workloads as W

D = 128                     # head dimension of every configuration
EPS = 1e-6
DEV = "cuda:0"


def _case(name, frame, layers, kv_heads, seqs, n, b, *, dtype="bf16", lam=0.5, rows, scores="queries", G=1, kernel=0):
    """frame: "event" (kvr_retain), "window" (kvr_score, kvr_score_pool, kvr_retain), "flat" (kvr_retain_flat) or
    "budgeted" (kvr_retain_budgeted).  scores: "queries" (computed from G queries per head) or "given"."""
    case = dict(frame=frame, layers=layers, kv_heads=kv_heads, seqs=seqs, n=n, b=b, dtype=dtype, lam=lam, rows=rows,
                scores=scores, G=G, kernel=kernel)
    return dict(case, name=name) if name else case


def listed():
    return [
        # The smallest call there is: one fp32 head with its one query (configuration c1).  Launches and latency.
        _case("one head fp32", "event", 1, 1, 1, 192, 64, dtype="f32", rows="clustered", G=1),
        # A decode-time event of one sequence, batch 1 (c2): what a serving loop calls once per compression.
        _case("decode event", "event", 28, 4, 1, 256, 128, rows="dup_normal", G=7),
        # The same of a batch of 32 sequences whose scorer is external and hands its scores in (c3).
        _case("batched event", "event", 32, 8, 32, 192, 64, rows="clustered", scores="given"),
        # A batch whose scores come from the queries, with sizes that are no multiple of anything.
        _case("batched event queries", "event", 28, 4, 24, 251, 101, rows="mixed", G=7),
        # The lambda sweep's main point (c5): medium heads, a large batch.
        _case("medium heads", "event", 28, 4, 64, 1024, 128, rows="mixed", G=7),
        # The sweep's lambda = 0 end, at its smaller budget: plain top-b, the baseline every user compares with.
        _case("medium heads top-b", "event", 28, 4, 64, 1024, 64, lam=0.0, rows="mixed", G=7),
        # One-shot compression after a long prefill (c4), the largest configuration.
        _case("long prefill", "event", 32, 8, 8, 4096, 128, rows="dup_student_t", G=4),
        # A long prefill whose scorer hands its scores in, of an ordinary, ragged length.
        _case("long prefill given", "event", 32, 8, 4, 3001, 128, rows="dup_student_t", scores="given"),
        # One long sequence scored by an observation window (32 positions x 7 grouped heads) and smoothed along the
        # tokens, as the scorers the method builds on do it.
        _case("window one sequence", "window", 28, 4, 1, 4000, 128, rows="dup_normal", G=224, kernel=7),
        # One sequence at the largest context and a budget of an eighth of it.
        _case("large budget", "event", 32, 8, 1, 8192, 1024, rows="dup_normal", G=4),
        # Flat-signature mode on c5's shape: one selection per sequence, shared by its 112 heads.
        _case("flat signature", "flat", 28, 4, 64, 1024, 128, rows="mixed", scores="given"),
        # The event inside a budget allocator: ragged candidate counts, per-head budgets, protected sinks and a
        # recent window, position ids.
        _case("budget allocator", "budgeted", 28, 4, 16, 1000, 128, rows="mixed", G=7),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    rows = rng.choice(["clustered", "dup_normal", "dup_student_t", "mixed"])
    geometry = [(28, 4, 7), (32, 8, 4)]                     # layers, kv heads, grouped queries of the configurations
    layers, kv, G = rng.choice(geometry)
    lam = rng.choice([0.25, 0.5, 0.5, 1.0])
    kind = rng.choice(["tiny", "decode", "batched", "long", "long", "top-b", "large", "window", "flat", "budgeted"])
    if kind == "tiny":
        n = _log_int(rng, 48, 256)
        return _case("", "event", 1, _log_int(rng, 1, 32), 1, n, _log_int(rng, 16, n // 2), dtype="f32", lam=lam,
                     rows=rows, G=rng.randint(1, 7))
    if kind == "decode":
        n = rng.randint(129, 256)
        given = rng.random() < 0.5
        return _case("", "event", layers, kv, 1, n, rng.randint(32, min(n - 1, 128)), lam=lam, rows=rows,
                     scores="given" if given else "queries", G=1 if given else G)
    if kind == "batched":
        n = rng.randint(97, 256)
        given = rng.random() < 0.5
        return _case("", "event", layers, kv, rng.randint(4, 24), n, rng.randint(24, min(n // 2, 128)), lam=lam,
                     rows=rows, scores="given" if given else "queries", G=1 if given else G)
    if kind in ("long", "top-b"):
        n = _log_int(rng, 257, 4096)
        seqs = _log_int(rng, 1, max(1, min(64, 8 * 2**20 // (n * layers * kv))))
        given = kind == "long" and rng.random() < 0.4
        return _case("", "event", layers, kv, seqs, n, rng.choice([64, 128, rng.randint(17, 128)]),
                     lam=0.0 if kind == "top-b" else lam, rows=rows, scores="given" if given else "queries",
                     G=1 if given else G)
    if kind == "large":
        n = rng.randint(1500, 8192)
        return _case("", "event", layers, kv, 1, n, _log_int(rng, 129, min(1024, n // 4)), lam=lam, rows=rows, G=G)
    if kind == "window":
        n = _log_int(rng, 600, 4096)
        return _case("", "window", layers, kv, 1, n, rng.randint(48, 128), lam=lam, rows=rows,
                     G=G * rng.choice([8, 16, 32]), kernel=rng.choice([5, 7, 13]))
    if kind == "flat":
        n = _log_int(rng, 192, 1024)
        return _case("", "flat", layers, kv, _log_int(rng, 2, 7 * 2**20 // (n * layers * kv)), n, rng.randint(48, 128), lam=lam,
                     rows=rows, scores="given")
    n = _log_int(rng, 180, 2000)
    return _case("", "budgeted", layers, kv, _log_int(rng, 1, max(1, 7 * 2**18 // (n * layers * kv))), n,
                 rng.randint(64, 128), lam=lam, rows=rows, G=G)


def _workload(case):
    kinds = {"clustered": dict(centres=32 if case["dtype"] == "bf16" else 16, sigma=0.1),
             "dup_normal": dict(dup_frac=0.25, dup_sigma=0.05), "dup_student_t": dict(dup_frac=0.2, dup_sigma=0.05),
             "mixed": dict(centres=32, sigma=0.1)}
    return W.Workload("%s-%d-%d" % (case["frame"], case["n"], case["seqs"]), case["layers"], case["kv_heads"], case["seqs"],
                      case["n"], case["b"], D, case["dtype"], case["lam"], case["rows"],
                      scores="computed" if case["scores"] == "queries" else "given", G=case["G"], **kinds[case["rows"]])


@dataclasses.dataclass
class State:
    case: dict
    data: dict
    out: object
    extra: dict


def prepare(case, seed):
    w = _workload(case)
    heads, n, b, lam = w.heads, w.n, w.b, w.lam
    data = W.generate(w, seed=seed, device=DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + n)
    extra = {}
    frame = case["frame"]
    if frame == "flat":
        # one score per token and sequence: the mean over the sequence's heads of softmaxes of normal logits
        group = case["layers"] * case["kv_heads"]
        acc = torch.zeros((case["seqs"], n), device=DEV)
        for _ in range(16):
            acc += torch.softmax(torch.randn((case["seqs"], group // 16, n), generator=g, device=DEV), dim=2).sum(1)
        data["s"] = acc / (16 * (group // 16))
        extra["group"] = group
        out = B.FlatBuffers(heads, group, n, b, D, w.torch_dtype, DEV)
    elif frame == "budgeted":
        n_h = torch.randint(max(b, n // 2), n + 1, (heads,), generator=g, device=DEV, dtype=torch.int32)
        j = torch.arange(n, device=DEV)
        keep = (j[None, :] < 4) | ((j[None, :] >= n_h[:, None] - 16) & (j[None, :] < n_h[:, None]))
        extra.update(n_h=n_h, keep=keep.to(torch.uint8).contiguous(),
                     b_h=torch.randint(b // 2, b + 1, (heads,), generator=g, device=DEV, dtype=torch.int32),
                     pos=(j.to(torch.int32)[None, :] * 2 + 5).expand(heads, n).contiguous())
        out = B.BudgetBuffers(heads, n, b, D, w.torch_dtype, DEV, with_pos=True)
    else:
        if frame == "window":
            extra.update(s_raw=torch.empty((heads, n), device=DEV), s=torch.empty((heads, n), device=DEV))
        out = B.RetainBuffers(heads, n, b, D, w.torch_dtype, DEV,
                              computed_scores=frame == "event" and case["scores"] == "queries")
    return State(case, data, out, extra)


def run(state):
    case, data, out, extra = state.case, state.data, state.out, state.extra
    K, V, b, lam = data["K"], data["V"], case["b"], case["lam"]
    if case["frame"] == "flat":
        B.kvr_retain_flat(K, V, data["s"], extra["group"], b, lam, EPS, out=out)
        scores = {"signature": out.u_out}
    elif case["frame"] == "budgeted":
        B.kvr_retain_budgeted(K, V, b, lam, EPS, Q=data.get("Q"), s=data.get("s"), n_h=extra["n_h"], b_h=extra["b_h"],
                              keep=extra["keep"], pos=extra["pos"], out=out)
        scores = {"s": out.s_work, "pos": out.pos_out}
    elif case["frame"] == "window":
        B.kvr_score(K, data["Q"], s_out=extra["s_raw"])
        B.kvr_score_pool(extra["s_raw"], case["kernel"], B.KVR_POOL_MAX, s_out=extra["s"])
        B.kvr_retain(K, V, b, lam, EPS, s=extra["s"], out=out)
        scores = {"s_raw": extra["s_raw"], "s": extra["s"]}
    else:
        B.kvr_retain(K, V, b, lam, EPS, Q=data.get("Q"), s=data.get("s"), out=out)
        scores = {"s": out.s_out}
    return {"kept": out.idx_sorted, "order": out.pick_order, "gain": out.pick_gain, "K": out.K_out, "V": out.V_out, **scores}


def work(case):
    """Each input row read once (of V only the kept rows when lambda is 0, of K only the kept ones when nothing is
    scored from it), each output written once; the products of the queries with K and of the picks with V."""
    e = 2 if case["dtype"] == "bf16" else 4
    n, b, G, seqs = case["n"], case["b"], case["G"], case["seqs"]
    heads = case["layers"] * case["kv_heads"] * seqs
    row = D * e
    queries = case["scores"] == "queries"
    if case["frame"] == "budgeted":                          # candidates n/2 .. n, budgets b/2 .. b, uniformly
        n, b = int(0.75 * n), int(0.75 * b)
    kept = 2 * b * row * heads + 3 * 4 * b * heads            # rows; index, pick and gain
    if case["frame"] == "flat":
        u = seqs * n * D * 4
        return {"bytes": heads * (n + b) * row + 4 * n * seqs + u + 2 * b * row * heads + 3 * 4 * b * seqs,
                "flops": heads * n * D + 2 * b * n * D * seqs}
    v = (n if case["lam"] else b) * row * heads
    k = (n if queries else b) * row * heads
    s = 4 * n * heads                                        # scores: written when computed, read when given
    if queries:
        s += G * row * heads
    flops = (2 * b * n * D if case["lam"] else 0) * heads + (2 * G * n * D * heads if queries else 0)
    if case["frame"] == "window":
        s += 4 * n * heads                                   # raw and smoothed scores are both returned
    if case["frame"] == "budgeted":
        s += (case["n"] + 4 * b) * heads + 8 * heads         # protection flags, position ids, counts
    return {"bytes": v + k + s + kept, "flops": flops}


def tolerance(case):
    """Measured by running each case with the 128 coordinates of every row permuted (the same sums in another order) and
    stated at about four times that: scores and gains move by at most 2.9e-7 (2-norm) and 1.5e-6 (one value).  Two
    tokens whose gains agree to the last bits may swap places in the order of the picks (at most 2.4e-5 of the entries).
    A tie across the budget's edge changes a kept row: top-b moved by 8.8e-3 in the kept rows, and with a budget above
    128 one of 256 heads went another way (8.8e-2 and 4e-3 of the entries)."""
    if case["lam"] == 0.0 or case["b"] > 128:
        return {"rel": 3e-2, "max": 0.99, "differ": 1e-2}
    return {"rel": 1.2e-6, "max": 6e-6, "differ": 1e-4}
