"""Measured cases of the route-step library: what a serving loop or a replay has it do, once per pass.

A pass is one call of a loop that keeps going: the requests that arrived since the last call join the waiting queues,
one scheduling round binds requests to workers, and the decode steps up to the next call run.  The cluster state lives
on from pass to pass, so what is measured is the regime the loop settles into.  Arrivals come from a short trace that
is walked in a circle; active sets are drawn as such a loop would hold them (a request is found active with a
probability proportional to its output length, somewhere along it), so the first pass is already typical.

Keys of a case:
  kind      "round": br_route_step / br_route_advance; "bypass": every arrival placed at once (br_route_bypass)
  call      "fused": round and decode steps in one call; "two": two calls; "host": the call of the README's loop,
            arrays in host memory in and out
  n_inst, G, B, max_wait, H, pred_mode, R_max, S_greedy, gate, watermark, gamma: as in RouteConfig
  outputs   "assign": decisions and counters; "scores": with the snapshot reductions; "matrix": with every score
  n_steps   decode steps between two rounds
  rate      mean arrivals per cluster and pass; rate_hi: the other mean of a bursty source (0: plain Poisson)
  fill      share of the slots that is taken when the measurement starts
  prompt_mu, prompt_sigma, prompt_hi, out_mu, out_sigma, out_hi: length mixes (log-normal, clipped)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2605_06113_amd import binding, workloads as wl

DEVICE = "cuda:0"
TABLE = 1 << 16  # lengths and prediction rows are drawn once and then picked from
SHORT = dict(prompt_mu=math.log(1000.0), prompt_sigma=1.0, prompt_hi=16384, out_mu=math.log(200.0), out_sigma=1.2, out_hi=4096)
LONG = dict(prompt_mu=math.log(2000.0), prompt_sigma=1.1, prompt_hi=32768, out_mu=math.log(300.0), out_sigma=1.3, out_hi=8192)


def _case(name, **kw):
    c = dict(kind="round", call="fused", n_inst=1, G=16, B=96, max_wait=256, H=0, pred_mode=0, R_max=4, S_greedy=-1,
             gate=0.5, watermark=0, gamma=0.9, outputs="assign", n_steps=1, rate=1.0, rate_hi=0.0, fill=1.0, **SHORT)
    c.update(kw)
    return dict(c, name=name) if name else c


def _mean_out(case):
    """Mean output length of the mix (log-normal, clipped above)."""
    mu, sd, hi = case["out_mu"], case["out_sigma"], math.log(case["out_hi"])
    cdf = lambda x: 0.5 * (1.0 + math.erf(x / math.sqrt(2.0)))
    return math.exp(mu + sd * sd / 2) * cdf((hi - mu - sd * sd) / sd) + case["out_hi"] * (1.0 - cdf((hi - mu) / sd))


def listed():
    return [
        # the smallest call: one small cluster under a token watermark, one decode step at a time
        _case("one_small_cluster", G=4, B=16, max_wait=32, watermark=58982, prompt_hi=8192, rate=0.3),
        # the README's loop on one cluster: host arrays in, every output back on the host
        _case("one_cluster_host_loop", call="host", outputs="matrix", watermark=235929, rate=40.0),
        # one large cluster with lookahead, a long queue and bursty arrivals (the stress configuration)
        _case("one_large_cluster", call="two", G=64, max_wait=2048, H=8, watermark=471859, outputs="scores", rate=60.0,
              rate_hi=300.0, **LONG),
        # the paper's deployment: one cluster, H = 80, the estimate maintained by the library
        _case("one_cluster_long_horizon", call="two", G=8, B=64, H=80, pred_mode=2, outputs="scores", rate=0.7, rate_hi=2.0,
              fill=0.95, **LONG),
        # many replays of an overloaded cluster side by side, a decode step per call
        _case("replay_1024", n_inst=1024, watermark=235929, rate=40.0),
        # the throughput batch in an overloaded steady state: full queues, a few slots free per step
        _case("batch_4096_step", n_inst=4096, B=144, outputs="scores", rate=7.0),
        # the throughput batch with rounds at intervals: 256 arrivals find 256 free slots
        _case("batch_4096_burst", n_inst=4096, B=144, outputs="scores", n_steps=48, rate=250.0, fill=0.89),
        # every score of the snapshot asked for, on odd sizes
        _case("batch_matrix_ragged", call="two", n_inst=1531, G=13, B=101, max_wait=307, outputs="matrix", n_steps=3, rate=17.0),
        # lookahead from termination hazards, rounds at intervals
        _case("batch_4096_lookahead", n_inst=4096, G=32, max_wait=512, H=4, outputs="scores", n_steps=40, rate=250.0, fill=0.79),
        # many clusters at the deployed horizon, overloaded
        _case("batch_2048_long_horizon", n_inst=2048, G=8, B=64, H=80, pred_mode=2, outputs="scores", rate=1.6),
        # Stage 2 over a wide window
        _case("batch_1024_wide_window", n_inst=1024, B=144, R_max=16, S_greedy=64, n_steps=8, rate=60.0),
        # arrivals dispatched at once, past the pool
        _case("bypass_4096", kind="bypass", n_inst=4096, B=144, n_steps=12, rate=60.0, fill=0.85),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    """One more case: any of the kinds of work above, at sizes anywhere between the smallest and the largest."""
    family = rng.choice(("plain", "plain", "plain", "short", "short", "long", "wide", "bypass"))
    mix = rng.choice((SHORT, LONG))
    G = _log_int(rng, 2, 64)
    B = rng.randint(12, 160)
    Q = _log_int(rng, 24, 2048)
    n_max = 4096
    kw = dict(G=G, B=B, max_wait=Q, **mix)
    if family == "short":
        kw.update(H=rng.randint(1, 8), pred_mode=rng.choice((0, 0, 1, 3)), gate=rng.choice((0.0, 0.5)), gamma=rng.choice((0.64, 0.9)))
    elif family == "long":
        kw.update(H=rng.randint(9, 128), pred_mode=rng.choice((1, 2, 2, 3)), gamma=rng.choice((0.86, 0.9)), G=_log_int(rng, 2, 32))
        n_max = 2048
    elif family == "wide":
        R = rng.choice((12, 16, 24))
        kw.update(R_max=R, S_greedy=rng.randint(16, 64))
        n_max = 512 if R <= 16 else 64
    elif family == "bypass":
        kw.update(kind="bypass")
    # no more active requests and no more queue entries in the batch than the largest listed case has
    slots = kw["G"] * B * (2 if kw.get("H", 0) > 0 else 1)
    n_max = max(1, min(n_max, 4096 * 2304 // slots, 4096 * 256 // Q))
    kw["n_inst"] = _log_int(rng, 1, n_max)
    if family != "bypass":
        kw["outputs"] = rng.choice(("assign", "scores", "scores", "matrix"))
        kw["call"] = rng.choice(("fused", "fused", "two", "host" if kw["n_inst"] <= 8 else "fused"))
    kw["n_steps"] = 1 if kw.get("pred_mode") == 2 else _log_int(rng, 1, 48)
    if rng.random() < 0.25:
        kw["watermark"] = int(B * 2600 * rng.uniform(0.8, 1.2))
    c = _case(None, **kw)
    load = rng.uniform(0.6, 1.5)  # offered load over what the workers can serve
    c["rate"] = round(min(load * c["G"] * B * c["n_steps"] / _mean_out(c), 1.5 * Q), 3)
    c["fill"] = round(min(load, 1.0), 3)
    return c


def _config(case, seed):
    return wl.RouteConfig(name="measured", n_inst=case["n_inst"], G=case["G"], B=case["B"], max_wait=case["max_wait"],
                          H=case["H"], R_max=case["R_max"], S_greedy=case["S_greedy"], token_watermark=case["watermark"],
                          gamma=case["gamma"], gate_pfin=case["gate"], pred_mode=case["pred_mode"], seed=seed % (1 << 31),
                          prompt_mu=case["prompt_mu"], prompt_sigma=case["prompt_sigma"], prompt_hi=case["prompt_hi"],
                          out_mu=case["out_mu"], out_sigma=case["out_sigma"], out_hi=case["out_hi"])


def _arrival_cap(case):
    """Row length of the arrival buffers: six deviations above the mean, at most what a pool-bypass call takes."""
    top = max(case["rate"], case["rate_hi"])
    return min(2048, int(top + 6.0 * math.sqrt(top)) + 8)


def prepare(case, seed):
    cfg = _config(case, seed)
    rng = np.random.Generator(np.random.PCG64([seed, 11]))
    N, G, B = cfg.n_inst, cfg.G, cfg.B
    s_tab, o_tab = wl.prompts(rng, cfg, TABLE), wl.outputs(rng, cfg, TABLE)
    pick = lambda tab, shape: tab[rng.integers(0, len(tab), size=shape, dtype=np.int32)]
    Pq, P = wl.pred_width(cfg), wl.slot_pred_width(cfg)
    rows = wl.hazards(rng, cfg, TABLE).reshape(TABLE, Pq) if Pq else None

    # active sets: length-biased outputs, a uniform age along each
    n = rng.binomial(B, case["fill"], size=(N, G)).astype(np.int32)
    heavy = o_tab[np.searchsorted(np.cumsum(o_tab, dtype=np.int64), rng.integers(0, int(o_tab.sum(dtype=np.int64)), size=TABLE), side="right")]
    o = pick(heavy, (N, G, B))
    rem = (rng.random((N, G, B), dtype=np.float32) * o).astype(np.int32) + 1
    rem = np.minimum(rem, o)
    age = o - rem
    kv = pick(s_tab, (N, G, B)) + age
    pred = None
    if P and cfg.pred_mode == 2:
        pred = wl.maintained_triples(rng, cfg, TABLE)[rng.integers(0, TABLE, size=(N, G, B), dtype=np.int32)]
        pred[..., 1] = age
    elif P:
        pred = pick(rows, (N, G, B))
    hist = wl.output_history(cfg, 8000) if cfg.pred_mode == 2 and cfg.H > 0 else None
    router = binding.Router(cfg, wl.InitState(n, kv, rem, pred), device=DEVICE, hist=hist)

    # arrivals: a short trace, walked in a circle
    steps = 64 if N <= 64 else 16 if N <= 1024 else 6
    mean = np.full((steps, 1), case["rate"])
    if case["rate_hi"] > 0:
        mean[rng.random(steps) < 0.5] = case["rate_hi"]
    cap = _arrival_cap(case)
    count = np.minimum(rng.poisson(mean, size=(steps, N)), cap).astype(np.int32)
    trace = []
    for k in range(steps):
        ids = np.broadcast_to(np.arange(k * cap, (k + 1) * cap, dtype=np.int32), (N, cap))
        arr = wl.Arrivals(count[k], pick(s_tab, (N, cap)), pick(o_tab, (N, cap)), ids, pick(rows, (N, cap)) if Pq else None)
        trace.append(arr if case["call"] == "host" else binding.DeviceArrivals(arr, DEVICE, Pq))
    at = lambda off, size: router.ws[off // 4: off // 4 + size]
    lay = router.layout
    # what the call leaves in the state, beside its outputs: loads and list lengths of the workers, queue lengths
    held = dict(L=at(lay.L, N * G), n=at(lay.n, N * G), qlen=at(lay.qlen, N))
    if case["kind"] == "bypass":
        out = dict(assign=torch.full((N, cap), -3, dtype=torch.int32, device=DEVICE),
                   stats=torch.zeros((N, binding.NSTATS), dtype=torch.int64, device=DEVICE))
    else:
        out = router.alloc_outputs(scores=case["outputs"] != "assign", matrix=case["outputs"] == "matrix")
    return dict(case=case, router=router, trace=trace, held=held, out=out, k=0)


def run(state):
    case, router = state["case"], state["router"]
    arrivals = state["trace"][state["k"]]
    state["k"] = (state["k"] + 1) % len(state["trace"])
    out = state["out"]
    if case["kind"] == "bypass":
        router.route_bypass_device(arrivals, out)
        router.advance(case["n_steps"])
    elif case["call"] == "host":
        out = router.route_step(arrivals, scores=case["outputs"] != "assign", matrix=case["outputs"] == "matrix",
                                advance=case["n_steps"])
    elif case["call"] == "two":
        router.route_step_device(arrivals, out)
        router.advance(case["n_steps"])
    else:
        router.route_advance_device(arrivals, out, case["n_steps"])
    return dict(out, **state["held"])


def work(case):
    """Expected work of a pass in the steady state: lists read and written once, the queue and the arrivals read once,
    outputs and what moves written once; operations of the scores that the method asks for."""
    N, G, B, Q, H = (case[k] for k in ("n_inst", "G", "B", "max_wait", "H"))
    cfg = _config(case, 0)
    P, Pq = wl.slot_pred_width(cfg), wl.pred_width(cfg)
    served = case["n_steps"] * G * B / _mean_out(case)          # slots that fall free per pass
    rate = 0.5 * (case["rate"] + case["rate_hi"]) if case["rate_hi"] > 0 else case["rate"]
    overload = rate > served
    active = G * B * (1.0 if overload else case["fill"])
    admitted = min(rate, served)
    waiting = min(rate, Q) if case["kind"] == "bypass" or not overload else Q
    joined = min(rate, Q) if not overload else min(rate, admitted)
    per = 16 * active + 16 * G                                   # kv and remaining steps, loads and lengths: in and out
    if H > 0:
        per += active * 4 * P * (2 if case["pred_mode"] == 2 else 1)
    per += 4 * waiting + (12 + 4 * Pq) * (rate + joined - admitted) + (8 + 4 * P) * admitted + 128
    if case["kind"] == "bypass":
        per += 4 * rate
    else:
        per += 8 * Q
        if case["outputs"] != "assign":
            per += 4 * Q + 4 * G
        if case["outputs"] == "matrix":
            per += 4 * waiting * G
    score = 4 if H == 0 else 3 * (H + 1) + 3
    if case["kind"] == "bypass":
        ops = rate * G * score
    else:
        ops = admitted * waiting * score + (waiting * G * score if case["outputs"] != "assign" else 0)
    return {"bytes": N * per, "flops": N * (ops + 4 * active)}


def tolerance(case):
    """Decisions, loads and integer scores are exact; lookahead scores are fp32 sums of up to H + 1 terms."""
    return {"rel": 1e-5} if case["H"] > 0 and case["outputs"] == "matrix" else "exact"
