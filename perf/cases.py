"""Timed cases of the shot pipeline: what programs built on this library spend their GPU time on.

Every case goes through the public binding (paper_2504_05611_amd.tmcs and, for training,
paper_2504_05611_amd.neural_bp).  Circuits come from workloads/: the surface-code memory,
non-local CNOT and Pauli-string circuits, and the bivariate-bicycle memory and teleportation.

Kinds of case (`kind`):
  step        one step of a Monte-Carlo run: sample_async -> decode -> count_errors, nothing waits
  sample      the sampler alone, for programs that store syndromes
  posteriors  BP without OSD with every per-shot output (hard decision, LLRs, iterations, flags)
  learned     BP-OSD with per-edge, per-iteration weights on given syndromes
  osd_cs      BP with the order-7 combination sweep on given syndromes
  train       one training step of the weights: forward, loss on the last iteration, backward
  plan        one replay of a captured plan over several circuits, and its counters
"""
from __future__ import annotations

import functools
import math
import os

import numpy as np
import torch

from paper_2504_05611_amd import neural_bp, tmcs
from workloads import BB_PARAMS, bb, pstring, sc, with_decoherence

SHOTS_PER_BLOCK = 4096


def listed():
    return [
        # a quick check of a small circuit: a dozen launches, bound by latency
        dict(name="sc3_memory_step", kind="step", code="sc", d=3, op="memory", rb=3, ra=0, p=1e-3, pe=1e-3, T=30,
             shots=10000),
        # the d = 5 non-local CNOT at the shot count of an error-rate point
        dict(name="sc5_nlcnot_step", kind="step", code="sc", d=5, op="nlcnot", rb=5, ra=5, p=1e-3, pe=1e-2, T=30,
             shots=1000000),
        # weight-6 Pauli string on d = 5 blocks: seven observables, a ragged shot count
        dict(name="sc5_pstring6_step", kind="step", code="sc", d=5, op="pstring", w=6, rb=4, ra=1, p=1e-3, pe=1e-3,
             T=30, shots=100003),
        # a bicycle-code memory point; checks of 35 mechanisms, one in twenty shots needs OSD
        dict(name="bb144_memory_step", kind="step", code="bb144", op="memory", rb=12, ra=0, p=1e-3, pe=1e-3, T=30,
             shots=65536),
        # the same with the ebit layer: checks of up to 161 mechanisms, a third of the shots need OSD
        dict(name="bb144_teleport_step", kind="step", code="bb144", op="teleport", rb=4, ra=3, p=1e-3, pe=1e-2, T=20,
             shots=32768),
        # decoding stored syndromes with the learned weights shipped with the package
        dict(name="bb144_teleport_learned", kind="learned", code="bb144", op="teleport", rb=4, ra=3, p=1e-3, pe=1e-2,
             T=20, shots=8192),
        # a batch of mid-size non-local CNOTs as one captured graph (two sizes, two noise strengths)
        dict(name="sc11_sc15_plan", kind="plan", code="sc", d=11, d2=15, op="nlcnot", p=1e-4, p2=1e-3, T=20,
             shots=4096),
        # a large block: BP state beyond one compute unit's LDS, windowed OSD on most shots
        dict(name="sc21_nlcnot_step", kind="step", code="sc", d=21, op="nlcnot", rb=21, ra=21, p=1e-3, pe=1e-2, T=20,
             shots=4096),
        # decoder studies: the posteriors of every shot, an odd shot count
        dict(name="sc11_posteriors", kind="posteriors", code="sc", d=11, op="nlcnot", rb=11, ra=11, p=1e-3, pe=1e-2,
             T=20, shots=1021),
        # the paper's BP-OSD order on a noisy bicycle memory
        dict(name="bb144_osd_cs", kind="osd_cs", code="bb144", op="memory", rb=12, ra=0, p=2e-3, pe=2e-3, T=30,
             shots=8192),
        # one step of the training that made the shipped weights
        dict(name="bb144_teleport_train", kind="train", code="bb144", op="teleport", rb=4, ra=3, p=1e-3, pe=1e-2,
             T=20, shots=512),
        # storing the syndromes of a large block
        dict(name="sc21_sample", kind="sample", code="sc", d=21, op="nlcnot", rb=21, ra=21, p=1e-3, pe=1e-2, T=20,
             shots=65536),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """A case of the same ranges: d = 3..21 surface codes and the bicycle codes, 1 to 10^6 shots."""
    kind = rng.choice(["step", "step", "step", "step", "sample", "posteriors", "osd_cs", "train", "learned", "plan"])
    p = float("%.2g" % _log(rng, 1e-4, 1e-3))
    if kind == "learned":                                   # the circuit the shipped weights are for
        return dict(kind=kind, code="bb144", op="teleport", rb=4, ra=3, p=1e-3, pe=1e-2, T=20,
                    shots=int(_log(rng, 257, 8192)))
    if kind == "plan":
        d = rng.choice([3, 5, 7, 9, 11])
        return dict(kind=kind, code="sc", d=d, d2=d + rng.choice([2, 4]), op="nlcnot", p=p, p2=float("%.2g" % (1.7 * p)),
                    T=20, shots=SHOTS_PER_BLOCK * rng.choice([1, 1, 2]))
    if kind == "osd_cs":
        c = dict(kind=kind, code=rng.choice(["bb18", "bb36", "bb54", "bb144"]), op="memory", rb=rng.randint(3, 12), ra=0)
        p = float("%.2g" % _log(rng, 5e-4, 2e-3))
        return dict(c, p=p, pe=p, T=30, shots=int(_log(rng, 257, 8192)))
    if kind == "train":
        c = rng.choice([dict(code="sc", d=3), dict(code="sc", d=5), dict(code="bb18"), dict(code="bb54")])
        return dict(kind=kind, **c, op="nlcnot", rb=4, ra=3, p=1e-3, pe=1e-2, T=rng.choice([6, 8, 10, 12, 20]),
                    shots=int(_log(rng, 63, 512)))
    if kind != "posteriors" and rng.random() < 0.3:         # bicycle codes
        code = rng.choice(["bb18", "bb36", "bb54", "bb90", "bb144"])
        op = rng.choice(["memory", "nlcnot", "teleport"])
        rb, ra = (rng.randint(3, 12), 0) if op == "memory" else (4, 3)
        return dict(kind=kind, code=code, op=op, rb=rb, ra=ra, p=p, pe=p if op == "memory" else 10 * p, T=30,
                    shots=int(_log(rng, 1, 24000)))
    d = rng.choice([3, 5, 7, 9, 11, 13, 15, 17, 21])
    c = dict(kind=kind, code="sc", d=d, T=rng.choice([20, 30]) if d < 17 else 20)
    op = rng.choice(["nlcnot", "nlcnot", "memory", "pstring"] if d <= 7 else ["nlcnot", "nlcnot", "memory"])
    if op == "pstring":
        c.update(op=op, w=rng.randint(2, 6), rb=4, ra=1, p=p, pe=p)
    elif op == "memory":
        c.update(op=op, rb=d, ra=0, p=p, pe=p)
    else:
        c.update(op=op, rb=d, ra=d, p=p, pe=10 * p)
        if rng.random() < 0.25:                             # ebits made a line at a time, some of them waiting
            c.update(rate=1e-3)
    most = 1000000 * (5.0 / d) ** 3 / 4 ** max(0.0, math.log(d / 5.0, 2.0))
    if kind == "posteriors":
        most = min(most, 4e8 / d ** 3 / 20)
    return dict(c, shots=int(_log(rng, 1, max(2.0, most))))


# ---------------------------------------------------------------- circuits
@functools.lru_cache(maxsize=None)
def _circuit(code, d, op, rb, ra, p, pe, w, rate):
    base = sc(d, op, rb, ra, p, pe) if code == "sc" else bb(code, op, rb, ra, p, pe)
    spec = pstring(base, w, rb) if op == "pstring" else base
    return tmcs.Circuit(with_decoherence(spec, rate, True) if rate else spec)


@functools.lru_cache(maxsize=None)
def _dem(*key):
    return tmcs.DEM(_circuit(*key))


def _key(c, d=None, p=None):
    d = c.get("d", 0) if d is None else d
    if c["kind"] == "plan":
        return c["code"], d, c["op"], d, d, p, 10 * p, 0, 0.0
    return c["code"], d, c["op"], c["rb"], c["ra"], c["p"], c["pe"], c.get("w", 0), c.get("rate", 0.0)


@functools.lru_cache(maxsize=None)
def _weights(T, edges):
    """The learned weights that the package ships for the teleport circuit."""
    name = "bb144_teleport_p0.001_pe0.01_r4-3_T20.npz"
    w = np.load(os.path.join(os.path.dirname(tmcs.__file__), "weights", name))["weights"].astype(np.float32)
    return torch.from_numpy(w).cuda() if w.shape == (T, edges) else None


def _train_weights(c, dem, seed):
    """Weights in the middle of a training run: near the shipped or unit weights, no two alike."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    w = _weights(c["T"], dem.edges) if c["code"] == "bb144" else None
    w = torch.ones((c["T"], dem.edges), device="cuda") if w is None else w
    return (w + 0.05 * torch.randn(w.shape, generator=g, device="cuda")).clamp_(0.05, 4.0)


def _plan_items(c):
    return [(d, p) for d in (c["d"], c["d2"]) for p in (c["p"], c["p2"])]


# ---------------------------------------------------------------- the four functions
def prepare(case, seed):
    c, n = case, case["shots"]
    s = dict(kind=c["kind"], case=c, seed=seed, n=n, at=0, span=(n + 63) // 64 * 64)
    if c["kind"] == "plan":
        s["circuits"] = [_circuit(*_key(c, d, p)) for d, p in _plan_items(c)]
        s["dems"] = [_dem(*_key(c, d, p)) for d, p in _plan_items(c)]
        items = [(a, b, tmcs.make_cfg(max_iter=c["T"]), seed, i) for i, (a, b) in enumerate(zip(s["circuits"], s["dems"]))]
        s["plan"] = tmcs.Plan(items, n, use_graph=True)
        return s
    s["circuit"] = circ = _circuit(*_key(c))
    s["det"], s["obs"] = det, obs = circ.alloc_outputs(n)
    s["overflow"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    if c["kind"] == "sample":
        return s
    s["dem"] = dem = _dem(*_key(c))
    s["pred"], s["stats"] = torch.zeros_like(obs), tmcs.new_stats()
    s["errors"] = torch.zeros(1, dtype=torch.int64, device="cuda")
    if c["kind"] == "step":
        return s
    circ.sample(seed, 0, 0, n, det, obs)
    if c["kind"] == "posteriors":
        s["out"] = dict(ehat=torch.empty((n, dem.cols), dtype=torch.uint8, device="cuda"),
                        llr=torch.empty((n, dem.cols), dtype=torch.float32, device="cuda"),
                        iters=torch.empty(n, dtype=torch.int32, device="cuda"),
                        flags=torch.empty(n, dtype=torch.uint8, device="cuda"))
    elif c["kind"] == "learned":
        s["weights"] = _weights(c["T"], dem.edges)
    elif c["kind"] == "train":
        s["weights"] = _train_weights(c, dem, seed).requires_grad_(True)
        s["supp"] = neural_bp.observable_support(dem).cuda()
        s["bits"] = neural_bp.unpack_obs(obs, n, circ.num_observables)
    return s


def run(s):
    c, n = s["case"], s["n"]
    if s["kind"] == "plan":
        s["plan"].run(1)
        got = [s["plan"].result(i) for i in range(len(s["dems"]))]
        return [np.array([r[k] for k in sorted(r) if k != "bp_iter_hist"] + r["bp_iter_hist"]) for r in got]
    if s["kind"] in ("step", "sample"):
        s["circuit"].sample_async(s["seed"], 0, s["at"] * s["span"], n, s["det"], s["obs"], s["overflow"])
        s["at"] += 1
        if s["kind"] == "sample":
            return dict(det=s["det"], obs=s["obs"], overflow=s["overflow"])
        s["dem"].decode(s["det"], n, s["pred"], max_iter=c["T"], stats=s["stats"])
        tmcs.count_errors(s["pred"], s["obs"], s["circuit"].num_observables, n, s["errors"])
        return dict(det=s["det"], obs=s["obs"], pred=s["pred"], stats=s["stats"], errors=s["errors"],
                    overflow=s["overflow"])
    if s["kind"] == "train":
        llr = neural_bp.WeightedBP.apply(s["weights"], s["det"], s["dem"], n)
        loss = neural_bp.observable_loss(llr[-1:], s["bits"], s["supp"]) / n
        (grad,) = torch.autograd.grad(loss, s["weights"])
        return dict(loss=loss.detach(), grad=grad)
    more = dict(weights=s.get("weights"), use_osd=s["kind"] != "posteriors", osd_order=7 if s["kind"] == "osd_cs" else 0)
    s["dem"].decode(s["det"], n, s["pred"], max_iter=c["T"], stats=s["stats"], **more, **s.get("out", {}))
    return dict(pred=s["pred"], stats=s["stats"], **s.get("out", {}))


def work(case):
    """Bytes: detector and observable bits written by the sampler, detector bits read and prediction bits
    written by the decoder, weights, posteriors and gradients where a case has them.  Operations: the
    sampler's frame updates (4 per CX and 64 shots) and ten per edge for one BP iteration of every shot
    (training: for each of its T iterations, both ways); more iterations depend on the shot."""
    c, n = case, case["shots"]
    keys = [_key(c, d, p) for d, p in _plan_items(c)] if c["kind"] == "plan" else [_key(c)]
    byts = ops = 0.0
    for key in keys:
        circ = _circuit(*key)
        det, obs = circ.num_detectors * n / 8.0, circ.num_observables * n / 8.0
        if c["kind"] in ("step", "sample", "plan"):
            byts += det + obs
            ops += 4.0 * circ.info["gates_2q"] * n / 64.0
        if c["kind"] == "sample":
            continue
        dem = _dem(*key)
        byts += det + obs
        ops += 10.0 * dem.edges * n * (2 * c["T"] if c["kind"] == "train" else 1)
        if c["kind"] == "posteriors":
            byts += n * (5.0 * dem.cols + 5.0)
        if c["kind"] == "learned":
            byts += 4.0 * c["T"] * dem.edges
        if c["kind"] == "train":
            byts += 8.0 * c["T"] * dem.edges
    return dict(bytes=byts, flops=ops)


def exact(case, seed):
    """Training: loss and gradient of weighted min-sum BP in 64 bits with torch's own autograd, for up to a
    dozen iterations: a rounding difference doubles every one or two on a loopy graph, and at twenty the
    64-bit gradient is another one (measured: 1.1 times its norm away).  The other kinds return whole
    numbers, or posteriors at the iteration where FP32 stops, which 64-bit BP does not define either."""
    if case["kind"] != "train" or case["T"] > 12:
        return None
    c, n = case, case["shots"]
    s = prepare(case, seed)
    h, T = s["dem"].export(), case["T"]
    m, cols, E = s["dem"].rows, s["dem"].cols, s["dem"].edges
    dev = "cuda"
    # edges in row order: check, column
    col = np.repeat(np.arange(cols), np.diff(h.col_ptr))
    order = np.lexsort((col, h.row_idx))
    ec, ev = (torch.from_numpy(x[order].astype(np.int64)).to(dev) for x in (h.row_idx, col))
    lam = torch.from_numpy(np.log((1.0 - h.priors) / h.priors)).to(dev)
    words = s["det"][:, :, None] >> torch.arange(64, device=dev)
    synd = (words & 1).reshape(m, -1)[:, :n].bool()                                    # [m, n]
    w = s["weights"].detach().double().requires_grad_(True)
    idx = torch.arange(E, device=dev)[:, None].expand(E, n)

    def per_check(x, fill, how):
        return torch.full((m, n), fill, dtype=x.dtype, device=dev).scatter_reduce(0, ec[:, None].expand(E, n), x, how)

    q, L = lam[ev][:, None].expand(E, n), None
    for t in range(T):
        with torch.no_grad():
            a = q.abs()
            first = per_check(torch.where(a == per_check(a, math.inf, "amin")[ec], idx, E), E, "amin")
            rest = torch.where(idx == first[ec], math.inf, a)
            low = per_check(rest, math.inf, "amin")
            second = per_check(torch.where((rest == low[ec]) & (rest < math.inf), idx, E), E, "amin")
            src = torch.where(idx == first[ec], second[ec], first[ec])
            lone = src >= E
            neg = q < 0
            odd = torch.zeros((m, n), dtype=torch.int64, device=dev).index_add_(0, ec, neg.long())
            sign = 1.0 - 2.0 * ((odd[ec] + neg.long() + synd[ec].long()) % 2).double()
        mu = torch.where(lone, 1e30, q.abs().gather(0, src.clamp(max=E - 1)))
        msg = w[t][:, None] * sign * mu
        L = lam[:, None] + torch.zeros((cols, n), dtype=torch.float64, device=dev).index_add(0, ev, msg)
        q = L[ev] - msg
    x = L.T                                                                            # [n, cols]
    a = x.abs().clamp_min(1e-6)
    logt = (torch.log1p(-torch.exp(-a)) - torch.log1p(torch.exp(-a))).clamp_min(-60.0)
    supp = s["supp"].double()
    tot = logt @ supp.T
    odd = torch.remainder((x < 0).double() @ supp.T, 2.0) > 0.5
    up, down = 1.0 + torch.exp(tot), -torch.expm1(tot)
    one, zero = torch.where(odd, up, down), torch.where(odd, down, up)
    y = s["bits"].double()
    half = math.log(2.0)
    loss = -(y * (one.clamp_min(1e-30).log() - half) + (1 - y) * (zero.clamp_min(1e-30).log() - half)).sum() / n
    (grad,) = torch.autograd.grad(loss, w)
    return dict(loss=loss.detach(), grad=grad)
