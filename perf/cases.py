"""Timed cases of the PM-LSH query path: what a program that uses this library has it do.

A case is one call (or one burst of calls) through the public binding: building an
index, (c,k)-ANN batches (Algorithm 2) with equal or per-query parameters, the serving
loop, and (c,k)-ACP in its three forms (Section 6.3 and 6.1).

  listed()             the fixed cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  data on the GPU and the index or server that a program keeps
  run(state)           one pass, returning its outputs
  work(case)           bytes and operations that one pass cannot do without
  exact(case, seed)    the outputs of run() in 64 bits, by plain torch
"""

import math
import random

import numpy as np
import torch

import paper_2107_05537_amd as pm

M = 15                      # hash functions (Section 7.1)
CONFIDENCE = 1 - 1 / math.e
SAMPLE_SEED = 0x5EED
KAPPA = 0.9
DEVICE = "cuda"
MIXED_K = (1, 10, 50, 100)
MIXED_C = (1.2, 1.5, 2.0)


def _ann(name, n, d, nq, k, beta, data="mixture", c=1.5, confidence=CONFIDENCE, gemm=0):
    return {"name": name, "kind": "ann", "data": data, "n": n, "d": d, "nq": nq, "k": k,
            "c": c, "confidence": confidence, "beta": beta, "gemm": gemm}


def listed():
    return [
        # one user's query against a resident index: latency and launches
        _ann("ann_single", 1_000_000, 256, 1, 10, 8.75e-4),
        # a small collection searched by a small batch, generous budget (the parity workload)
        _ann("ann_small", 10_000, 128, 100, 10, 0.1, confidence=0.9),
        # the benchmark's batch: 1M x 256 at recall@10 >= 0.9
        _ann("ann_headline", 1_000_000, 256, 1024, 10, 8.75e-4),
        # sizes that are multiples of nothing, long answers, the FP16 filter projection
        _ann("ann_ragged_fp16", 300_007, 203, 777, 50, 2.5e-3, gemm=1),
        # wide rows without contrast (1M x 960): the range filter prunes nothing
        _ann("ann_low_contrast", 1_000_000, 960, 1024, 10, 1e-3, data="heavy"),
        # the paper's beta for c = 2 (beta = 2 alpha2 of Eq. 10): a budget of 4,800 points
        _ann("ann_c2_paper_beta", 1_000_000, 256, 1024, 10, -1.0, c=2.0),
        # every parameter left at its default: c = 1.5, a budget of 10 % of the points
        _ann("ann_defaults", 200_000, 128, 256, 10, -1.0),
        # the serving configuration's index (10M x 128) and a launch of mixed requests
        {"name": "mixed_10m", "kind": "mixed", "data": "bytes", "n": 10_000_000, "d": 128,
         "nq": 1024, "beta": 7.5e-5},
        # a burst of requests of all sizes through the serving loop
        {"name": "serve_burst", "kind": "serve", "data": "bytes", "n": 2_000_000, "d": 128,
         "requests": 96, "largest": 512, "beta": 2.5e-4},
        # indexing a new collection
        {"name": "build_1m", "kind": "build", "data": "mixture", "n": 1_000_000, "d": 256,
         "gemm": 0},
        # near-duplicate search over a collection: the benchmark's closest-pair workload
        {"name": "acp_planted", "kind": "acp", "variant": "filter", "n": 200_000, "d": 512,
         "k": 10, "beta": -1.0},
        # the same question by FindLCA (Algorithms 4 and 5) on a smaller, odd-sized collection
        {"name": "acp_lca", "kind": "acp", "variant": "lca", "n": 50_021, "d": 130, "k": 100,
         "beta": -1.0},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("ann", "ann", "ann", "budget", "contrast", "mixed", "serve", "build",
                       "acp", "acp"))
    n = _log(rng, 4_000, 1_000_000)
    d = min(_log(rng, 24, 960), 256_000_000 // n)
    if kind == "ann":
        budget = _log(rng, 150, 1_900)
        return {"kind": "ann", "data": rng.choice(("mixture", "bytes")), "n": n, "d": d,
                "nq": _log(rng, 1, 3_000), "k": rng.choice((1, 5, 10, 50, 100)),
                "c": rng.choice(MIXED_C), "confidence": rng.choice((CONFIDENCE, 0.9)),
                "beta": round(budget / n, 7), "gemm": rng.choice((0, 0, 1, 2))}
    if kind == "budget":    # 2,000 points up to a tenth of the collection, or the paper's beta
        n, d = _log(rng, 30_000, 600_000), _log(rng, 24, 300)
        budget = _log(rng, 2_000, min(n // 10, 20_000))
        return {"kind": "ann", "data": "mixture", "n": n, "d": d,
                "nq": _log(rng, 8, max(9, 2_500_000 // budget)),
                "k": rng.choice((1, 10, 100)), "c": rng.choice((1.5, 2.0)),
                "confidence": CONFIDENCE, "beta": round(budget / n, 6), "gemm": 0}
    if kind == "contrast":
        n, d = _log(rng, 50_000, 600_000), _log(rng, 200, 960)
        return {"kind": "ann", "data": "heavy", "n": n, "d": min(d, 400_000_000 // n),
                "nq": _log(rng, 16, 600), "k": 10, "c": rng.choice(MIXED_C),
                "confidence": CONFIDENCE, "beta": round(_log(rng, 300, 3_000) / n, 7), "gemm": 0}
    if kind == "mixed":
        return {"kind": "mixed", "data": "bytes", "n": n, "d": d, "nq": _log(rng, 2, 2_000),
                "beta": round(_log(rng, 200, 1_500) / n, 7)}
    if kind == "serve":
        return {"kind": "serve", "data": "bytes", "n": n, "d": d,
                "requests": _log(rng, 8, 150), "largest": _log(rng, 16, 600),
                "beta": round(_log(rng, 200, 900) / n, 7)}
    if kind == "build":
        return {"kind": "build", "data": rng.choice(("mixture", "bytes")), "n": n, "d": d,
                "gemm": rng.choice((0, 0, 1, 2))}
    variant = rng.choice(("filter", "filter", "lca", "bb"))
    n = _log(rng, 4_000, 180_000 if variant == "filter" else 50_000)
    # Algorithm 3 collects beta n^2 / 2 pairs: a beta that keeps them near a million
    return {"kind": "acp", "variant": variant, "n": n, "d": _log(rng, 24, 512),
            "k": rng.choice((1, 10, 30)),
            "beta": round(_log(rng, 20_000, 1_000_000) * 2.0 / n / n, 9) if variant == "bb"
            else -1.0}


# ---------------------------------------------------------------- inputs

def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    return g


def _rows(case, count, g, centres, sigmas):
    d = case["d"]
    if case["data"] == "heavy":
        # non-negative heavy-tailed features, rows scaled to norm 100
        x = torch.randn(count, d, generator=g, device=DEVICE).abs_().pow_(1.5)
        return x.mul_(100.0 / x.norm(dim=1, keepdim=True))
    lab = torch.randint(centres.shape[0], (count,), generator=g, device=DEVICE)
    x = torch.randn(count, d, generator=g, device=DEVICE)
    x.mul_(sigmas[lab, None]).add_(centres[lab])
    if case["data"] == "bytes":
        # pixel-like values, held to 16 bits
        x = x.clamp_(0.0, 255.0).half().float()
    return x


def _inputs(case, seed, nq):
    """Points, queries and hash matrix of a case."""
    g = _generator(seed)
    n, d = case["n"], case["d"]
    centres = sigmas = None
    if case["data"] != "heavy":
        nc = max(16, n // 1000)
        centres = torch.randn(nc, d, generator=g, device=DEVICE).mul_(2.0)
        sigmas = torch.rand(nc, generator=g, device=DEVICE).mul_(0.3).add_(0.2)
        if case["data"] == "bytes":
            centres = torch.rand(nc, d, generator=g, device=DEVICE).mul_(255.0)
            sigmas = torch.rand(nc, generator=g, device=DEVICE).mul_(12.0).add_(4.0)
    D = _rows(case, n, g, centres, sigmas)
    Q = _rows(case, nq, g, centres, sigmas)
    A = torch.randn(M, d, generator=g, device=DEVICE)
    return D, Q, A


def _planted(case, seed):
    """A mixture in which every hundredth point is a near copy of another one."""
    g = _generator(seed)
    n, d = case["n"], case["d"]
    copies = max(case["k"], n // 100)
    centres = torch.randn(max(8, n // 400), d, generator=g, device=DEVICE).mul_(2.0)
    sigmas = torch.rand(centres.shape[0], generator=g, device=DEVICE).mul_(0.3).add_(0.2)
    X = _rows({"d": d, "data": "mixture"}, n - copies, g, centres, sigmas)
    src = torch.randperm(n - copies, generator=g, device=DEVICE)[:copies]
    noise = torch.randn(copies, d, generator=g, device=DEVICE)
    A = torch.randn(M, d, generator=g, device=DEVICE)
    return torch.cat([X, X[src] + 1e-3 * noise]), A, src


def _mixed_params(case, seed):
    rng = random.Random(int(seed) ^ 0x51)
    return [{"k": rng.choice(MIXED_K), "c": rng.choice(MIXED_C), "beta": case["beta"]}
            for _ in range(case["nq"])]


def _requests(case, seed):
    """(queries, k, c) of each request, its sizes log-uniform in [1, largest]. The sizes belong
    to the case, so that a burst of another seed is another set of points of the same load."""
    sizes = random.Random(case["requests"] * 1009 + case["largest"])
    out = []
    for _ in range(case["requests"]):
        out.append((_log(sizes, 1, case["largest"]), sizes.choice(MIXED_K),
                    sizes.choice(MIXED_C)))
    return out


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case}
    if kind == "acp":
        D, A, _ = _planted(case, seed)
        state["index"] = pm.Index(D, A)
        return state
    if kind == "build":
        state["data"], _, state["hash"] = _inputs(case, seed, 1)
        return state
    reqs = _requests(case, seed) if kind == "serve" else None
    nq = sum(r[0] for r in reqs) if reqs else case["nq"]
    D, Q, A = _inputs(case, seed, nq)
    index = state["index"] = pm.Index(D, A, filter_gemm=case.get("gemm", 0))
    state["queries"] = Q
    if kind == "mixed":
        state["params"] = _mixed_params(case, seed)
    elif kind == "serve":
        # answers go to one buffer per output, a contiguous piece for each request
        total = sum(b * k for b, k, _ in reqs)
        state["ids"] = torch.empty(total, dtype=torch.int64, device=DEVICE)
        state["dist"] = torch.empty(total, dtype=torch.float32, device=DEVICE)
        state["server"] = pm.Server(index)
        work, q, o = [], 0, 0
        for b, k, c in reqs:
            work.append((Q[q:q + b], k, c, (state["ids"][o:o + b * k].view(b, k),
                                           state["dist"][o:o + b * k].view(b, k))))
            q, o = q + b, o + b * k
        state["requests"] = work
    return state


# ---------------------------------------------------------------- the pass

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "ann":
        return state["index"].ann(state["queries"], case["k"], c=case["c"],
                                  confidence=case["confidence"], beta=case["beta"])
    if kind == "mixed":
        return state["index"].ann_mixed(state["queries"], state["params"])
    if kind == "serve":
        server, beta = state["server"], case["beta"]
        pending = [server.submit(q, k, c=c, beta=beta, out=out)
                   for q, k, c, out in state["requests"]]
        for p in pending:
            p.wait()
        return state["ids"], state["dist"]
    if kind == "build":
        index = pm.Index(state["data"], state["hash"], filter_gemm=case["gemm"])
        perm, offsets = index.export_leaves()
        # the nodes come level by level, the leaves last; the inner ones are as many as the
        # data makes them
        return perm, offsets, index.export_nodes()["radius"][1 - len(offsets):]
    call = {"filter": state["index"].acp, "lca": state["index"].acp_lca,
            "bb": state["index"].acp_bb}[case["variant"]]
    pairs, dist, _ = call(case["k"], beta=case["beta"])
    return pairs, dist


# ---------------------------------------------------------------- what a pass needs

def _chi2_cdf(x):
    return float(torch.special.gammainc(torch.tensor(M / 2, dtype=torch.float64),
                                        torch.tensor(x / 2, dtype=torch.float64)))


def _plan(n, k, c, confidence, beta):
    """t and B of Algorithm 2 (Eq. 10, Lemma 5)."""
    lo, hi = 0.0, 200.0
    for _ in range(200):    # t^2: the point that a chi-square variable stays below w.p. confidence
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if _chi2_cdf(mid) < confidence else (lo, mid)
    t2 = 0.5 * (lo + hi)
    if beta < 0:
        beta = 2 * _chi2_cdf(t2 / (c * c))
    return math.sqrt(t2), min(n, math.ceil(beta * n) + k)


def work(case):
    """Every candidate's row and projection read once (a row that several queries verify counts
    once), the queries read and the answers written; the projections and the distances computed."""
    n, d, kind = case["n"], case["d"], case["kind"]
    if kind == "build":
        # the data in; rows in 32 and 16 bits and projections (two halves, filter rows) out
        return {"bytes": n * (4 * d + 4 * d + 2 * d + 2 * 64 + 48), "flops": 2 * n * d * M}
    if kind == "acp":
        # every row, and every pair inside a leaf of 64 points by the Gram matrix
        return {"bytes": 4 * n * d + 8 * n * M + 20 * case["k"],
                "flops": 2 * n * 32 * d + 2 * n * M * 64}
    if kind == "ann":
        parts = [(case["nq"], case["k"], case["c"], case["confidence"])]
    elif kind == "mixed":
        share = case["nq"] / (len(MIXED_K) * len(MIXED_C))
        parts = [(share, k, c, CONFIDENCE) for k in MIXED_K for c in MIXED_C]
    else:
        parts = [(b, k, c, CONFIDENCE) for b, k, c in _requests(case, 0)]
    rows = sum(nq * _plan(n, k, c, conf, case["beta"])[1] for nq, k, c, conf in parts)
    nq = sum(p[0] for p in parts)
    return {"bytes": min(n, rows) * (4 * d + 4 * M) + nq * 4 * d
            + sum(12 * q * k for q, k, _, _ in parts),
            "flops": 2 * nq * d * M + 3 * rows * (d + M)}


# ---------------------------------------------------------------- 64 bits

def _splitmix64(x):
    """First output of the SplitMix64 generator (Steele, Lea and Flood 2014) for each state."""
    z = x + np.uint64(0x9E3779B97F4A7C15)
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _sample(D):
    """Sorted distances of the pair sample behind the first radius (Section 5.2)."""
    n = D.shape[0]
    s = min(n * (n - 1) // 2, 100_000)
    j = np.arange(s, dtype=np.uint64)
    i = _splitmix64(j + np.uint64(SAMPLE_SEED)) % np.uint64(n)
    step = _splitmix64(j + np.uint64(SAMPLE_SEED + s)) % np.uint64(n - 1)
    l = (i + np.uint64(1) + step) % np.uint64(n)
    i = torch.from_numpy(i.astype(np.int64)).to(D.device)
    l = torch.from_numpy(l.astype(np.int64)).to(D.device)
    out = []
    for a in range(0, s, 10_000):
        diff = D[i[a:a + 10_000]].double() - D[l[a:a + 10_000]].double()
        out.append(diff.square().sum(1).sqrt())
    return torch.cat(out).sort().values.cpu()


def _algorithm2(D, Q, A, params):
    """Algorithm 2 for each query: (ids, distances) with params[i] = (k, c, confidence, beta)."""
    n = D.shape[0]
    A64 = A.double()
    P = torch.cat([D[a:a + 1_000_000].double() @ A64.T for a in range(0, n, 1_000_000)])
    QP = Q.double() @ A64.T
    pp = P.square().sum(1)
    sample = _sample(D)
    plans = {}
    for p in set(params):
        t, B = _plan(n, *p)
        at = max(0, math.ceil(min(1.0, B / n) * sample.numel()) - 1)
        plans[p] = (t, B, KAPPA * float(sample[at]))
    most = max(B for _, B, _ in plans.values())
    step = max(1, min(64, int(2e9 / 8 / max(n, most * (D.shape[1] + M)))))
    answers = []
    for a in range(0, Q.shape[0], step):
        q, qp = Q[a:a + step].double(), QP[a:a + step]
        near = torch.topk((pp - 2.0 * (qp @ P.T)), most, dim=1, largest=False).indices
        pd = (P[near] - qp[:, None, :]).square().sum(2).sqrt()
        pd, order = pd.sort(dim=1)
        near = near.gather(1, order)
        dist = torch.empty_like(pd)
        for b in range(q.shape[0]):
            dist[b] = (D[near[b]].double() - q[b]).square_().sum(1).sqrt()
        inside, found = pd.cpu().numpy(), dist.cpu().numpy()
        ids = near.cpu().numpy()
        for b in range(q.shape[0]):
            k, c = params[a + b][:2]
            t, B, r = plans[params[a + b]]
            members = 0
            for rounds in range(1000):
                if rounds and np.count_nonzero(found[b, :members] <= c * r) >= k:
                    break
                ball = int(np.searchsorted(inside[b, :B], t * r, side="right"))
                members = ball
                if ball >= B:
                    break
                r *= c
            best = np.lexsort((ids[b, :members], found[b, :members]))[:k]
            answers.append((ids[b, best], found[b, best]))
    return answers


def exact(case, seed):
    kind = case["kind"]
    if kind == "build":
        return None         # the partition and its radii are the index's own choice
    if kind == "acp":
        # the closest pairs: the copies, next to which every other pair is far
        D, _, src = _planted(case, seed)
        first = case["n"] - src.numel()
        dist = (D[first:].double() - D[src].double()).square().sum(1).sqrt()
        dist, order = dist.sort()
        pairs = torch.stack([src[order], order + first], 1)
        return pairs[:case["k"]], dist[:case["k"]]
    if kind == "serve":
        reqs = _requests(case, seed)
        params = [(k, c, CONFIDENCE, case["beta"]) for b, k, c in reqs for _ in range(b)]
    elif kind == "mixed":
        params = [(p["k"], p["c"], CONFIDENCE, p["beta"]) for p in _mixed_params(case, seed)]
    else:
        params = [(case["k"], case["c"], case["confidence"], case["beta"])] * case["nq"]
    D, Q, A = _inputs(case, seed, len(params))
    answers = _algorithm2(D, Q, A, params)
    if kind == "serve":
        return (np.concatenate([i for i, _ in answers]),
                np.concatenate([x for _, x in answers]))
    wide = max(p[0] for p in params)
    ids = np.full((len(params), wide), -1, dtype=np.int64)
    dist = np.full((len(params), wide), np.inf)
    for row, (i, x) in enumerate(answers):
        ids[row, :len(i)], dist[row, :len(x)] = i, x
    return ids, dist
