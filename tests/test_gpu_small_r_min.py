"""Algorithm 2 with a first radius far below that of a large budget: rounds answered
from one ball's points, the undecided queries from the budget's, against the per-query
kernel."""

import math

import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N, DIM, NQ, CONF = 60_011, 24, 200, 1 - 1 / math.e


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    return pm


def _call(idx, Q, k, c, beta, r_min, noalloc=False):
    nq = Q.shape[0]
    out = (torch.empty((nq, k), dtype=torch.int64, device="cuda"),
           torch.empty((nq, k), dtype=torch.float32, device="cuda"),
           torch.empty((nq, 4), dtype=torch.int32, device="cuda"))
    (idx.ann_noalloc if noalloc else idx.ann_into)(Q, k, c, CONF, beta, r_min, *out)
    return out[0], out[1], out[2][:, :3]


def _same(pm, idx, Q, *args):
    pm.tune(pm.TUNE_FP32_PATH, 1)
    try:
        ref = _call(idx, Q, *args)
    finally:
        pm.tune(pm.TUNE_FP32_PATH)
    one = Q[3:4].contiguous()
    for got, rows in ((_call(idx, Q, *args), slice(None)), (_call(idx, one, *args), slice(3, 4)),
                      (_call(idx, Q, *args, noalloc=True), slice(None))):
        for x, y in zip(got, ref):
            assert torch.equal(x, y[rows])
    return ref


# queries decided in the first round, in later ones, and not before the budget's radius;
# first radii on both sides of the rule's two steps (0.3 and 0.7 of that radius)
@pytest.mark.parametrize("k,c", [(1, 1.5), (10, 1.1), (10, 1.5), (200, 4.0)])
@pytest.mark.parametrize("kind,mode", [("clusters", 0), ("clusters", 2), ("plain", 0), ("plain", 1)])
@pytest.mark.parametrize("budget", [2_049, 9_000])
def test_first_radii(budget, kind, mode, k, c):
    pm = _gpu()
    g = torch.Generator(device="cuda").manual_seed(13)
    x = torch.randn(N, DIM, generator=g, device="cuda")
    if kind == "clusters":
        x = x + 4 * torch.randn(40, DIM, generator=g, device="cuda")[
            torch.randint(40, (N,), generator=g, device="cuda")]
    # groups of 20 near duplicates
    x[-4_000:] = x[:200].repeat_interleave(20, 0) + 1e-2 * torch.randn(
        4_000, DIM, generator=g, device="cuda")
    Q = torch.cat([x[:50] + 1e-3, x[300:400] + 0.3 * torch.randn(100, DIM, generator=g, device="cuda"),
                   3 * torch.randn(50, DIM, generator=g, device="cuda")])
    Q[7, 3], Q[8, 0] = math.nan, math.inf
    idx = pm.Index(x, torch.randn(15, DIM, generator=g, device="cuda"), filter_gemm=mode)
    beta = (budget - k) / N
    assert pm.plan_params(N, 15, k, c, CONF, beta)["budget"] == budget
    full = idx.default_r_min(budget)
    near = 0
    for f in (1e-4, 0.05, 0.2, 0.2999, 0.3001, 0.55, 0.6999, 0.7001, 1.0):
        say(f"case: small r_min B={budget} {kind} gemm={mode} k={k} c={c} r_min={f} of the budget's")
        ref = _same(pm, idx, Q.contiguous(), k, c, beta, f * full)
        near += int((ref[2][:, 2] == pm.EXIT_NEAR).sum())
    assert near > 0


def test_lists_that_outgrow_the_pools():
    """18,000 points within reach of some queries, where the sampled distances expect
    fewer than 2,049."""
    pm = _gpu()
    n = 200_000
    g = torch.Generator(device="cuda").manual_seed(14)
    x = 20 * torch.rand(n + 100, 8, generator=g, device="cuda")
    x[:18_000] = 5 + 0.01 * torch.randn(18_000, 8, generator=g, device="cuda")
    D, Q = x[:n].contiguous(), x[n:].contiguous()
    Q[:30] = D[:30]
    idx = pm.Index(D, torch.randn(10, 8, generator=g, device="cuda"))
    for f in (0.01, 0.2, 0.5):
        say(f"case: small r_min with lists of 18,000, r_min={f} of the budget's")
        _same(pm, idx, Q, 10, 1.5, (2_049 - 10) / n, f * idx.default_r_min(2_049))


def test_mixed_launches():
    """Queries with first radii of all sizes and budgets on both sides of 2,048 in one
    launch, alone and through the server."""
    pm = _gpu()
    g = torch.Generator(device="cuda").manual_seed(15)
    x = torch.randn(N, DIM, generator=g, device="cuda")
    x = x + 4 * torch.randn(40, DIM, generator=g, device="cuda")[
        torch.randint(40, (N,), generator=g, device="cuda")]
    x[-4_000:] = x[:200].repeat_interleave(20, 0) + 1e-2 * torch.randn(
        4_000, DIM, generator=g, device="cuda")
    Q = torch.cat([x[:60] + 1e-3, 3 * torch.randn(60, DIM, generator=g, device="cuda")])
    idx = pm.Index(x, torch.randn(15, DIM, generator=g, device="cuda"))
    params = []
    for i in range(120):
        budget = (200, 2_049, 9_000)[i % 3]
        k = (1, 10, 40)[i // 3 % 3]
        p = {"k": k, "c": (1.2, 2.0)[i // 9 % 2], "beta": (budget - k) / N}
        f = (0.0, 0.01, 0.25, 0.5, 1.5)[i // 18 % 5]
        if f:
            p["r_min"] = f * idx.default_r_min(budget)
        params.append(p)
    say("case: small r_min, mixed")
    ids, dist = idx.ann_mixed(Q, params, out_stride=40)
    server = pm.Server(idx)
    pending = [server.submit(Q[i:i + 1].contiguous(), p["k"], c=p["c"], beta=p["beta"],
                             r_min=p.get("r_min", 0.0)) for i, p in enumerate(params)]
    for i, (p, t) in enumerate(zip(params, pending)):
        t.wait()
        a, b, _ = _same(pm, idx, Q[i:i + 1].contiguous().expand(4, DIM).contiguous(), p["k"], p["c"],
                        p["beta"], p.get("r_min", 0.0))
        assert torch.equal(ids[i, :p["k"]], a[0]) and torch.equal(dist[i, :p["k"]], b[0])
        assert torch.equal(t.ids[0], a[0]) and torch.equal(t.dist[0], b[0])
    server.close()
