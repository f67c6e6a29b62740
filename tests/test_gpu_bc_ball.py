"""(r,c)-BC with budgets above 2,048: a filter that looks for the ball's points where the
ball is expected to hold fewer than the budget, against the per-query kernel."""

import math

import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N, DIM, NQ = 60_011, 24, 300


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    return pm


def _same(pm, idx, Q, r, beta):
    got = idx.bc(Q, r, beta=beta, stats=True)
    alone = idx.bc(Q[1:2].contiguous(), r, beta=beta)
    pm.tune(pm.TUNE_FP32_PATH, 1)
    try:
        ref = idx.bc(Q, r, beta=beta, stats=True)
    finally:
        pm.tune(pm.TUNE_FP32_PATH)
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    assert torch.equal(got[2][:, :3], ref[2][:, :3])
    assert torch.equal(alone[0], ref[0][1:2]) and torch.equal(alone[1], ref[1][1:2])
    return ref


# balls from empty to beyond the budget, on both sides of the rule (0.7 of the radius
# at which a ball is expected to hold the budget)
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("kind", ["clusters", "plain"])
@pytest.mark.parametrize("budget", [2_048, 2_049, 9_000])
def test_balls(budget, kind, mode):
    pm = _gpu()
    g = torch.Generator(device="cuda").manual_seed(11)
    x = torch.randn(N + NQ, DIM, generator=g, device="cuda")
    if kind == "clusters":
        centres = 4 * torch.randn(40, DIM, generator=g, device="cuda")
        x = x + centres[torch.randint(40, (N + NQ,), generator=g, device="cuda")]
    D, Q = x[:N].contiguous(), x[N:].contiguous()
    Q[:40] = D[:40]
    Q[7, 3], Q[8, 0], Q[9, 1] = math.nan, math.inf, 1e30
    idx = pm.Index(D, torch.randn(15, DIM, generator=g, device="cuda"), filter_gemm=mode)
    beta = (budget - 1) / N
    assert pm.plan_params(N, 15, 1, 1.5, 1 - 1 / math.e, beta)["budget"] == budget
    base = idx.default_r_min(budget)
    full = 0
    for f in (1e-6, 0.1, 0.3, 0.5, 0.6, 0.6999, 0.7001, 0.85, 1.0, 1.5):
        say(f"case: ball cover B={budget} {kind} gemm={mode} r={f} of r_min")
        ref = _same(pm, idx, Q, f * base, beta)
        full += int((ref[2][:, 2] == pm.EXIT_BUDGET).sum())
    assert 0 < full


def test_balls_that_outgrow_the_pools():
    """18,000 points within reach of some queries, where the sampled distances expect
    fewer than 2,049: their lists overflow, and the per-query kernel answers."""
    pm = _gpu()
    n = 200_000
    g = torch.Generator(device="cuda").manual_seed(12)
    x = 20 * torch.rand(n + 100, 8, generator=g, device="cuda")
    x[:18_000] = 5 + 0.01 * torch.randn(18_000, 8, generator=g, device="cuda")
    D, Q = x[:n].contiguous(), x[n:].contiguous()
    Q[:30] = D[:30]
    idx = pm.Index(D, torch.randn(10, 8, generator=g, device="cuda"))
    r = 0.5 * idx.default_r_min(2_049)
    say(f"case: ball cover with lists of 18,000, r={r}")
    ref = _same(pm, idx, Q, r, 2_048 / n)
    assert (ref[2][:30, 2] == pm.EXIT_BUDGET).all()


@pytest.mark.parametrize("nq", [512, 513])
def test_balls_far_below_the_budgets(nq):
    """Few and many queries of small balls: the routes on both sides of the rule agree."""
    pm = _gpu()
    g = torch.Generator(device="cuda").manual_seed(16)
    x = torch.randn(N, DIM, generator=g, device="cuda") + 4 * torch.randn(
        40, DIM, generator=g, device="cuda")[torch.randint(40, (N,), generator=g, device="cuda")]
    Q = (x[:nq] + 1e-2).contiguous()
    idx = pm.Index(x, torch.randn(15, DIM, generator=g, device="cuda"))
    for f in (0.02, 0.1999, 0.2001):
        say(f"case: ball cover nq={nq} r={f} of r_min")
        _same(pm, idx, Q, f * idx.default_r_min(2_049), 2_048 / N)
