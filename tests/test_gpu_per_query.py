"""The per-query kernel for whole launches (the plain FP32 path, budgets beyond the
batched path's limit, a fixed workspace too small for the candidate pools), and the
largest budgets of the batched path against it."""

import numpy as np
import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CONF = 1 - 1 / np.e


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    pm.load_library()
    return pm


def _tuned(pm, settings, fn):
    for key, value in settings:
        pm.tune(key, value)
    try:
        return [t.cpu().numpy() for t in fn()]
    finally:
        for key, _ in settings:
            pm.tune(key)


def _same(a, b):
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x[:, :3] if x.shape[1] == 4 else x,
                                      y[:, :3] if y.shape[1] == 4 else y)


def _points(n, d, kind, seed, nq):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(n + nq, d, generator=g, device="cuda")
    if kind == "clusters":
        centres = 4 * torch.randn(200, d, generator=g, device="cuda")
        x = 0.4 * x + centres[torch.randint(200, (n + nq,), generator=g, device="cuda")]
    return x[:n].contiguous(), x[n:].contiguous(), torch.randn(15, d, generator=g, device="cuda")


def test_mixed_parameters_on_the_per_query_kernel():
    """Every query with its own parameters, none of them on the batched path."""
    pm = _gpu()
    say("case: mixed parameters, per-query kernel")
    D, Q, A = _points(12_007, 24, "clusters", 1, 90)
    idx = pm.Index(D, A)
    params = [{"k": 1 + 7 * (i % 9), "c": (1.2, 1.5, 2.0)[i % 3],
               "beta": (0.01, 0.1, 0.3)[i % 3 if i % 2 else 0]} for i in range(90)]
    got = _tuned(pm, [(pm.TUNE_FP32_PATH, 1)], lambda: idx.ann_mixed(Q, params, stats=True))
    for i in range(90):
        p = params[i]
        alone = [t.cpu().numpy() for t in idx.ann(Q[i:i + 1], p["k"], c=p["c"], beta=p["beta"],
                                                  stats=True)]
        np.testing.assert_array_equal(got[0][i, :p["k"]], alone[0][0])
        np.testing.assert_array_equal(got[1][i, :p["k"]], alone[1][0])
        np.testing.assert_array_equal(got[2][i, :3], alone[2][0, :3])


@pytest.mark.parametrize("budget", [300, 4_050])
def test_frontier_lists_in_the_fixed_workspace(budget):
    pm = _gpu()
    say(f"case: noalloc on the per-query kernel B={budget}")
    D, Q, A = _points(20_000, 32, "clusters", 2, 300)
    idx = pm.Index(D, A)
    beta = (budget - 50) / 20_000
    ref = [t.cpu().numpy() for t in idx.ann(Q, 50, c=2.0, beta=beta)]
    ids = torch.empty((300, 50), dtype=torch.int64, device="cuda")
    dist = torch.empty((300, 50), dtype=torch.float32, device="cuda")

    def call():
        idx.ann_noalloc(Q, 50, 2.0, CONF, beta, 0.0, ids, dist)
        return ids, dist
    _same(_tuned(pm, [(pm.TUNE_FP32_PATH, 1)], call), ref)


def test_fixed_workspace_too_small_for_the_pools():
    """34 million points: one query's chunk distances alone exceed the fixed array, so a
    budget above 2,048 takes the per-query kernel there, and the pools in pmlsh_ann."""
    pm = _gpu()
    say("case: noalloc without room for the pools, n=34M")
    D, Q, A = _points(34_000_000, 4, "clusters", 3, 3)
    idx = pm.Index(D, A[:4].contiguous())
    del D
    beta = 2_500 / 34_000_000
    ref = [t.cpu().numpy() for t in idx.ann(Q, 10, beta=beta, stats=True)]
    ids = torch.empty((3, 10), dtype=torch.int64, device="cuda")
    dist = torch.empty((3, 10), dtype=torch.float32, device="cuda")
    st = torch.empty((3, 4), dtype=torch.int32, device="cuda")
    idx.ann_noalloc(Q, 10, 1.5, CONF, beta, 0.0, ids, dist, st)
    _same([t.cpu().numpy() for t in (ids, dist, st)], ref)
    with pytest.raises(pm.PmlshError) as e:
        idx.ann_noalloc(Q, 10, 1.5, CONF, 1e-5, 0.0, ids, dist, st)
    assert e.value.code == pm.EUNSUPPORTED


def test_fixed_workspace_with_room_for_an_exact_filters_pools():
    """29.8 million points: the fixed array holds one query with 16,384 pool entries, not
    with the 32,768 that a low-precision filter takes at the largest lean budget."""
    pm = _gpu()
    say("case: noalloc with the least pools, n=29.765M")
    n = 29_765_000
    D, Q, A = _points(n, 4, "clusters", 5, 3)
    idx = pm.Index(D, A[:4].contiguous(), filter_gemm=pm.FILTER_GEMM_FP16)
    del D
    beta = (2_048 - 10) / n
    assert pm.plan_params(n, 4, 10, 1.5, CONF, beta)["budget"] == 2_048
    ref = [t.cpu().numpy() for t in idx.ann(Q, 10, beta=beta, stats=True)]
    ids = torch.empty((3, 10), dtype=torch.int64, device="cuda")
    dist = torch.empty((3, 10), dtype=torch.float32, device="cuda")
    st = torch.empty((3, 4), dtype=torch.int32, device="cuda")
    idx.ann_noalloc(Q, 10, 1.5, CONF, beta, 0.0, ids, dist, st)
    _same([t.cpu().numpy() for t in (ids, dist, st)], ref)


# budgets whose chosen chunks outgrow the usual list (from 32,736 points), at which its
# cap is reached (without contrast), and on both sides of the batched path's limit
@pytest.mark.parametrize("n,budget,kind", [
    (130_001, 32_736, "clusters"), (130_001, 32_800, "clusters"), (130_001, 60_000, "clusters"),
    (130_001, 33_000, "plain"), (220_000, 140_000, "plain"),
    (200_003, 196_608, "clusters"), (200_003, 196_609, "clusters"), (200_003, 196_608, "plain"),
])
def test_largest_budgets(n, budget, kind):
    pm = _gpu()
    say(f"case: largest budgets n={n} B={budget} {kind}")
    D, Q, A = _points(n, 12, kind, 4, 3)
    idx = pm.Index(D, A)
    assert pm.plan_params(n, 15, 9, 1.5, CONF, (budget - 9) / n)["budget"] == budget
    call = lambda: idx.ann(Q, 9, beta=(budget - 9) / n, stats=True)
    ref = _tuned(pm, [(pm.TUNE_FP32_PATH, 1)], call)
    for lds in (1, 0):
        for groups in (2048, 0):
            _same(_tuned(pm, [(pm.TUNE_GROUP_MINIMA_LDS, lds), (pm.TUNE_GROUP_LIST, groups)], call), ref)
    params = [{"k": 9, "beta": (budget - 9) / n}, {"k": 3, "beta": 1e-3}, {"k": 9, "beta": 0.02}]
    ids, dist = idx.ann_mixed(Q, params)
    for i, p in enumerate(params):
        a, b = idx.ann(Q[i:i + 1], p["k"], beta=p["beta"])
        assert torch.equal(ids[i, :p["k"]], a[0]) and torch.equal(dist[i, :p["k"]], b[0])


@pytest.mark.parametrize("n,nq", [(2_060, 257), (3_072, 256), (3_072, 257), (3_073, 257)])
def test_budgets_of_most_points(n, nq):
    """A few thousand points, most of them in the budget: the same answers by the hundred
    and one by one, whichever path takes them."""
    pm = _gpu()
    say(f"case: budgets of most points n={n} nq={nq}")
    D, Q, A = _points(n, 20, "clusters", 7, nq)
    idx = pm.Index(D, A)
    beta = (2_052 - 10) / n
    ref = [t.cpu().numpy() for t in idx.ann(Q, 10, beta=beta, stats=True)]
    for i in (0, 17, nq - 1):
        one = [t.cpu().numpy() for t in idx.ann(Q[i:i + 1].contiguous(), 10, beta=beta, stats=True)]
        _same(one, [t[i:i + 1] for t in ref])
    mixed = idx.ann_mixed(Q, [{"k": 10, "beta": beta}] * nq)
    _same([t.cpu().numpy() for t in mixed], ref[:2])
