"""Budgets beyond one workgroup's LDS lists, and long candidate lists, on the
batched path.

The per-query kernel (PMLSH_TUNE_FP32_PATH: a walk of the tree in FP32 with the
same FP64 decisions) answers the same calls; ids, distances, rounds, |C| and
exit kinds have to be equal. One case of each kind is also held to the oracle.
"""

import numpy as np
import pytest

import synth
from parity import compare_ann, oracle_ann, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    pm.load_library()
    return pm


def _both(pm, idx, Q, k, **kw):
    out = []
    for plain in (0, 1):
        pm.tune(pm.TUNE_FP32_PATH, plain)
        try:
            out.append([t.cpu().numpy() for t in idx.ann(Q, k, stats=True, **kw)])
        finally:
            pm.tune(pm.TUNE_FP32_PATH)
    (i0, d0, s0), (i1, d1, s1) = out
    np.testing.assert_array_equal(i0, i1)
    np.testing.assert_array_equal(d0, d1)
    np.testing.assert_array_equal(s0[:, :3], s1[:, :3])
    return out[0]


def _index(pm, D, A, **kw):
    return pm.Index(torch.from_numpy(D).cuda(), torch.from_numpy(A).cuda(), **kw)


# n, d, nq, k, budget, c, r_min (0: the default), filter_gemm: the smallest wide
# budget and its neighbours, B = n, several rounds, more than 512 members in the
# re-rank, ragged sizes
@pytest.mark.parametrize("n,d,nq,k,budget,c,r_min,gemm", [
    (9_001, 33, 5, 1, 2_048, 1.5, 0.0, 0),
    (9_001, 33, 5, 1, 2_049, 1.5, 0.0, 0),
    (9_001, 33, 70, 600, 2_700, 1.5, 0.0, 0),
    (4_097, 64, 3, 10, 4_097, 2.0, 1e30, 0),
    (20_000, 20, 33, 100, 5_000, 1.2, 1.5, 0),
    (70_003, 40, 129, 10, 20_011, 1.5, 0.0, 1),
    (70_003, 40, 9, 50, 30_000, 1.1, 0.4, 2),
])
def test_wide_budget_equals_the_per_query_kernel(n, d, nq, k, budget, c, r_min, gemm):
    pm = _gpu()
    say(f"case: wide n={n} d={d} nq={nq} k={k} B={budget} c={c} r_min={r_min} gemm={gemm}")
    spec = synth.MixtureSpec(n=n, d=d, n_centres=40, centre_std=1.0, sigma_lo=0.2, sigma_hi=0.6,
                             n_queries=nq)
    w = synth.mixture(spec, 11)
    D, A, Q = w["D"], w["A"], w["Q"]
    idx = _index(pm, D, A, filter_gemm=gemm)
    beta = (budget - k) / n
    ids, dist, st = _both(pm, idx, torch.from_numpy(Q).cuda(), k, c=c, beta=beta, r_min=r_min)
    sub = Q[:3]
    r0 = r_min if r_min > 0 else idx.default_r_min(pm.plan_params(n, 15, k, c, 1 - 1 / np.e,
                                                                 beta)["budget"])
    res, _ = oracle_ann(D, A, sub, k, c, 1 - 1 / np.e, beta, r_min=r0)
    compare_ann(D, sub, res, ids[:3], dist[:3], st[:3], fp64=True, min_exact_frac=0.0)


@pytest.mark.parametrize("budget", [300, 2_500, 9_000])
def test_many_equal_points(budget):
    """Every point occurs up to 40 times: ties at the budget cut by id."""
    pm = _gpu()
    say(f"case: equal points B={budget}")
    rng = np.random.default_rng(5)
    base = rng.standard_normal((1_000, 24)).astype(np.float32)
    D = base[rng.integers(0, 1_000, 30_000) % rng.integers(1, 1_001, 30_000)]
    A = rng.standard_normal((15, 24)).astype(np.float32)
    Q = np.concatenate([base[:4], rng.standard_normal((6, 24)).astype(np.float32)])
    idx = _index(pm, D, A)
    for r_min in (0.0, 1e30):
        _both(pm, idx, torch.from_numpy(Q).cuda(), 10, beta=(budget - 10) / 30_000, r_min=r_min)


@pytest.mark.parametrize("n,d,nq,budget", [(60_000, 96, 40, 900), (60_000, 96, 40, 3_000),
                                           (120_000, 32, 600, 1_500)])
def test_no_contrast(n, d, nq, budget):
    """Gaussian data without clusters: candidate lists several times the budget."""
    pm = _gpu()
    say(f"case: no contrast n={n} nq={nq} B={budget}")
    rng = np.random.default_rng(6)
    D = rng.standard_normal((n, d)).astype(np.float32)
    Q = rng.standard_normal((nq, d)).astype(np.float32)
    A = rng.standard_normal((15, d)).astype(np.float32)
    idx = _index(pm, D, A)
    _both(pm, idx, torch.from_numpy(Q).cuda(), 10, beta=(budget - 10) / n)


def test_wide_budgets_in_one_launch_and_without_allocation():
    """Budgets on both sides of the LDS limit in one launch equal the queries
    alone, and the fixed-workspace call equals the allocating one."""
    pm = _gpu()
    say("case: mixed wide budgets, noalloc")
    w = synth.parity(n=30_000, n_queries=64)
    idx = _index(pm, w["D"], w["A"])
    Q = torch.from_numpy(w["Q"]).cuda()
    params = [{"k": 1 + i % 7, "c": (1.2, 1.5, 2.0)[i % 3],
               "beta": (0.005, 0.06, 0.0685, 0.3)[i % 4]} for i in range(64)]
    ids, dist = idx.ann_mixed(Q, params)
    for i in (0, 1, 2, 3, 34, 63):
        p = params[i]
        a, b = idx.ann(Q[i:i + 1], p["k"], c=p["c"], beta=p["beta"])
        assert torch.equal(ids[i, :p["k"]], a[0]) and torch.equal(dist[i, :p["k"]], b[0])
    a, b = idx.ann(Q, 10, beta=0.3)
    c, e = torch.empty_like(a), torch.empty_like(b)
    idx.ann_noalloc(Q, 10, 1.5, 1 - 1 / np.e, 0.3, 0.0, c, e)
    assert torch.equal(a, c) and torch.equal(b, e)
