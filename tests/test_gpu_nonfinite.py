"""Queries that are not finite end, find nothing, and leave the others alone."""

import math

import numpy as np
import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N, DIM, K = 5_003, 20, 7
BAD = {3: math.nan, 40: math.inf, 41: -math.inf, 69: math.nan}


def _setup(num_pivots):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    rng = np.random.default_rng(8)
    D = (rng.standard_normal((N, DIM)) + 5 * rng.integers(0, 9, (N, 1))).astype(np.float32)
    A = rng.standard_normal((15, DIM)).astype(np.float32)
    Q = (D[:70] + 0.1).astype(np.float32)
    idx = pm.Index(torch.from_numpy(D).cuda(), torch.from_numpy(A).cuda(), num_pivots=num_pivots)
    good = torch.from_numpy(Q).cuda()
    bad = good.clone()
    for row, value in BAD.items():
        bad[row, row % DIM] = value
    keep = torch.ones(70, dtype=torch.bool, device="cuda")
    keep[list(BAD)] = False
    return pm, idx, good, bad, keep


def _check(ids, dist, ref_ids, ref_dist, keep):
    assert torch.equal(ids[keep], ref_ids[keep]) and torch.equal(dist[keep], ref_dist[keep])
    for row, value in BAD.items():
        assert torch.isinf(dist[row]).all() and (dist[row] > 0).all(), (row, dist[row])
        if math.isnan(value):
            assert (ids[row] == -1).all(), (row, ids[row])


@pytest.mark.parametrize("plain", [0, 1])
@pytest.mark.parametrize("num_pivots", [0, 5])
@pytest.mark.parametrize("budget", [100, 2_500])
def test_ann(budget, num_pivots, plain):
    pm, idx, good, bad, keep = _setup(num_pivots)
    say(f"case: non-finite queries B={budget} pivots={num_pivots} plain path={plain}")
    beta = (budget - K) / N
    pm.tune(pm.TUNE_FP32_PATH, plain)
    try:
        ref = idx.ann(good, K, beta=beta)
        ids, dist, st = idx.ann(bad, K, beta=beta, stats=True)
        _check(ids, dist, *ref, keep)
        assert (st[[r for r, v in BAD.items() if math.isnan(v)], 1:3] == 0).all()
        _check(*idx.ann_mixed(bad, [{"k": K, "beta": beta}] * 70), *ref, keep)
    finally:
        pm.tune(pm.TUNE_FP32_PATH)


def test_ball_cover():
    pm, idx, good, bad, keep = _setup(5)
    say("case: non-finite ball cover queries")
    ref = idx.bc(good, 2.0)
    ids, dist = idx.bc(bad, 2.0)
    assert torch.equal(ids[keep], ref[0][keep]) and torch.equal(dist[keep], ref[1][keep])
    assert (ids[list(BAD)] == -1).all() and torch.isinf(dist[list(BAD)]).all()
