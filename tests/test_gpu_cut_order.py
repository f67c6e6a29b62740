"""The budget cut of candidate lists longer than one workgroup's LDS keys.

The points around the B-th projected distance tie in FP32 and differ in FP64 (a
coordinate that the hash weighs with 2^-30), so the members of C, and with them
the answer, show which order cut the list. It has to be the FP64 one whichever
kernels finish the query: they are chosen by the number of queries, the budget and
the largest budget of the launch.
"""

import numpy as np
import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

K = 10
INNER = 400      # tied points


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    pm.load_library()
    return pm


def _data(budget):
    """budget - 200 points nearer in projection but far in space, 400 tied ones of
    which 200 fit the budget, 2,000 just behind them, and far clusters. The ids of
    the tied points run against their FP64 order."""
    rng = np.random.default_rng(3)
    near = np.zeros((budget - INNER // 2, 4), np.float32)
    near[:, 0] = rng.uniform(0.2, 0.9, near.shape[0])
    near[:, 3] = 100.0
    tied = np.zeros((INNER, 4), np.float32)
    tied[:, 0] = 1.0
    tied[:, 1] = np.arange(INNER, 0, -1) / 128.0
    behind = np.zeros((2_000, 4), np.float32)
    behind[:, 0] = 1.0005
    behind[:, 3] = 100.0
    far = np.repeat(rng.uniform(20.0, 200.0, (80, 1)), 64, axis=0).astype(np.float32)
    far = np.concatenate([far, np.zeros_like(far), far, np.zeros_like(far)], axis=1)
    D = np.concatenate([near, tied, behind, far])
    A = np.array([[1.0, 2.0 ** -30, 0.0, 0.0], [0.0, 0.0, 1.0, 0.0]], np.float32)
    # the answer from q = 0: the tied points of smallest second coordinate
    want = near.shape[0] + np.arange(INNER - 1, INNER - 1 - K, -1)
    return D, A, want


@pytest.mark.parametrize("budget", [800, 1_000, 1_535, 1_536, 2_048])
@pytest.mark.parametrize("nq", [1, 32, 33, 257, 513])
def test_long_list_is_cut_in_the_fp64_order(budget, nq):
    pm = _gpu()
    say(f"case: cut of a long list B={budget} nq={nq}")
    D, A, want = _data(budget)
    idx = pm.Index(torch.from_numpy(D).cuda(), torch.from_numpy(A).cuda())
    Q = torch.zeros((nq, 4), device="cuda")
    beta = (budget - K) / D.shape[0]
    kw = dict(c=1.5, beta=beta, r_min=50.0)
    assert pm.plan_params(D.shape[0], 2, K, 1.5, 1 - 1 / np.e, beta)["budget"] == budget
    ids, dist, st = idx.ann(Q, K, stats=True, **kw)
    np.testing.assert_array_equal(ids.cpu().numpy(), np.tile(want, (nq, 1)))
    assert (st[:, 1] == budget).all()
    # the fixed workspace (lists without their pd^2 bits), and a launch that a wide
    # budget takes to other kernels
    a, b = torch.empty_like(ids), torch.empty_like(dist)
    idx.ann_noalloc(Q, K, 1.5, 1 - 1 / np.e, beta, 50.0, a, b)
    assert torch.equal(a, ids) and torch.equal(b, dist)
    params = [{"k": K, **kw} for _ in range(nq)] + [{"k": K, "beta": 0.4, "r_min": 50.0}]
    a, b = idx.ann_mixed(torch.zeros((nq + 1, 4), device="cuda"), params)
    assert torch.equal(a[:nq], ids) and torch.equal(b[:nq], dist)
    if nq == 1:
        pm.tune(pm.TUNE_FP32_PATH, 1)
        try:
            a, b = idx.ann(Q, K, **kw)
        finally:
            pm.tune(pm.TUNE_FP32_PATH)
        assert torch.equal(a, ids) and torch.equal(b, dist)
