"""Queries of a wide budget finish in an order of their own: every answer has to
stay with its query, whatever their number."""

import numpy as np
import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# below and at the least number ordered, around a wave's 64 and a window's 1,024
@pytest.mark.parametrize("nq", [63, 64, 65, 127, 1_023, 1_024, 1_025, 1_100, 2_049])
@pytest.mark.parametrize("kind", ["distinct", "equal"])
def test_answers_stay_with_their_queries(nq, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    say(f"case: query order nq={nq} {kind}")
    rng = np.random.default_rng(nq)
    n, d, budget = 12_289, 24, 2_100
    D = (rng.standard_normal((n, d)) + 6 * rng.integers(0, 5, (n, 1))).astype(np.float32)
    A = rng.standard_normal((15, d)).astype(np.float32)
    Q = (D[rng.integers(0, n, nq)] + 0.1 * rng.standard_normal((nq, d))).astype(np.float32)
    if kind == "equal":         # one group for all: ranked by index
        Q[:] = Q[0]
    idx = pm.Index(torch.from_numpy(D).cuda(), torch.from_numpy(A).cuda())
    q = torch.from_numpy(Q).cuda()
    ids, dist, st = idx.ann(q, 7, beta=(budget - 7) / n, stats=True)
    for i in range(0, nq, 50):  # calls too small to be ordered
        a, b, s = idx.ann(q[i:i + 50], 7, beta=(budget - 7) / n, stats=True)
        assert torch.equal(ids[i:i + 50], a)
        np.testing.assert_array_equal(dist[i:i + 50].cpu().numpy(), b.cpu().numpy())
        assert torch.equal(st[i:i + 50, :3], s[:, :3])
