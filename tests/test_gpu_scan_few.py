"""The range filter on indexes of a few chunks, where every point may be a
candidate of every query: the same answers in every block shape, and as the
per-query kernel gives them."""

import numpy as np
import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# queries around a wave's 64 and a workgroup's 256; one point to some chunks
@pytest.mark.parametrize("nq", [1, 63, 65, 255, 257, 1_000])
@pytest.mark.parametrize("n,budget", [(1, 1), (65, 60), (200, 100), (1_111, 1_111)])
def test_few_chunks(n, budget, nq):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    say(f"case: few chunks n={n} B={budget} nq={nq}")
    rng = np.random.default_rng(n + nq)
    D = rng.standard_normal((n, 20)).astype(np.float32)
    A = rng.standard_normal((15, 20)).astype(np.float32)
    Q = torch.from_numpy(rng.standard_normal((nq, 20)).astype(np.float32)).cuda()
    idx = pm.Index(torch.from_numpy(D).cuda(), torch.from_numpy(A).cuda())
    k = min(5, n)
    out = []
    for key, value in ((pm.TUNE_SCAN_SHAPE, 0), (pm.TUNE_SCAN_SHAPE, 1), (pm.TUNE_SCAN_SHAPE, 2),
                       (pm.TUNE_FP32_PATH, 1)):
        pm.tune(key, value)
        try:
            ids, dist, st = idx.ann(Q, k, beta=(budget - k) / n, stats=True)
        finally:
            pm.tune(key)
        out.append((ids.cpu().numpy(), dist.cpu().numpy(), st[:, :3].cpu().numpy()))
    for o in out[1:]:
        for a, b in zip(out[0], o):
            np.testing.assert_array_equal(a, b)
