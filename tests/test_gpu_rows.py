"""The copies of the rows that a build makes: with a budget of every point the
answer is the exact one, whatever the rows' length and alignment."""

import numpy as np
import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# columns: one, around a lane's four, a wave's 64 and 256, and the 1,024 that a
# wave holds; the rows from an aligned base and from one 4 bytes on; magnitudes
# whose power of two has no normal inverse (their squares are zero in FP32, so
# all points are equally near and the smallest ids win)
@pytest.mark.parametrize("d", [1, 3, 4, 5, 63, 64, 65, 255, 256, 257, 1_023, 1_024, 1_025, 1_030, 2_052])
@pytest.mark.parametrize("shift,scale", [(0, 1.0), (1, 1.0), (0, 1e-37)])
def test_exact_answers(d, shift, scale):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    say(f"case: rows d={d} shift={shift} scale={scale}")
    rng = np.random.default_rng(d)
    n, nq, k = 1_000, 9, 5
    flat = (rng.standard_normal(n * d + shift) * scale).astype(np.float32)
    if scale == 1.0:
        flat[::97] = 0
    D = flat[shift:].reshape(n, d)
    rows = torch.from_numpy(flat).cuda()[shift:].view(n, d)
    Q = (rng.standard_normal((nq, d)) * scale).astype(np.float32)
    A = rng.standard_normal((15, d)).astype(np.float32)
    idx = pm.Index(rows, torch.from_numpy(A).cuda())
    ids, dist = idx.ann(torch.from_numpy(Q).cuda(), k, beta=1.0, r_min=1e30)[:2]
    if scale != 1.0:
        np.testing.assert_array_equal(ids.cpu().numpy(), np.tile(np.arange(k), (nq, 1)))
        return
    d2 = ((Q[:, None].astype(np.float64) - D[None]) ** 2).sum(2)
    order = np.argsort(d2, axis=1, kind="stable")[:, :k]
    np.testing.assert_array_equal(ids.cpu().numpy(), order)
    want = np.sqrt(np.take_along_axis(d2, order, 1))
    np.testing.assert_allclose(dist.cpu().numpy(), want, rtol=2.0 ** -23)
