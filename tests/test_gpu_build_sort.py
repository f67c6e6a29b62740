"""The leaf order of one-dimensional data: every split sorts by the same
coordinate, so the order is the stable sort of all points by value, whatever the
sizes of the ranges that the level sorts cut."""

import numpy as np
import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _perm(values):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    D = torch.from_numpy(values.astype(np.float32).reshape(-1, 1)).cuda()
    A = torch.ones(1, 1, device="cuda")
    return pm.Index(D, A).export_leaves()[0]


# one workgroup's largest range and one more; the smallest and largest ranges of
# one bucket pass; enough points that buckets are cut again
@pytest.mark.parametrize("n", [65, 4_096, 4_097, 6_145, 786_431, 786_433, 2_400_001])
@pytest.mark.parametrize("kind", ["distinct", "ties", "outliers"])
def test_order_is_the_stable_sort(n, kind):
    say(f"case: build sort n={n} {kind}")
    rng = np.random.default_rng(n)
    x = rng.standard_normal(n).astype(np.float32)
    if kind == "ties":      # 7 values, and a tenth of the points in one
        x = np.round(x).clip(-3, 3)
    elif kind == "outliers":
        x[rng.integers(0, n, 5)] *= np.float32(1e12)
    np.testing.assert_array_equal(_perm(x), np.argsort(x + np.float32(0), kind="stable"))


def test_equal_points_keep_their_order():
    say("case: build sort, equal points")
    np.testing.assert_array_equal(_perm(np.full(50_000, 3.25)), np.arange(50_000))
