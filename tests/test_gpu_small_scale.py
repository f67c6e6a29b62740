"""Data and queries of any magnitude: powers of two scale every coordinate exactly,
so the answers are those at scale one while squared distances are normal FP32
numbers, and are still answers where they are not (there the batched path's scan
rows cannot be formed)."""

import numpy as np
import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nq,budget", [(100, 200), (20, 900), (65, 2_500)])
def test_scaled_data(nq, budget):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    n, d, k = 9_000, 24, 10
    g = torch.Generator(device="cuda").manual_seed(5)
    centres = torch.randn(40, d, generator=g, device="cuda") * 3
    D = torch.randn(n, d, generator=g, device="cuda") * 0.5
    D += centres[torch.randint(40, (n,), generator=g, device="cuda")]
    Q = (D[:nq] + 0.1 * torch.randn(nq, d, generator=g, device="cuda")).contiguous()
    A = torch.randn(15, d, generator=g, device="cuda")
    want = None
    for scale in (0, -40, 40, 55, 66, 68, 70):
        say(f"case: scale 2^-{scale} nq={nq} B={budget}")
        s = 2.0 ** -scale
        idx = pm.Index(D * s, A)
        ids, dist, st = idx.ann(Q * s, k, beta=(budget - k) / n, stats=True)
        ids, dist, st = ids.cpu().numpy(), dist.cpu().numpy().astype(np.float64), st.cpu().numpy()
        if want is None:
            want = ids, dist, st
        if scale <= 55:
            np.testing.assert_array_equal(ids, want[0])
            np.testing.assert_array_equal(dist, want[1] * s)
            np.testing.assert_array_equal(st[:, :3], want[2][:, :3])
        else:
            # points of the collection, each once, at their distances
            assert ((ids >= 0) & (ids < n)).all()
            assert all(len(set(row)) == k for row in ids.tolist())
            rows = (D * s).double().cpu().numpy()[ids] - (Q * s).double().cpu().numpy()[:, None]
            np.testing.assert_allclose(dist, np.sqrt((rows ** 2).sum(2)), rtol=1e-6)
