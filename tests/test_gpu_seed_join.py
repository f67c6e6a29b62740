"""The pairs inside leaves through FindLCA with a gamma so small that it finds no
node: the answer is the k nearest of them, and the reported upper bound the k-th
FP32 distance."""

import numpy as np
import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# columns: one block, below, at and above each half and whole of a 64-column
# step; leaves: full, the smallest, a last one of one, two and 63 points
@pytest.mark.parametrize("d", [1, 31, 33, 64, 65, 97, 128, 130, 260])
@pytest.mark.parametrize("n,leaf", [(193, 64), (130, 64), (1_087, 64), (640, 16), (101, 17)])
def test_pairs_inside_leaves(n, d, leaf):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    say(f"case: pairs inside leaves n={n} d={d} leaf={leaf}")
    rng = np.random.default_rng(1000 * n + d)
    D = rng.standard_normal((n, d)).astype(np.float32)
    A = rng.standard_normal((15, d)).astype(np.float32)
    idx = pm.Index(torch.from_numpy(D).cuda(), torch.from_numpy(A).cuda(), leaf_size=leaf)
    perm, off = idx.export_leaves()
    pairs = []
    for b, e in zip(off[:-1], off[1:]):
        ids = np.sort(np.asarray(perm[b:e], dtype=np.int64))
        i, j = np.triu_indices(len(ids), 1)
        pairs.append(np.stack([ids[i], ids[j]], 1))
    pairs = np.concatenate(pairs)
    d2 = ((D[pairs[:, 0]].astype(np.float64) - D[pairs[:, 1]]) ** 2).sum(1)
    order = np.lexsort((pairs[:, 1], pairs[:, 0], d2))
    for k in (1, 10, 100):
        got, dist, st = idx.acp_lca(k, beta=0.0, gamma=1e-12)
        torch.cuda.synchronize()
        best = order[:k]
        np.testing.assert_array_equal(got.cpu().numpy(), pairs[best])
        np.testing.assert_allclose(dist.cpu().numpy(), np.sqrt(d2[best]), rtol=2.0 ** -23)
        assert st["n_seed"] == len(pairs) and st["n_cand"] == 0
        # the differences' rounding enters a squared distance twice and each
        # sum's once: half of (d_pad / 4 + 4) u of it on the distance
        u = 2.0 ** -24
        assert abs(st["ub"] - np.sqrt(d2[best[-1]])) <= ((d + 3) / 8 + 4) * u * st["ub"]
