"""Closest pairs of data so small that squared projected distances are below the
smallest normal FP32 number: the pairs of the same data at scale one (powers of two
scale every coordinate exactly)."""

import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,d,leaf", [(4_000, 16, 64), (20_000, 24, 32), (3_000, 16, 128)])
def test_scaled_data_has_the_same_pairs(n, d, leaf):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    say(f"case: small scales n={n} d={d} leaf={leaf}")
    g = torch.Generator(device="cuda").manual_seed(3)
    centres = torch.randn(40, d, generator=g, device="cuda") * 3
    D = torch.randn(n, d, generator=g, device="cuda") * 0.5
    D += centres[torch.randint(40, (n,), generator=g, device="cuda")]
    A = torch.randn(15, d, generator=g, device="cuda")
    want = None
    for scale in (0, 40, 64, 66, 68):
        idx = pm.Index(D * 2.0 ** -scale, A, leaf_size=leaf)
        got = [idx.acp(50)[0], idx.acp_lca(50)[0], idx.acp_bb(50, beta=1e-3)[0]]
        if want is None:
            want = got
        for name, a, b in zip(("filter", "lca", "bb"), want, got):
            assert torch.equal(a, b), (name, scale)
