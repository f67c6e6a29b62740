"""Candidate lists of a low-precision filter, several times as long as an exact one's,
in the pools: the answers are the exact index's."""

import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# lists around the LDS lists' 2,048 entries, in the usual pools, in the longer ones and
# beyond them; budgets on both sides of 2,048
@pytest.mark.parametrize("mode", ["FP16", "BF16"])
@pytest.mark.parametrize("kind", ["clusters", "plain"])
@pytest.mark.parametrize("budget", [40, 700, 2_048, 2_049, 6_000])
def test_same_answers(mode, kind, budget):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    say(f"case: filter pools {mode} {kind} B={budget}")
    n, d, k = 150_001, 96, 10
    g = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn(n + 70, d, generator=g, device="cuda")
    if kind == "clusters":
        centres = 4 * torch.randn(60, d, generator=g, device="cuda")
        x = x + centres[torch.randint(60, (n + 70,), generator=g, device="cuda")]
    D, Q = x[:n].contiguous(), x[n:].contiguous()
    A = torch.randn(15, d, generator=g, device="cuda")
    exact = pm.Index(D, A)
    low = pm.Index(D, A, filter_gemm=getattr(pm, f"FILTER_GEMM_{mode}"))
    beta = (budget - k) / n
    for nq in (1, 70):
        ref = exact.ann(Q[:nq], k, beta=beta, stats=True)
        got = low.ann(Q[:nq], k, beta=beta, stats=True)
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
        assert torch.equal(got[2][:, :3], ref[2][:, :3])
