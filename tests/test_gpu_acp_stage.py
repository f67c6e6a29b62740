"""Branch and bound around the sizes where the pair scan's stage and the cut of the
collected pairs change step: whatever T is, exactly the T projected-nearest pairs
are verified."""

import numpy as np
import pytest

import synth
from oracle import acp as oacp
from oracle import ann as oann
from oracle import chi2
from parity import compare_acp, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# T: a wave's 64 pairs, its stage of 256 and the 512 that a wave cuts at once, each
# with its neighbours; many stages; leaves: one ballot, a wave, narrow
@pytest.mark.parametrize("leaf", [8, 17, 64])
@pytest.mark.parametrize("T", [63, 64, 65, 255, 256, 257, 511, 512, 513, 2_049, 20_000, 200_000])
def test_branch_and_bound_verifies_T_pairs(T, leaf):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    say(f"case: branch and bound stage T={T} leaf={leaf}")
    w = synth.parity(n=900, n_queries=1)
    D, A = w["D"], w["A"]
    n, k = D.shape[0], 10
    idx = pm.Index(torch.from_numpy(D).cuda(), torch.from_numpy(A).cuda(), leaf_size=leaf)
    beta = (T - k - 0.5) / (n * (n - 1) / 2)     # rounded up
    assert chi2.acp_budget(beta, n, k) == T
    pairs, dist, st = idx.acp_bb(k, c=1.5, beta=beta)
    torch.cuda.synchronize()
    Dp = oann.project(D, A)

    def rerun(dT=0):
        return oacp.branch_and_bound(D, Dp, k, T + dT)

    assert st["n_cand"] == T and st["n_cand_raw"] >= T
    say(compare_acp(D, rerun(), pairs.cpu().numpy(), dist.cpu().numpy(), rerun=rerun))
