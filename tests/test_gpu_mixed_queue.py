"""Calls with per-query parameters queued behind other work: none waits for it, and
each reads its own parameters."""

import pytest

from parity import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_forty_calls_behind_a_long_kernel():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_05537_amd as pm
    say("case: forty mixed calls queued behind a kernel")
    g = torch.Generator(device="cuda").manual_seed(4)
    D = torch.randn(3_000, 16, generator=g, device="cuda")
    idx = pm.Index(D, torch.randn(15, 16, generator=g, device="cuda"))
    Q = torch.randn(64, 16, generator=g, device="cuda")
    sets = [[{"k": 1 + (i + j) % 9, "c": (1.2, 1.5, 2.0)[(i * j) % 3], "beta": 0.01 + 0.01 * (i % 5)}
             for j in range(64)] for i in range(40)]
    want = []
    for params in sets:         # one at a time
        want.append(idx.ann_mixed(Q, params))
        torch.cuda.synchronize()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        idx.ann_mixed(Q, sets[0])
        st.synchronize()
        torch.cuda._sleep(2_000_000_000)     # about a second
        busy = torch.cuda.Event()
        busy.record(st)
        got = [idx.ann_mixed(Q, params) for params in sets]
        waited = busy.query()
    st.synchronize()
    assert not waited, "a call waited for the work queued before it"
    for (a, b), (c, d) in zip(want, got):
        assert torch.equal(a, c) and torch.equal(b, d)
