"""Calls of handles that got no page-locked host memory, and the report of a walk
that outgrows even its last tier's queues."""
import numpy as np
import pytest

from paper_1005_5384_amd import learned as L
from paper_1005_5384_amd import octgrav as og
from paper_1005_5384_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [None, "64"])  # "64": items go to the later tiers
@pytest.mark.parametrize("n", [1000, 30000])
def test_forces_without_pinned_memory(n, cap, monkeypatch):
    import torch
    pos, m = W.plummer(n, 11)
    if cap:
        monkeypatch.setenv("OCTGRAV_LDS_QUEUE", cap)
    A = og.Tree(pos, m, 16, 64)
    monkeypatch.setenv("OCTGRAV_FAIL_ALLOC", "2")
    B = og.Tree(pos, m, 16, 64)
    monkeypatch.delenv("OCTGRAV_FAIL_ALLOC")
    for theta in (0.6, 0.4, 0.6):
        a, b = A.forces(theta, 0.01), B.forces(theta, 0.01)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
        assert A.last_counts() == B.last_counts()
        da, db = A.diagnostics(), B.diagnostics()
        assert np.array_equal(da[0], db[0]) and da[1] == db[1]


def test_training_without_pinned_memory(monkeypatch):
    import torch
    x = torch.from_numpy(np.random.default_rng(1).uniform(0, 2, (700, 12)).astype(np.float32)).cuda()
    t = x[:, 0] - 4
    got = []
    for fault in ("0", "2"):
        monkeypatch.setenv("OCTGRAV_FAIL_ALLOC", fault)
        m = og.Mlp(L.init_params(3))
        loss, g = m.loss_grad(x, t)
        m.adam(1)
        got.append((loss, g, m.params()))
    assert got[0][0] == got[1][0]
    assert np.array_equal(got[0][1], got[1][1]) and np.array_equal(got[0][2], got[1][2])


@pytest.mark.parametrize("fault", ["0", "2"])
@pytest.mark.parametrize("n", [5003, 16384])  # two waves per work item, and one
def test_overflow_of_the_last_tier_is_reported(n, fault, monkeypatch):
    """Queues of 8 entries in the first tiers and 256 in the last: each call whose walks need more says
    that it failed, and a call whose walks fit is right again."""
    import torch
    pos, m = W.plummer(n, 3)
    ref = og.Tree(pos, m, 1, 1).forces(1.0, 0.01)
    monkeypatch.setenv("OCTGRAV_FAIL_ALLOC", fault)
    monkeypatch.setenv("OCTGRAV_LDS_QUEUE", "64")
    monkeypatch.setenv("OCTGRAV_FALLBACK_QUEUE", "256")
    T = og.Tree(pos, m, 1, 1)
    for _ in range(2):
        with pytest.raises(og.OctgravError, match="overflow") as e:
            T.forces(0.1, 0.01)  # walks of more than 512 entries
        assert e.value.code == og.ECAPACITY
    a = T.forces(1.0, 0.01)
    assert torch.equal(a[0], ref[0]) and torch.equal(a[1], ref[1])
