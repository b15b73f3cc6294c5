"""Calls whose walks outgrow the first tier's queues: what the later tiers need is
made inside the call."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_1005_5384_amd import octgrav as og
from paper_1005_5384_amd import workloads as W

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("path", ["fused_wave", "fused_block", "two_pass"])
@pytest.mark.parametrize("n", [3000, 40000])
def test_little_memory_left_for_the_queues(n, path, monkeypatch):
    """The device refuses the queues of all waves: fewer waves walk, with the same results; it refuses a
    single queue: the call says so, and works once there is memory."""
    import torch
    pos, m = W.plummer(n, 5)
    monkeypatch.setenv("OCTGRAV_LDS_QUEUE", "64")
    ref = og.Tree(pos, m, 1, 64).forces(0.5, 0.01, path=path)
    T = og.Tree(pos, m, 1, 64)
    acc = torch.empty((n, 3), dtype=torch.float32, device="cuda")
    monkeypatch.setenv("OCTGRAV_ALLOC_LIMIT", "1000")
    with pytest.raises(og.OctgravError) as e:
        T.forces(0.5, 0.01, acc=acc, path=path)
    assert e.value.code == og.ENOMEM
    queue = 4  # bytes of a queue: 2 x the widest level + 64 entries of 4, up to a power of two
    while queue < 4 * (2 * T.stats["max_level_cells"] + 64):
        queue *= 2
    # the two-pass path also allocates its lists: all that is needed but the queues of more than 3 waves
    lists = 0 if path != "two_pass" else 64 << 20
    monkeypatch.setenv("OCTGRAV_ALLOC_LIMIT", str(max(3 * queue, lists)))
    a = T.forces(0.5, 0.01, path=path)
    assert torch.equal(a[0], ref[0]) and torch.equal(a[1], ref[1])


def test_little_memory_left_in_a_rebuilt_handle(monkeypatch):
    pos, vel, m = W.plummer_with_velocities(6000, 5)
    monkeypatch.setenv("OCTGRAV_LDS_QUEUE", "64")
    S = og.Sim(pos, vel, m, 1, 64)
    S.run(0.5, 0.01, 1.0 / 64, 3)
    F = og.Sim(pos, vel, m, 1, 64)
    F.run(1.0, 0.01, 0.0, 1)  # the arrays of the tree are in place, with headroom
    cells = og.Tree(pos, m, 1, 64, device_build=True).stats["n_cells"]
    # every array of the tree (80 bytes per cell the largest), not the 2048 waves' queues
    monkeypatch.setenv("OCTGRAV_ALLOC_LIMIT", str(100 * (2 * 6000 + 64)))
    assert 2048 * 4 * 4096 > 100 * (2 * 6000 + 64) > 80 * cells
    F.run(0.5, 0.01, 1.0 / 64, 3)
    for a, b in zip(S.state(), F.state()):
        assert np.array_equal(a, b)


TIERS = """
import sys, torch
from paper_1005_5384_amd import octgrav as og, workloads as W
pos, m = W.plummer(16384, 3)
T = og.Tree(pos, m, 1, 1)
for theta in (0.5, 0.1, 0.1, 0.5, 0.5):
    print("#", file=sys.stderr, flush=True)
    a = T.forces(theta, 0.01)
    print("# fresh", file=sys.stderr, flush=True)
    b = og.Tree(pos, m, 1, 1).forces(theta, 0.01)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
"""


def test_tiers_follow_the_calls():
    """After a call that left items to the later tiers the next one launches them at once, until one
    leaves none; the results are a fresh handle's."""
    r = subprocess.run([sys.executable, "-c", TIERS], cwd=ROOT, env=dict(os.environ, OCTGRAV_DEBUG="1"),
                       capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stderr
    ran = [["(run)" in l for l in c.splitlines() if "items" in l] for c in r.stderr.split("#")[1:]]
    # the first tier alone; the others after it; with it; with it once more, for nothing; alone again
    assert ran[::2] == [[False], [False, True], [True], [True], [False]], r.stderr
    assert ran[1::2] == [[False], [False, True], [False, True], [False], [False]], r.stderr


@pytest.mark.parametrize("n,theta", [(16384, 0.1), (5003, 0.1), (70000, 0.12)])
@pytest.mark.parametrize("learned", [False, True])
def test_more_items_than_the_later_tiers_hold(n, theta, learned):
    """Several items for each wave of the second tier, with its own queues: lists of the two-pass walk's
    lengths, forces within the gates of the oracle's."""
    import oracle
    from paper_1005_5384_amd import learned as L
    pos, m = W.plummer(n, 3)
    T = og.Tree(pos, m, 1, 1 if n < 20000 else 32)
    if learned:  # never accepted: the lists of theta
        T.set_mac(og.Mlp(L.init_params(1)), theta, 1.0, 0.0, float("inf"))
    acc, pot = T.forces(theta, 0.01)
    g = T.group_counts()
    T.set_mac(None)
    co, _, lo, _ = T.lists(theta, path="two_pass")
    assert np.array_equal(g[:, 0], np.diff(co)) and np.array_equal(g[:, 1], np.diff(lo))
    O = oracle.Tree(pos, m, 1, 1 if n < 20000 else 32)
    sel = np.random.default_rng(1).choice(O.n_groups, 100, replace=False)
    ar, pr = O.forces(theta, 0.01, groups=sel)
    k = ~np.isnan(pr)
    ea = oracle.rel_err(acc.double().cpu().numpy()[k], ar[k])
    ep = oracle.rel_err(pot.double().cpu().numpy()[k], pr[k])
    assert np.median(ea) <= 1e-5 and ea.max() <= 1e-4 and ep.max() <= 1e-4


@pytest.mark.parametrize("n,n_group", [(5003, 1), (10000, 1), (60000, 64)])
@pytest.mark.parametrize("theta", [0.1, float(np.nextafter(np.float32(0.3), np.float32(0))), 0.3])
def test_two_waves_with_the_larger_queue(n, n_group, theta):
    """Either side of the angle below which teams of two have it; some items outgrow it."""
    import oracle
    pos, m = W.plummer(n, 3)
    T = og.Tree(pos, m, 1, n_group)
    acc, pot = T.forces(theta, 0.01)
    g = T.group_counts()
    co, _, lo, _ = T.lists(theta, path="two_pass")
    assert np.array_equal(g[:, 0], np.diff(co)) and np.array_equal(g[:, 1], np.diff(lo))
    O = oracle.Tree(pos, m, 1, n_group)
    sel = np.random.default_rng(1).choice(O.n_groups, 100, replace=False)
    ar, pr = O.forces(theta, 0.01, groups=sel)
    k = ~np.isnan(pr)
    ea = oracle.rel_err(acc.double().cpu().numpy()[k], ar[k])
    ep = oracle.rel_err(pot.double().cpu().numpy()[k], pr[k])
    assert np.median(ea) <= 1e-5 and ea.max() <= 1e-4 and ep.max() <= 1e-4
