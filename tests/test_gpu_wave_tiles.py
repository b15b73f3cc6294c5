"""Edges of the fused wave kernel's tiles: every slice count that a work item
can have (targets 1 ... 32, hence tiles of 60 ... 64 sources), partial last
tiles, walk windows with few children per cell, and entries that pad a tile."""
import numpy as np
import pytest

import oracle
from paper_1005_5384_amd import octgrav as og
from paper_1005_5384_amd import workloads as W

pytestmark = pytest.mark.gpu


def _check(pos, m, n_leaf, n_group, theta, eps, acc_gate=True):
    T = og.Tree(pos, m, n_leaf, n_group)
    O = oracle.Tree(pos, m, n_leaf, n_group)
    for a, b in zip(T.lists(theta, path="fused_wave"), O.lists(theta)):
        assert np.array_equal(a, b)
    acc, pot = T.forces(theta, eps, path="fused_wave")
    ar, pr = O.forces(theta, eps)
    if len(m) == 1:  # the references are zero: nothing to be relative to
        assert (acc == 0).all() and (pot == 0).all() and not ar.any() and not pr.any()
        return
    ea = oracle.rel_err(acc.double().cpu().numpy(), ar)
    ep = oracle.rel_err(pot.double().cpu().numpy(), pr)
    # the gates of the parity tests
    if acc_gate:
        assert np.median(ea) <= 1e-5 and ea.max() <= 1e-4, (np.median(ea), ea.max())
    assert np.median(ep) <= 1e-5 and ep.max() <= 1e-4, (np.median(ep), ep.max())


@pytest.mark.parametrize("n_group", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 13, 16, 17, 21, 22, 31, 32, 33, 64])
def test_every_slice_count(n_group):
    pos, m = W.plummer(1500, 60 + n_group)
    _check(pos, m, min(16, n_group), n_group, 0.6, 0.01)


@pytest.mark.parametrize("n", [1, 2, 3, 31, 33, 59, 60, 61, 63, 64, 65, 127, 129])
def test_few_sources(n):
    """Leaf tiles of n sources for up to 32 targets, one leaf or several."""
    pos, m = W.plummer(n, 9)
    _check(pos, m, 16, 64, 0.5, 0.02)
    _check(pos, m, 64, 64, 0.5, 0.02)


def test_narrow_branching():
    """A line of points: at most two children per cell, windows mostly empty.
    Forces along a line nearly cancel (the net force of a point can be 1e-3 of
    its terms), so the relative gate holds for the potentials only."""
    x = np.sort(np.random.default_rng(4).uniform(-1, 1, 700)).astype(np.float32)
    pos = np.stack([x, 0 * x, 0 * x], axis=1)
    _check(pos, np.full(700, 1 / 700, np.float32), 2, 8, 0.7, 0.01, acc_gate=False)


def test_padding_at_a_target():
    """A target at the origin, its tree tiny and the softening far below the
    spacing: entries that pad a tile must not meet it at zero distance."""
    rng = np.random.default_rng(5)
    pos = rng.uniform(-1, 1, (40, 3)).astype(np.float32)
    pos[7] = 0.0
    m = rng.uniform(0.5, 1.0, 40).astype(np.float32)
    for n_leaf, n_group in ((1, 1), (4, 8), (16, 64)):
        T = og.Tree(pos, m, n_leaf, n_group)
        acc, pot = T.forces(0.8, 1e-6)
        assert np.isfinite(acc.cpu().numpy()).all() and np.isfinite(pot.cpu().numpy()).all()
        O = oracle.Tree(pos, m, n_leaf, n_group)
        ar, _ = O.forces(0.8, 1e-6)
        assert oracle.rel_err(acc.double().cpu().numpy(), ar).max() <= 1e-4


@pytest.mark.parametrize("n", [40, 900, 9000, 20000, 70000, 230000])
@pytest.mark.parametrize("cap", [None, "64"])
def test_waves_per_item(n, cap, monkeypatch):
    """Sizes on every branch of the waves-per-item rule (8, 4, 2, 1), with queues
    that hold every walk and with queues so small that items go to the later
    tiers: the same counts, diagnostics that match the outputs, forces against
    the oracle's on a sample of groups."""
    pos, m = W.plummer(n, 21)
    if cap:
        monkeypatch.setenv("OCTGRAV_LDS_QUEUE", cap)
    T = og.Tree(pos, m, 16, 64)
    monkeypatch.delenv("OCTGRAV_LDS_QUEUE", raising=False)
    O = oracle.Tree(pos, m, 16, 64)
    acc, pot = T.forces(0.6, 0.01)
    g = T.group_counts()
    co, _, lo, _ = O.lists(0.6)
    assert np.array_equal(g[:, 0], np.diff(co)) and np.array_equal(g[:, 1], np.diff(lo))
    c = T.last_counts()
    assert c["n_c"] == co[-1] and c["n_l"] == lo[-1]
    a, p = acc.double().cpu().numpy(), pot.double().cpu().numpy()
    sel = np.random.default_rng(2).choice(O.n_groups, min(200, O.n_groups), replace=False)
    ar, pr = O.forces(0.6, 0.01, groups=sel)
    k = ~np.isnan(pr)
    ea, ep = oracle.rel_err(a[k], ar[k]), oracle.rel_err(p[k], pr[k])
    assert np.median(ea) <= 1e-5 and ea.max() <= 1e-4 and ep.max() <= 1e-4
    mom, w = T.diagnostics()
    md = m.astype(np.float64)
    # FP64 sums of the same FP32 outputs in another order
    scale = np.abs(md[:, None] * a).sum(0)
    assert (np.abs(mom - (md[:, None] * a).sum(0)) <= 1e-12 * scale).all()
    assert abs(w - 0.5 * (md * p).sum()) <= 1e-12 * np.abs(md * p).sum()
    again = T.forces(0.6, 0.01)
    assert (again[0] == acc).all() and (again[1] == pot).all()
    assert T.diagnostics()[1] == w and (T.diagnostics()[0] == mom).all()


@pytest.mark.parametrize("n,n_leaf,n_group,theta", [(1500, 1, 64, 0.1), (3000, 1, 8, 0.3), (9000, 2, 64, 0.25),
                                                    (4000, 64, 64, 0.2), (24000, 1, 32, 0.35)])
def test_long_lists_of_few_items(n, n_leaf, n_group, theta):
    """Several rounds of cell tiles and of leaves for the waves of one item, and shared remainders."""
    pos, m = W.plummer_clumps(n, n)
    _check(pos, m, n_leaf, n_group, theta, 0.01, acc_gate=False)
    T = og.Tree(pos, m, n_leaf, n_group)
    O = oracle.Tree(pos, m, n_leaf, n_group)
    T.forces(theta, 0.01)
    co, _, lo, _ = O.lists(theta)
    g = T.group_counts()
    assert np.array_equal(g[:, 0], np.diff(co)) and np.array_equal(g[:, 1], np.diff(lo))
