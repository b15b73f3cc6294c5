"""Device builds at their limits: trees of too many cells, the lines between the
builds' paths, and what a handle that is rebuilt in place falls back to."""
import numpy as np
import pytest

from paper_1005_5384_amd import octgrav as og
from paper_1005_5384_amd import workloads as W

pytestmark = pytest.mark.gpu


# One block, one block's sums, and (above 2^20 particles) the scan of the counts.
@pytest.mark.parametrize("n", [1500, 20000, (1 << 20) + 5])
def test_too_many_cells_are_refused(n, monkeypatch):
    pos, vel, m = W.plummer_with_velocities(n, 3)
    S = og.Sim(pos, vel, m, 16, 64)
    S.run(0.6, 0.01, 0.0, 1)
    before = S.state()
    cells = og.Tree(pos, m, 16, 64, device_build=True).stats["n_cells"]
    monkeypatch.setenv("OCTGRAV_MAX_CELLS", str(cells - 1))
    for device in (True, False):
        with pytest.raises(og.OctgravError, match=f"{cells} cells"):
            og.Tree(pos, m, 16, 64, device_build=device)
    F = og.Sim(pos, vel, m, 16, 64)
    with pytest.raises(og.OctgravError, match=f"{cells} cells") as e:
        F.run(0.6, 0.01, 0.0, 0)
    assert e.value.code == og.EINVAL
    monkeypatch.setenv("OCTGRAV_MAX_CELLS", str(cells))  # exactly as many as there may be
    F.run(0.6, 0.01, 0.0, 1)
    for a, b in zip(before, F.state()):
        assert np.array_equal(a, b)


def _same_tree(pos, m, n_leaf, n_group):
    H = og.Tree(pos, m, n_leaf, n_group)
    D = og.Tree(pos, m, n_leaf, n_group, device_build=True)
    assert D.stats == H.stats
    eh, ed = H.export(), D.export()
    for k in eh:
        assert np.array_equal(eh[k].view(np.uint8), ed[k].view(np.uint8)), k
    return H, D


# Either side of the line between the one-block build and the general one, 1400 + 470 n_leaf particles up to
# 7168, at the ends and in the middle of its range: bit for bit the host's tree, and the same forces.
@pytest.mark.parametrize("n_leaf,n_group", [(1, 1), (1, 64), (2, 17), (8, 64), (12, 200), (13, 64), (16, 64), (64, 1024)])
@pytest.mark.parametrize("past", [0, 1])
def test_line_of_the_one_block_build(n_leaf, n_group, past):
    import torch
    n = min(7168, 1400 + 470 * n_leaf) + past
    pos, m = W.milky_way(n, n_leaf)
    H, D = _same_tree(pos, m * np.random.default_rng(n).uniform(0.5, 2, n).astype(np.float32), n_leaf, n_group)
    a, b = H.forces(0.6, 0.01), D.forces(0.6, 0.01)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("n", [3000, 60000, (1 << 20) + 5])
@pytest.mark.parametrize("device", [True, False])
def test_memory_in_pieces(n, device, monkeypatch):
    """The device has room for every array of a tree, but not for several of them in one piece."""
    import torch
    pos, m = W.plummer(n, 4)
    ref = og.Tree(pos, m, 16, 64, device_build=device)
    a = ref.forces(0.75, 0.01)
    # the largest arrays: 16 bytes per particle, 80 per cell (for cells the arrays hold in the one-block build);
    # the library sort's scratch above 2^20 particles takes 16 more
    cells = 2 * n + 64 if n < 7168 else ref.stats["n_cells"]
    most = max((16 if n <= 1 << 20 else 32) * n, 80 * cells) + 4096
    assert most < 60 * n or n < 7168
    monkeypatch.setenv("OCTGRAV_ALLOC_LIMIT", str(most))
    T = og.Tree(pos, m, 16, 64, device_build=device)
    b = T.forces(0.75, 0.01)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    monkeypatch.setenv("OCTGRAV_ALLOC_LIMIT", str(4 * n))
    with pytest.raises(og.OctgravError, match="alloc|hipMalloc"):
        og.Tree(pos, m, 16, 64, device_build=device)
