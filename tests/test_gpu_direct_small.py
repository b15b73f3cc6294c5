"""Direct sums that leave the chip idle: one target per lane, one tile per range;
and the line to two targets per lane."""
import numpy as np
import pytest

import oracle
from paper_1005_5384_amd import octgrav as og
from paper_1005_5384_amd import workloads as W

pytestmark = pytest.mark.gpu


# One target and its neighbours in a block of 64, one range and two, a ragged last range, and both sides of
# 4096 blocks of 128 targets times tiles of 256 particles (45 x 90 and 46 x 92; 9000 targets of 16385: 71 x 65).
@pytest.mark.parametrize("n,nt", [(1, None), (2, None), (63, None), (64, None), (65, None), (256, None), (257, None),
                                  (256, 64), (300, 65), (513, 1), (1000, 999), (4096, 63), (11520, None),
                                  (11700, None), (16385, 7000), (16385, 9000)])
def test_small_direct_sums_match_oracle(n, nt):
    pos, m = W.plummer(n, 7)
    T = og.Tree(pos, m, 16, 64)
    tg = None if nt is None else W.sample_indices(n, nt, 3)[::-1].copy()  # not in order
    acc, pot = T.direct(0.02, tg)
    ra, rp = oracle.direct(pos, m, 0.02, tg)
    a, p = acc.cpu().numpy().astype(np.float64), pot.cpu().numpy().astype(np.float64)
    # FP32 terms (relative error below 4 eps each: differences, r^2, rsq, products) under a
    # compensated sum, against the largest acceleration / potential of the set
    tol = 8 * 2.0 ** -24
    assert np.abs(a - ra).max() <= tol * max(np.abs(ra).max(), 1.0) * 4
    assert np.abs(p - rp).max() <= tol * max(np.abs(rp).max(), 1.0) * 4
    again = T.direct(0.02, tg)
    assert (again[0] == acc).all() and (again[1] == pot).all()


@pytest.mark.parametrize("n", [600, 12000])
def test_without_scratch(n, monkeypatch):
    """No memory for the ranges' sums: one range, the same sums to rounding."""
    pos, m = W.plummer(n, 7)
    T = og.Tree(pos, m, 16, 64)
    monkeypatch.setenv("OCTGRAV_ALLOC_LIMIT", "1000")
    a = T.direct(0.02)
    monkeypatch.delenv("OCTGRAV_ALLOC_LIMIT")
    b = T.direct(0.02)
    for u, v in zip(a, b):
        d = (u.double() - v.double()).abs().max()
        assert d <= 8 * 2.0 ** -24 * max(v.abs().max(), 1.0)


def test_absurd_number_of_targets_is_an_error():
    import ctypes
    import torch
    pos, m = W.plummer(100, 7)
    T = og.Tree(pos, m, 16, 64)
    out = torch.zeros(300, device="cuda")
    idx = torch.zeros(1, dtype=torch.int32, device="cuda")
    rc = og.lib().octgrav_direct(T._h, 0.01, ctypes.c_void_p(idx.data_ptr()), 1 << 61,
                                 ctypes.c_void_p(out.data_ptr()), None)
    assert rc == og.EINVAL and "nt" in og.last_error()
    assert (T.direct(0.01)[0] != 0).any()
