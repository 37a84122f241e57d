"""Alias tables among empty distributions.  Empty ones break the offsets' rule,
but each is only reported (RTF_ERR_ZERO_TOTAL) and samples to -1; the others'
tables are built whatever their size, also where the average or the number of
distributions leaves no room for it under the rule."""
import ctypes

import numpy as np
import pytest

from gpu_util import note, to_dev


@pytest.fixture(scope="module")
def rtf():
    import torch  # noqa: F401 (its HIP runtime first)
    import paper_1901_05423_amd as rtf
    rtf.lib()
    return rtf


# one table beyond the 4096 items a block keeps in LDS, the others empty
EMPTY = [(130, 40, 4200), (2, 1, 4097), (104, 0, 4199), (1000, 999, 32000)]


@pytest.mark.parametrize("D,d,n", EMPTY)
def test_workspace_holds_the_sums_of_a_large_table(rtf, D, d, n):
    """records (16 bytes an item), the list (4) and the 128-bit sums (16)"""
    assert rtf.lib().rtf_alias_workspace_bytes(D, n) >= 36 * n


def export_all(rtf, t):
    n, D = t.desc.n_total, t.desc.D
    thr, alias, W = np.zeros(n, np.uint64), np.zeros(n, np.int32), np.zeros(D, np.uint64)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    code = rtf.lib().rtf_alias_export(ctypes.byref(t.desc), p(thr), p(alias), p(W), None)
    assert code == rtf.RTF_ERR_ZERO_TOTAL
    return thr, alias, W


@pytest.mark.gpu
@pytest.mark.parametrize("D,d,n", EMPTY)
def test_large_table_among_empty_ones(rtf, orc, D, d, n):
    note(f"alias among empty D={D} d={d} n={n}")
    rng = np.random.default_rng(n)
    w = np.floor(np.exp(rng.uniform(0, np.log(2.0 ** 32 - 1), n))).astype(np.uint32)
    off = lambda c: np.concatenate([np.zeros(d + 1, np.int64), np.full(D - d, c, np.int64)])  # noqa: E731
    t = rtf.alias_build(to_dev(w), to_dev(off(n)))
    thr, alias, W = export_all(rtf, t)
    ref = orc.alias_build(w)
    assert int(W[d]) == ref.W and not np.delete(W, d).any()
    assert np.array_equal(thr, ref.thr) and np.array_equal(alias, ref.alias)
    u = rng.integers(0, 2 ** 64, 5000, dtype=np.uint64)
    idx = rtf.alias_sample(t, to_dev(u), to_dev(off(u.size))).cpu().numpy()
    assert np.array_equal(idx, orc.alias_sample(ref, u))


@pytest.mark.gpu
def test_2d_row_among_empty_ones(rtf, orc):
    """a marginal of five items, one row of 4150, the other rows empty"""
    note("alias 2D among empty rows")
    rng = np.random.default_rng(7)
    w = rng.integers(1, 2 ** 32, 4155, dtype=np.uint32)
    eo = np.concatenate([[0, 5], np.full(129, 4155)]).astype(np.int64)
    t = rtf.alias_build(to_dev(w), to_dev(eo))
    export_all(rtf, t)
    u = rng.integers(0, 2 ** 64, (5000, 2), dtype=np.uint64)
    rc = rtf.alias_sample_2d(t, to_dev(u)).cpu().numpy()
    r_ref = orc.alias_sample(orc.alias_build(w[:5]), np.ascontiguousarray(u[:, 0]))
    c_ref = orc.alias_sample(orc.alias_build(w[5:]), np.ascontiguousarray(u[:, 1]))
    assert np.array_equal(rc[:, 0], r_ref)
    assert np.array_equal(rc[:, 1], np.where(r_ref == 0, c_ref, -1))
