"""2D sampling of distributions without mass: the build writes no guide cell
and no collapsed record for them, so nothing that the workspace held there may
start a search.  With a workspace of zeros such a search would stay at
collapsed record 0 for as many steps as the forest has nodes (a second here,
against microseconds); it must not begin."""
import ctypes

import numpy as np
import pytest

from gpu_util import assert_samples, note, to_dev

pytestmark = pytest.mark.gpu

COLS, PAIRS = 1 << 19, 4096
LIMIT_MS = 50  # the search takes well under 1 ms, the walk it replaces a few hundred


@pytest.fixture(scope="module")
def rtf():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1901_05423_amd as rtf
    rtf.lib()
    return rtf


def widened(rtf, w, eo, co):
    """A forest with collapsed records, built over workspaces of zeros."""
    import torch
    D, n, m = eo.size - 1, int(eo[-1]), int(co[-1])
    L = rtf.lib()
    nb = L.rtf_workspace_bytes_batched(D, n, m)
    ws = torch.zeros(nb, dtype=torch.uint8, device="cuda:0")
    wd, eod, cod = to_dev(w), to_dev(eo), to_dev(co)
    desc = rtf.rtf_forest()
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.rtf_build_batched(p(wd), p(eod), p(cod), D, n, m, p(ws), nb, st, ctypes.byref(desc)) == rtf.RTF_OK
    f = rtf.Forest(ws, desc, ws.device)
    return f.widen(ws=torch.zeros(L.rtf_wide_workspace_bytes(n), dtype=torch.uint8, device="cuda:0"))


@pytest.mark.parametrize("want_xy", [True, False])
@pytest.mark.parametrize("marginal", [(5, 0, 9), (0, 0, 0), (0, 7, 0)], ids=str)
@pytest.mark.parametrize("cells", [16, 2048])
def test_2d_without_mass(rtf, orc, cells, marginal, want_xy):
    """rows 0 and 2 hold mass, row 1 none"""
    import torch
    note(f"2D without mass cells={cells} marginal={marginal} want_xy={want_xy}")
    rng = np.random.default_rng(cells + sum(marginal))
    rows = [rng.integers(0, 2 ** 32, COLS, dtype=np.uint32) for _ in range(3)]
    rows[1][:] = 0
    marg = np.array(marginal, np.uint32)
    w = np.concatenate([marg, *rows])
    eo = np.concatenate([[0], 3 + COLS * np.arange(4)]).astype(np.int64)
    co = np.concatenate([[0], cells + cells * np.arange(4)]).astype(np.int64)
    f = widened(rtf, w, eo, co)
    u2 = rng.integers(0, 2 ** 64, 2 * PAIRS, dtype=np.uint64)
    u2[:4] = [0, 0, 2 ** 64 - 1, 2 ** 64 - 1]
    ud = to_dev(u2)
    rtf.sample_2d(f, ud[:2], want_xy=want_xy)  # loads the kernel
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    rc, xy = rtf.sample_2d(f, ud, want_xy=want_xy)
    b.record()
    b.synchronize()
    assert a.elapsed_time(b) < LIMIT_MS
    rc = rc.cpu().numpy()
    xy = xy.cpu().numpy() if want_xy else np.full((PAIRS, 2), np.nan)
    if not any(marginal):
        assert (rc == -1).all() and np.isnan(xy).all()
        return
    r_ref, y_ref = orc.search(marg, u2[0::2])
    assert np.array_equal(rc[:, 0], r_ref)
    if want_xy:
        assert_samples(rc[:, 0], xy[:, 0], r_ref, y_ref)
    for r in (0, 1, 2):
        sel = r_ref == r
        if r == 1:
            assert (rc[sel, 1] == -1).all() and np.isnan(xy[sel, 1]).all()
        elif sel.any():
            c_ref, x_ref = orc.search(rows[r], u2[1::2][sel])
            assert np.array_equal(rc[sel, 1], c_ref)
            if want_xy:
                assert_samples(rc[sel, 1], xy[sel, 1], c_ref, x_ref)
