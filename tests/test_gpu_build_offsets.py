"""The check of a batch's build offsets, which one block makes for all of
them: a single wrong offset anywhere among many is reported, at the ends of
its rounds too, and offsets that are right are not."""
import numpy as np
import pytest

from gpu_util import note, to_dev

pytestmark = pytest.mark.gpu

ROUND = 256  # threads of the block; it takes four rounds together


@pytest.fixture(scope="module")
def rtf():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1901_05423_amd as rtf
    rtf.lib()
    return rtf


@pytest.mark.parametrize("D", [2, 3, ROUND - 1, ROUND, 4 * ROUND - 1, 4 * ROUND, 5 * ROUND + 7])
@pytest.mark.parametrize("which", ["elements", "cells"])
def test_one_wrong_offset(rtf, D, which):
    note(f"build offsets D={D} {which}")
    n = 4 * D
    w = to_dev(np.full(n, 3, np.uint32))
    good = 4 * np.arange(D + 1, dtype=np.int64)
    at = sorted({0, 1, 2, D // 2, D - 1, D} | {q for q in (ROUND - 1, ROUND, ROUND + 1, 4 * ROUND, 4 * ROUND + 1) if q <= D})
    for q in [None, *at]:
        for wrong in ([None] if q is None else [good[q - 1] if 0 < q < D else good[q] + (1 if q == 0 else -1)]):
            off = good.copy()
            if q is not None:
                off[q] = wrong
            # (m_total is read back from the last cell offset: keep it where it counts the cells)
            eo, co = (off, good) if which == "elements" else (good, off)
            if which == "cells" and q == D:
                continue
            f = rtf.build_batched(w, to_dev(eo), to_dev(co))
            if q is None:
                f.check()
            else:
                with pytest.raises(rtf.RtfError) as e:
                    f.check()
                assert e.value.code == rtf.RTF_ERR_INVALID_ARG, q
