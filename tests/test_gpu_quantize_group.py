"""Quantisation in one launch: block- and wave-owned distributions at the
edges of a wave's and a block's registers, on either side of the rule, with
weights that are refused, against the oracle bit for bit."""
import numpy as np
import pytest

from gpu_util import note, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rtf():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1901_05423_amd as rtf
    rtf.lib()
    return rtf


def weights(rng, n):
    v = np.exp(rng.uniform(-60, 60, n)).astype(np.float32)
    v[rng.random(n) < 0.1] = 0
    if n > 3:
        v[1] = -0.0
    return v


SIZES = [
    (1,), (64,), (1024,), (16384,), (16385,),  # one distribution: registers, then the even cut
    (1024, 1025, 1, 7), (16384, 16385, 3), (40000, 2, 2),  # a block each
    (1,) * 17 + (1024, 1025) + (3,) * 40,  # a wave each, two blocks, one distribution the block's
    (5,) * 600 + (20000,),
    (131071, 1), (131072, 1),  # the totals of the rule
]


@pytest.mark.parametrize("sizes", SIZES, ids=lambda s: f"{len(s)}x{max(s)}")
def test_quantize_group(rtf, orc, sizes):
    note(f"quantize group D={len(sizes)} max={max(sizes)}")
    rng = np.random.default_rng(sum(sizes))
    vs = [weights(rng, n) for n in sizes]
    eo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    v = np.concatenate(vs)
    status = to_dev(np.zeros(1, np.int32))
    q, s = rtf.quantize(to_dev(v), to_dev(eo) if len(sizes) > 1 else None, status=status)
    q, s = q.cpu().numpy(), s.cpu().numpy()
    assert int(status.item()) == 0
    for d, vd in enumerate(vs):
        q_ref, s_ref = orc.quantize(vd)
        assert np.array_equal(q[eo[d]:eo[d + 1]], q_ref), d
        assert s[d] == s_ref[0], d


@pytest.mark.parametrize("bad", [-1.0, np.nan, np.inf])
@pytest.mark.parametrize("sizes", [(300,), (20, 2000, 30), (5,) * 40])
def test_quantize_group_refuses(rtf, sizes, bad):
    note(f"quantize group refuses {bad} sizes={len(sizes)}")
    v = np.ones(sum(sizes), np.float32)
    v[-2] = bad
    eo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    status = to_dev(np.zeros(1, np.int32))
    rtf.quantize(to_dev(v), to_dev(eo) if len(sizes) > 1 else None, status=status)
    assert int(status.item()) == 1 << rtf.RTF_ERR_VALUE


@pytest.mark.parametrize("sizes", [(20, 2000, 30), (40000, 2, 50), (5,) * 1100])
def test_quantize_group_outer_offsets(rtf, orc, sizes):
    """offsets that do not reach 0 and n (the build refuses them): the first
    and the last distribution take the elements left over"""
    note(f"quantize group outer offsets D={len(sizes)}")
    v = weights(np.random.default_rng(len(sizes)), sum(sizes))
    eo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    short = eo.copy()
    short[0], short[-1] = 3, eo[-1] - 2
    q_ref, s_ref = orc.quantize(v, eo)
    q, s = rtf.quantize(to_dev(v), to_dev(short))
    assert np.array_equal(q.cpu().numpy(), q_ref) and np.array_equal(s.cpu().numpy(), s_ref)
