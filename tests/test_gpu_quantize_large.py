"""One-launch quantisation of batches with distributions too large for the
block or the wave that owns them: they are read and quantised slice by slice.
Sizes at the slices' edges, ranges that start at any alignment, two of them in
one slice, refused weights, and the cost of one large distribution."""
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


BLOCK, WAVE = 16384, 1024  # weights a block and a wave hold
SIZES = [
    (BLOCK + 1, 7), (7, BLOCK + 1), (BLOCK - 1, BLOCK + 1, BLOCK + 1), (3, 20000, 20001, 20002, 5),
    (2 * BLOCK, 2 * BLOCK + 1, 1), (1, 130000, 70), (100,) * 400 + (100003,) + (9,) * 300, (2,) * 600 + (250000,),
    # more than 1024 distributions
    (WAVE, WAVE + 1) * 40 + (1,) * 1100, (1,) * 1021 + (WAVE + 1,) * 120, (3,) * 1500 + (200001,) + (3,) * 500,
    (5,) * 1023 + (2 * WAVE, 3 * WAVE + 2), (2048, 1500, 1025) * 30 + (33,) * 1000,
]


def offsets(sizes):
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)


@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("sizes", SIZES, ids=lambda s: f"{len(s)}x{max(s)}")
def test_large_among_small(rtf, orc, sizes, shift):
    """shift: the weights start that many floats past a 16-byte boundary"""
    import torch
    note(f"quantize large D={len(sizes)} max={max(sizes)} shift={shift}")
    rng = np.random.default_rng(sum(sizes) + shift)
    n, eo = sum(sizes), offsets(sizes)
    v = np.exp(rng.uniform(-60, 60, n)).astype(np.float32)
    v[rng.random(n) < 0.1] = 0
    for d in np.flatnonzero(np.asarray(sizes) > WAVE)[::3]:  # the largest at an end
        v[eo[d] if d % 2 else eo[d + 1] - 1] = np.float32(3e38)
    room = torch.zeros(n + 4, dtype=torch.float32, device="cuda:0")
    vd = room[shift:shift + n]
    vd.copy_(to_dev(v))
    status = to_dev(np.zeros(1, np.int32))
    q, s = rtf.quantize(vd, to_dev(eo), status=status)
    q_ref, s_ref = orc.quantize(v, eo)
    assert int(status.item()) == 0
    assert np.array_equal(s.cpu().numpy(), s_ref)
    assert np.array_equal(q.cpu().numpy(), q_ref)


@pytest.mark.parametrize("sizes", [(5, 700), (3, 60000, 7), (2,) * 1100 + (120000, 900)], ids=lambda s: f"{len(s)}x{max(s)}")
def test_in_place(rtf, orc, sizes):
    """the quantised weights over the real ones"""
    import torch
    note(f"quantize in place D={len(sizes)} max={max(sizes)}")
    v = np.random.default_rng(sum(sizes)).random(sum(sizes), np.float32)
    eo = offsets(sizes)
    vd, scale = to_dev(v), torch.empty(len(sizes), dtype=torch.float64, device="cuda:0")
    q, s = rtf.quantize(vd, to_dev(eo), out=(vd.view(torch.uint32), scale))
    q_ref, s_ref = orc.quantize(v, eo)
    assert np.array_equal(s.cpu().numpy(), s_ref)
    assert np.array_equal(q.cpu().numpy(), q_ref)


@pytest.mark.parametrize("bad", [-1.0, np.nan, np.inf])
@pytest.mark.parametrize("sizes,at", [((40000, 9), 0), ((40000, 9), 39999), ((9, 40000), 17000),
                                      ((3,) * 1100 + (5000,), 3302), ((3,) * 1100 + (5000,), 8299)])
def test_large_refuses(rtf, sizes, at, bad):
    note(f"quantize large refuses {bad} at {at} of D={len(sizes)}")
    v = np.ones(sum(sizes), np.float32)
    v[at] = bad
    status = to_dev(np.zeros(1, np.int32))
    rtf.quantize(to_dev(v), to_dev(offsets(sizes)), status=status)
    assert int(status.item()) == 1 << rtf.RTF_ERR_VALUE


def test_one_large_costs_no_chain(rtf):
    """Seven small distributions and one of 130000 against eight equal ones,
    20 calls in a graph: 12.2 and 5.4 us a call (41 with the large one left to
    a single block)."""
    import torch
    note("quantize large: cost")

    def us(sizes):
        eo = to_dev(offsets(sizes))
        v = torch.rand(sum(sizes), device="cuda:0")
        out = rtf.quantize(v, eo)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(20):
                rtf.quantize(v, eo, out=out)
        times = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            g.replay()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 50)
        return sorted(times)[len(times) // 2]

    assert us([130000] + [100] * 7) < 4 * us([16337] * 8)
