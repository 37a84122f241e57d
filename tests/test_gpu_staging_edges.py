"""Batched sampling on either side of the rules that choose its kernel: one
distribution staged in LDS or not, the segment length, and the chunks."""
import numpy as np
import pytest

from gpu_util import assert_samples, note, random_weights, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rtf():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1901_05423_amd as rtf
    rtf.lib()
    return rtf


def offsets(c):
    return np.concatenate([[0], np.cumsum(c)]).astype(np.int64)


def check(rtf, orc, ws, cells, counts, seed, collapsed=False):
    f = rtf.build_batched(to_dev(np.concatenate(ws)), to_dev(offsets([w.size for w in ws])), to_dev(offsets(cells)))
    if collapsed:
        f.widen()
    so = offsets(counts)
    u = np.random.default_rng(seed).integers(0, 2 ** 64, int(so[-1]), dtype=np.uint64)
    u[-1] = 2 ** 64 - 1
    u[0] = 0
    idx, x = rtf.sample_batched(f, to_dev(so), to_dev(u))
    only, _ = rtf.sample_batched(f, to_dev(so), to_dev(u), want_x=False)
    assert bool((only == idx).all())
    idx, x = idx.cpu().numpy(), x.cpu().numpy()
    for d, w in enumerate(ws):
        a, b = so[d], so[d + 1]
        if a < b:
            i_ref, x_ref = orc.search(w, u[a:b])
            assert_samples(idx[a:b], x[a:b], i_ref, x_ref)


@pytest.mark.parametrize("collapsed", [False, True])
@pytest.mark.parametrize("n,m", [(16, 4), (3000, 1000), (5000, 1024), (5000, 1025)])
@pytest.mark.parametrize("S", [(1 << 21) - 1, 1 << 21, (1 << 22) + 3])
def test_one_distribution(rtf, orc, n, m, S, collapsed):
    note(f"staging edges one n={n} m={m} S={S} collapsed={collapsed}")
    w = random_weights(np.random.default_rng(n + m), n, zero_frac=0.1, skew=True)
    check(rtf, orc, [w], [m], [S], S, collapsed)


@pytest.mark.parametrize("extra", [-1, 0])
@pytest.mark.parametrize("D", [2, 300])
def test_segments(rtf, orc, D, extra):
    """4096 samples a distribution, one of them beyond the LDS table"""
    note(f"staging edges D={D} extra={extra}")
    rng = np.random.default_rng(D)
    ws = [random_weights(rng, int(n), zero_frac=0.1, skew=True) for n in rng.integers(1, 200, D)]
    ws[D // 2] = random_weights(rng, 4000, zero_frac=0.1, skew=True)
    cells = [max(1, w.size // 2) for w in ws]
    if D == 2:
        cells[1] = 1025
    check(rtf, orc, ws, cells, [4096] * (D - 1) + [4096 + extra], D)


@pytest.mark.parametrize("total", [(1 << 21) - 1, 1 << 21])
@pytest.mark.parametrize("D", [2, 3000])
def test_chunks(rtf, orc, D, total):
    note(f"chunk edges D={D} total={total}")
    rng = np.random.default_rng(D + 1)
    ws = [random_weights(rng, int(n), zero_frac=0.1, skew=True) for n in rng.integers(1, 100, D)]
    cells = [4 * w.size if D == 3000 else 3000 for w in ws]  # short segments, or too many cells to stage
    counts = rng.multinomial(total, np.full(D, 1.0 / D))
    check(rtf, orc, ws, cells, counts, D)
