"""The sampling kernels at the edges between them: records fetched by quads of
lanes or by single lanes (by the guide table's size), waves that are not full,
and batches on either side of the staging rule."""
import numpy as np
import pytest

from gpu_util import assert_samples, critical_u, note, random_weights, to_dev

pytestmark = pytest.mark.gpu

QUAD_CELLS = (12 << 20) // 64  # cells of the largest table fetched by quads


@pytest.fixture(scope="module")
def rtf():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1901_05423_amd as rtf
    rtf.lib()
    return rtf


@pytest.mark.parametrize("m", [1, 64, QUAD_CELLS - 1, QUAD_CELLS, QUAD_CELLS + 1])
@pytest.mark.parametrize("count", [1, 3, 63, 64, 65, 257, 0])
def test_record_fetch(rtf, orc, m, count):
    note(f"record fetch m={m} count={count}")
    rng = np.random.default_rng(m * 1000 + count)
    w = random_weights(rng, 3000, zero_frac=0.2, skew=True)
    w[:3] = 0  # several lower bounds of 0
    f = rtf.build(to_dev(w), m)
    f.check()
    key = f.node_view().cpu().numpy()[:, 0].view(np.uint64)
    u = critical_u(key, int(w.sum(dtype=np.uint64)), min(m, 2000))
    if count:
        u = rng.permutation(u)[:count]
        u[-1] = 2 ** 64 - 1
    idx, x = rtf.sample(f, to_dev(u))
    only, _ = rtf.sample(f, to_dev(u), want_x=False)
    i_ref, x_ref = orc.search(w, u)
    assert_samples(idx.cpu().numpy(), x.cpu().numpy(), i_ref, x_ref)
    assert np.array_equal(only.cpu().numpy(), i_ref)


@pytest.mark.parametrize("collapsed", [False, True])
@pytest.mark.parametrize("counts", [(4096, 4096, 4095), (4096, 4096, 4096), (0, 1, 12287), (8191, 0, 4097)])
def test_staging_rule(rtf, orc, counts, collapsed):
    note(f"staging rule counts={counts} collapsed={collapsed}")
    rng = np.random.default_rng(sum(counts) + collapsed)
    sizes, cells = [700, 4096, 31], [700, 1024, 31]
    ws = [random_weights(rng, n, zero_frac=0.1, skew=True) for n in sizes]
    off = lambda c: np.concatenate([[0], np.cumsum(c)]).astype(np.int64)  # noqa: E731
    f = rtf.build_batched(to_dev(np.concatenate(ws)), to_dev(off(sizes)), to_dev(off(cells)))
    if collapsed:
        f.widen()
    so = off(counts)
    u = rng.integers(0, 2 ** 64, int(so[-1]), dtype=np.uint64)
    u[-1] = 2 ** 64 - 1
    idx, x = rtf.sample_batched(f, to_dev(so), to_dev(u))
    idx, x = idx.cpu().numpy(), x.cpu().numpy()
    for d, w in enumerate(ws):
        a, b = so[d], so[d + 1]
        if a < b:
            i_ref, x_ref = orc.search(w, u[a:b])
            assert_samples(idx[a:b], x[a:b], i_ref, x_ref)
