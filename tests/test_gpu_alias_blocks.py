"""Alias tables built by one block per distribution: sizes at the edges of a
thread's run, of a round, of the LDS form and of the rule that chooses it,
against the oracle's serial construction, bit for bit."""
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


def weights(rng, n, kind):
    if kind == "equal":
        w = np.full(n, 2 ** 32 - 1, np.uint32)
    elif kind == "few":  # many masses of exactly W, many ties
        w = rng.integers(0, 3, n).astype(np.uint32)
    elif kind == "one":
        w = np.zeros(n, np.uint32)
        w[n // 2] = 7
    else:  # over the whole range of sizes
        w = np.floor(np.exp(rng.uniform(0, np.log(2.0 ** 32 - 1), n))).astype(np.uint32)
    if not w.any():
        w[-1] = 1
    return w


@pytest.mark.parametrize("kind", ["equal", "few", "one", "skew"])
@pytest.mark.parametrize("sizes", [(1,), (31,), (32,), (7, 8, 9, 511, 512, 513), (4095,), (4096, 4097),
                                   (1, 70000, 5), (33, 31), (32, 31)])
def test_alias_blocks(rtf, orc, sizes, kind):
    note(f"alias blocks sizes={sizes} kind={kind}")
    rng = np.random.default_rng(sum(sizes) + len(kind))
    ws = [weights(rng, n, kind) for n in sizes]
    eo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    t = rtf.alias_build(to_dev(np.concatenate(ws)), to_dev(eo) if len(sizes) > 1 else None)
    thr, alias, W = t.export()
    for d, w in enumerate(ws):
        ref = orc.alias_build(w)
        a, b = eo[d], eo[d + 1]
        assert int(W[d]) == ref.W, d
        assert np.array_equal(thr[a:b], ref.thr), d
        assert np.array_equal(alias[a:b], ref.alias), d
