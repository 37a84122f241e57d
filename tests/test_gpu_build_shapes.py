"""Builds at the edges of the shapes that small ones take: one distribution in
a single launch, 512-element tiles that work out their own prefix, and the
sizes from which the tile asked for is used; with covered cells at window and
tile edges, long runs and many deferred nodes."""
import numpy as np
import pytest

from gpu_util import assert_forest, note, random_weights, to_dev
from test_gpu_batched import check_batched
from test_gpu_parity import build_and_compare, rtf  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def weights(rng, n, kind):
    if kind == "heavy":  # one interval over nearly all cells
        w = np.ones(n, np.uint32)
        w[n // 3] = 2 ** 32 - 1
    elif kind == "zeros":  # long zero runs: nodes deferred, equal keys
        w = np.zeros(n, np.uint32)
        w[rng.integers(0, n, max(1, n // 100))] = rng.integers(1, 2 ** 32, max(1, n // 100))
        w[0] = 7
    else:
        w = random_weights(rng, n, zero_frac=0.1, skew=(kind == "skew"))
    return w


@pytest.mark.parametrize("kind", ["plain", "skew", "heavy", "zeros"])
@pytest.mark.parametrize("n,m", [(1, 1), (2, 4096), (512, 513), (513, 2049), (2047, 4096), (2048, 4096), (2048, 4097),
                                 (2049, 4096), (2049, 513), (5000, 64), (40000, 90000)])
def test_small_single(rtf, orc, n, m, kind):  # noqa: F811
    note(f"small single n={n} m={m} {kind}")
    build_and_compare(rtf, orc, weights(np.random.default_rng(n * 31 + m), n, kind), m, seed=n + m)


@pytest.mark.parametrize("n", [1 << 20, (1 << 20) + 1])
def test_single_rule(rtf, orc, n):  # noqa: F811
    note(f"single rule n={n}")
    w = weights(np.random.default_rng(n), n, "skew")
    f = rtf.build(to_dev(w), n // 4)
    f.check()
    assert_forest(f, orc.forest(w, m=n // 4), f"n={n}")


@pytest.mark.parametrize("extra", [0, 1])
@pytest.mark.parametrize("tile", [1024, 2048])
def test_batched_rule(rtf, orc, extra, tile):  # noqa: F811
    note(f"batched rule extra={extra} tile={tile}")
    rng = np.random.default_rng(77 + extra)
    sizes = [511, 1, 512, 513, 300000, 70, 1024]
    sizes.append((3 << 18) + extra - sum(sizes))
    ws = [weights(rng, n, k) for n, k in zip(sizes, ["plain", "plain", "heavy", "zeros", "skew", "heavy", "skew", "plain"])]
    cells = [max(1, n // 4) for n in sizes]
    cells[0], cells[2] = 3000, 5  # more cells than the window holds, long tails
    check_batched(rtf, orc, ws, cells, [200] * len(sizes), seed=5 + extra, tile=tile)


@pytest.mark.parametrize("D", [1, 3, 1100])
@pytest.mark.parametrize("tiles,over", [(2048, 0), (2048, 1), (4097, 5)])
def test_scan_blocks(rtf, orc, tiles, over, D):  # noqa: F811
    """tile sums scanned by one block, two and three, with an odd number of
    them and with the parameters in the same launch or the next"""
    note(f"scan blocks tiles={tiles} over={over} D={D}")
    rng = np.random.default_rng(tiles + over + D)
    n = tiles * 1024 + over
    if D == 1:
        f = rtf.build(to_dev(w := weights(rng, n, "skew")), n // 4, tile=1024)
        f.check()
        assert_forest(f, orc.forest(w, m=n // 4), f"n={n}")
        return
    sizes = [n // D] * (D - 1)
    sizes.append(n - sum(sizes))
    check_batched(rtf, orc, [weights(rng, k, "skew") for k in sizes], [max(1, k // 4) for k in sizes],
                  [50] * D, seed=tiles + D, tile=1024)


def test_all_zero_small(rtf):  # noqa: F811
    note("all zero small")
    for n in (1, 2048, 3000):
        f = rtf.build(to_dev(np.zeros(n, np.uint32)), 16)
        with pytest.raises(rtf.RtfError):
            f.check()
        idx, x = rtf.sample(f, to_dev(np.arange(100, dtype=np.uint64) << np.uint64(57)))
        assert (idx.cpu().numpy() == -1).all() and np.isnan(x.cpu().numpy()).all()
