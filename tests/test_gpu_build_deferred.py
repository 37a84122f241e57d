"""Builds whose tiles defer many node records to the fix-up (deep cell trees:
power densities, one weight over nearly all cells, sparse weights), in small
tiles: within what a tile always lists, within what it lists while no tile is
redone, and beyond, alone and mixed in one batch; with tile counts that do not
divide by the number of lists."""
import numpy as np
import pytest

from gpu_util import assert_forest, note, to_dev
from test_gpu_batched import check_batched
from test_gpu_parity import rtf  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def weights(rng, n, kind):
    if kind == "power":  # (i / n)^20: the first weights share few cells
        v = (np.arange(1, n + 1) / n) ** 20
        return np.maximum(np.rint(v * (2 ** 32 - 1)), 1).astype(np.uint32)
    if kind == "heavy":
        w = np.full(n, 4, np.uint32)
        w[n // 3] = 2 ** 32 - 1
        return w
    if kind == "sparse":
        w = np.where(rng.random(n) < 0.01, rng.integers(1, 2 ** 32, n), 0).astype(np.uint32)
        w[0] = 9
        return w
    return rng.integers(1, 2 ** 32, n, dtype=np.uint32)


BATCHES = {
    "power": [("power", 17475)] * 30,  # a few tiles with 33 to 128 deferred, none above
    "power of four": [("power", 32767)] * 4,
    "heavy": [("heavy", 30011)] * 7,
    "sparse": [("sparse", 4001)] * 9,  # nearly every tile above 128
    "mixed": [("power", 17475)] * 12 + [("sparse", 5000), ("heavy", 9999), ("plain", 700)] * 3,
    "one tile over": [("power", 17475)] * 6 + [("sparse", 600)] + [("plain", 3000)] * 4,
}


@pytest.mark.parametrize("name", BATCHES)
@pytest.mark.parametrize("ratio", [0.25, 1.0])
def test_batched(rtf, orc, name, ratio):  # noqa: F811
    note(f"deferred batch {name} ratio={ratio}")
    rng = np.random.default_rng(len(name))
    ws = [weights(rng, n, kind) for kind, n in BATCHES[name]]
    check_batched(rtf, orc, ws, [max(1, int(ratio * w.size)) for w in ws], [300] * len(ws), seed=3)


@pytest.mark.parametrize("kind", ["power", "heavy", "sparse"])
@pytest.mark.parametrize("n", [2049, 5 * 512 + 1, 131071, 1 << 20])
def test_single(rtf, orc, n, kind):  # noqa: F811
    note(f"deferred single n={n} {kind}")
    w = weights(np.random.default_rng(n), n, kind)
    f = rtf.build(to_dev(w), n // 4)
    f.check()
    assert_forest(f, orc.forest(w, m=n // 4), f"n={n} {kind}")
