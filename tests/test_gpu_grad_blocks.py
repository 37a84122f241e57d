"""The adjoint's scatter blocks at the edges of their forms: several
distributions whose elements just fit or just miss the LDS bins, more
distributions than bins, odd sample counts (half a lane pair), and chunks
that end inside a step."""
import numpy as np
import pytest

from test_gpu_batched import raw_grad, rtf  # noqa: F401 (fixture)

from gpu_util import note

pytestmark = pytest.mark.gpu


def weights(rng, n):
    v = (0.01 + rng.random(n)).astype(np.float32)
    if n > 10:
        v[rng.integers(0, n, n // 10)] = 0
    if not v.any():
        v[0] = 1
    return v


@pytest.mark.parametrize("last", [1091, 1092, 1093])  # bins: elements and 4 distributions, 4096 in all
@pytest.mark.parametrize("counts", [(301, 0, 299, 1), (1, 700, 5000, 333)])
def test_grad_bins_edge(rtf, orc, last, counts):  # noqa: F811
    note(f"grad bins edge last={last} counts={counts}")
    rng = np.random.default_rng(last)
    raw_grad(rtf, orc, [weights(rng, n) for n in (1000, 1000, 1000, last)], counts, last)


@pytest.mark.parametrize("D,top", [(3000, 4), (5000, 2)])
def test_grad_many_distributions(rtf, orc, D, top):  # noqa: F811
    """One block over thousands of distributions: elements beyond the bins,
    and distributions beyond them too."""
    note(f"grad many D={D}")
    rng = np.random.default_rng(D)
    counts = np.where(rng.random(D) < 0.2, rng.integers(1, 4, D), 0)
    counts[[0, -1]] = 1
    raw_grad(rtf, orc, [weights(rng, int(n)) for n in rng.integers(1, top + 1, D)], counts, D)


@pytest.mark.parametrize("n", [4096, 4097])
@pytest.mark.parametrize("S", [1, 2047, 2049, 70001])
def test_grad_odd_counts(rtf, orc, n, S):  # noqa: F811
    note(f"grad odd n={n} S={S}")
    raw_grad(rtf, orc, [weights(np.random.default_rng(n + S), n)], [S], S)
