"""Chaining where the block-wise scan can go wrong: sets around the edges of
64-anchor blocks, of four wavefronts per set and of the LDS limits, ties
between candidates on either side of a block, scans that end inside a set
because of the genome distance, and chains of negative score; checked as the
other chaining tests check (fp64 scores within 1e-9, chains exactly)."""
import numpy as np
import pytest

from paper_2210_08052_amd import mpg
from tests.test_gpu_parity import _check_chaining

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    with mpg.Context(0) as c:
        yield c


def _sorted(a):
    a = np.asarray(a, np.int64).reshape(-1, 2)
    return a[np.lexsort((a[:, 1], a[:, 0]))].astype(np.int32)


def _set(rng, n, spread, residues, binned):
    """Half on a few diagonals (chains), half anywhere."""
    h = n // 2
    y = rng.integers(0, residues, h)
    x = 3 * y + rng.choice([0, 0, 0, 400, 90000], h)
    noise = np.stack([rng.integers(0, spread, n - h), rng.integers(0, residues, n - h)], axis=1)
    a = np.concatenate([np.stack([x, y], axis=1), noise])
    if binned:
        a[:, 0] //= 256
    return _sorted(a)


@pytest.mark.parametrize("binned", [True, False])
@pytest.mark.parametrize("sizes", [(1, 2, 63, 64, 65, 127, 128, 129, 192, 511),
                                   (512, 513, 640, 1, 64, 65), (3006, 3007, 3008, 70),
                                   (7015, 7025, 100)])
def test_sizes(ctx, sizes, binned):
    rng = np.random.default_rng(sum(sizes) + binned)
    sets = [_set(rng, n, 2_000_000, 900, binned) for n in sizes]
    for kw in (dict(), dict(k=3, beta=2.5, G=5000, max_chains=7), dict(beta=0.0, G=100)):
        print("case sizes=%s binned=%d %s" % (sizes, binned, kw), flush=True)
        cp = mpg.chaining_params(binned=int(binned), **kw)
        for a, r in zip(sets, ctx.chain_anchors(sets, cp)):
            assert r["status"] == 0
            _check_chaining(r, a, cp.k, cp.beta, cp.G, binned, cp.max_chains)


@pytest.mark.parametrize("binned", [True, False])
def test_ties_and_negative_scores(ctx, binned):
    """Many candidates of one value (equal anchors, one diagonal, a grid), and
    links whose penalty exceeds what the anchor adds."""
    step = 1 if binned else 3
    sets = [_sorted([(7, 5)] * 150), _sorted([(7, y) for y in range(300)]),
            _sorted([(step * y, y) for y in range(200)] * 2),
            _sorted([(step * (y // 2), y % 40) for y in range(400)]),
            _sorted([(3000 * q, 10 * q) for q in range(200)]),
            _sorted([(q, 2000 - 9 * q) for q in range(200)])]
    for kw in (dict(), dict(k=1, beta=0.3, max_chains=500), dict(k=40, beta=5.0)):
        print("case ties binned=%d %s" % (binned, kw), flush=True)
        cp = mpg.chaining_params(binned=int(binned), **kw)
        for a, r in zip(sets, ctx.chain_anchors(sets, cp)):
            assert r["status"] == 0
            _check_chaining(r, a, cp.k, cp.beta, cp.G, binned, cp.max_chains)
