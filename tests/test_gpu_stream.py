"""The streaming candidate pass at the edges of its blocks: rows of each
operand length it takes (128, 256, 384 and 512 bytes), relations one row
around its 16-row blocks, strips, stages and row blocks, few rows against
many (waves along S), both join forms.  Pairs equal the oracle's exactly."""
import numpy as np
import pytest

from paper_1812_07607_amd import synth

pytestmark = pytest.mark.gpu

# values per operand row: one K-chunk to four, whole and with a padded tail
DIMS = {"bf16": [33, 64, 128, 190, 256], "fp16": [64, 100, 192, 250], "fp8": [100, 256, 300, 512]}
SIZES = [(1, 1), (15, 300), (129, 31), (255, 257), (1025, 513), (40, 9001), (2100, 1023)]


def near_eps(orc, R, S, self_join):
    """A radius exactly at a pair's distance (the boundary pair is in)."""
    n = R.shape[0] * S.shape[0]
    rng = np.random.default_rng(7)
    t = rng.integers(0, n, size=min(n, 4000))
    d2 = np.sort(orc.pair_d2(R, S, t // S.shape[0], t % S.shape[0]))
    return float(np.sqrt(d2[min(len(d2) - 1, len(d2) // 50 + (1 if self_join else 0))]))


@pytest.mark.parametrize("prec,d", [(p, d) for p in DIMS for d in DIMS[p]])
def test_stream_edges(orc, prec, d):
    from gpu_util import assert_eps_equal, dev
    from paper_1812_07607_amd import ops
    for nr, ns in SIZES:
        R = synth.gaussian_mixture_unit(nr, d, 5, 0.05, seed=d, stream=0)
        S = synth.gaussian_mixture_unit(ns, d, 5, 0.05, seed=d, stream=1)
        eps = near_eps(orc, R, S, False)
        assert_eps_equal(ops.join_eps(dev(R), dev(S), eps, prec), orc.eps_join(R, S, eps), d, "%s %dx%d" % (prec, nr, ns))
        eps = near_eps(orc, S, S, True)
        assert_eps_equal(ops.join_eps(dev(S), None, eps, prec), orc.eps_join(S, None, eps), d, "%s self %d" % (prec, ns))


@pytest.mark.parametrize("prec", ["bf16", "fp16", "fp8"])
def test_stream_every_pair(orc, prec):
    """eps = inf: every output of every block is a candidate (the queue's
    flush in the middle of a block)."""
    from gpu_util import assert_eps_equal, dev
    from paper_1812_07607_amd import ops
    R = synth.uniform_rows(300, 128, seed=3, stream=0)
    S = synth.uniform_rows(517, 128, seed=3, stream=1)
    assert_eps_equal(ops.join_eps(dev(R), dev(S), float("inf"), prec), orc.eps_join(R, S, float("inf")), 128, prec)
    assert_eps_equal(ops.join_eps(dev(S), None, float("inf"), prec), orc.eps_join(S, None, float("inf")), 128, prec)


@pytest.mark.parametrize("prec,d", [("bf16", 64), ("bf16", 128), ("fp16", 100), ("fp16", 256), ("fp8", 256), ("fp8", 500)])
def test_stream_topk_edges(orc, prec, d):
    """Row blocks, strips and stages of the top-k band, the group maxima's
    runs, S that fits a row's buffer whole, k from one to nearly all of S."""
    from gpu_util import assert_topk_equal, dev
    from paper_1812_07607_amd import ops
    for nr, ns, k in [(1, 40, 5), (130, 511, 3), (257, 513, 32), (40, 9001, 10), (1025, 2100, 1), (70, 4500, 256)]:
        R = synth.gaussian_mixture_unit(nr, d, 5, 0.05, seed=d, stream=0)
        S = synth.gaussian_mixture_unit(ns, d, 5, 0.05, seed=d, stream=1)
        j, _, dist = orc.topk(R, S, k)
        assert_topk_equal(ops.join_topk(dev(R), dev(S), k, prec=prec), j, dist, d, "%s %dx%d k=%d" % (prec, nr, ns, k))
    j, _, dist = orc.topk(S, None, 7, exclude_self=True)
    got = ops.join_topk(dev(S), None, 7, exclude_self=True, prec=prec)
    assert_topk_equal(got, j, dist, d, "%s self" % prec)


def test_stream_topk_sample_misses_the_neighbours(orc):
    """Every near row of S lies in stages the group maxima skip, and there are
    more of them than a row's buffer holds: the rows' bounds are loose, the
    buffers overflow, and the call still returns the oracle's rows."""
    from gpu_util import assert_topk_equal, dev, host
    from paper_1812_07607_amd import ops
    rng = np.random.default_rng(5)
    ns, d, k = 45000, 64, 10
    S = synth.uniform_rows(ns, d, lo=2.0, hi=3.0, seed=1)
    near = np.nonzero((np.arange(ns) // 256) % 2 == 1)[0]
    near = rng.choice(near, size=4000, replace=False)
    S[near] = synth.uniform_rows(4000, d, lo=-0.01, hi=0.01, seed=2)
    R = synth.uniform_rows(70000, d, lo=-0.01, hi=0.01, seed=3)
    got = ops.join_topk(dev(R), dev(S), k, prec="bf16")
    rows = rng.choice(len(R), size=60, replace=False)
    j, _, dist = orc.topk(R[rows], S, k)
    got.j, got.dist = got.j[rows.tolist()], got.dist[rows.tolist()]
    assert_topk_equal(got, j, dist, d, "sampled rows")
