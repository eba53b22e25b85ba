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
