"""Top-k thresholds from the sampled maxima: rows few enough for eight keys a
lane and too many for it, strides of few and of many rows, and neighbours that
lie together where the sample skips."""
import numpy as np
import pytest

from paper_1812_07607_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,ns,k", [(8192, 2100, 10), (8193, 2100, 10), (8300, 3000, 60), (1023, 40000, 1),
                                     (1024, 40000, 1), (1100, 13000, 10), (600, 33000, 120), (2200, 5000, 256)])
def test_rows_and_strides(orc, nr, ns, k):
    from gpu_util import assert_topk_equal, dev
    from paper_1812_07607_amd import ops
    d = 48
    R = synth.gaussian_mixture_unit(nr, d, 20, 0.05, seed=d, stream=0)
    S = synth.gaussian_mixture_unit(ns, d, 20, 0.05, seed=d, stream=1)
    S = S[np.argsort(S[:, 0], kind="stable")]  # near rows together
    j, _, dist = orc.topk(R, S, k)
    assert_topk_equal(ops.join_topk(dev(R), dev(S), k, prec="bf16"), j, dist, d, "%dx%d k=%d" % (nr, ns, k))
