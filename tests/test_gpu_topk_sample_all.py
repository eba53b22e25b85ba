"""Streaming top-k whose sample is every row of S (S short for its k): R goes
whole up to four times k of room and in blocks beyond, and the rows equal the
oracle's either way."""
import numpy as np
import pytest

from paper_1812_07607_amd import ops, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,k,ordered,whole", [("bf16", 127, False, True), ("bf16", 128, True, True), ("fp16", 129, True, False),
                                                  ("bf16", 250, False, False)])
def test_room_of_a_whole_sample(orc, prec, k, ordered, whole):
    from gpu_util import assert_topk_equal, dev
    n = 65536  # one split: buffers of 1,024 entries
    R = synth.gaussian_mixture_unit(n, 64, 12, 0.05, seed=k, stream=0)
    S = synth.gaussian_mixture_unit(4100, 64, 12, 0.05, seed=k, stream=1)
    if ordered:
        S = S[np.argsort(S @ S[0])]
    c = ops.context()
    c.set_timing(True)
    c.timing(reset=True)
    got = ops.join_topk(dev(R), dev(S), k, prec=prec)
    passes = c.timing(reset=True)["contract"][1]
    c.set_timing(False)
    assert (passes == 1) == whole
    rows = np.arange(0, n, 1021)
    j, _, dist = orc.topk(np.ascontiguousarray(R[rows]), S, k)
    assert_topk_equal(ops.TopkResult(got.j[dev(rows)], got.dist[dev(rows)], 0, 0), j, dist, 64, "%s k=%d" % (prec, k))
