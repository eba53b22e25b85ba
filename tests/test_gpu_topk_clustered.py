"""Top-k against an S whose near rows lie together (frames of one scene, rows
in order of their cluster): the sample that bounds each row's band reaches
them whatever their order, so the streaming pass suffices as often as for the
same rows shuffled, and the rows equal the oracle's."""
import numpy as np
import pytest

from paper_1812_07607_amd import ops, synth

pytestmark = pytest.mark.gpu


def mixture(rng, mu, c):
    x = mu[c] + 0.05 * rng.standard_normal((len(c), mu.shape[1]), dtype=np.float32)
    return x / np.linalg.norm(x, axis=1, keepdims=True)


def passes(f):
    """f's result and the candidate passes it ran"""
    c = ops.context()
    c.set_timing(True)
    c.timing(reset=True)
    r = f()
    n = c.timing(reset=True)["contract"][1]
    c.set_timing(False)
    return r, n


@pytest.mark.parametrize("prec,nr,ns,d,k,centres", [("bf16", 131072, 300000, 64, 10, 100), ("fp16", 200000, 120000, 128, 10, 60),
                                                    ("fp16", 140000, 100000, 128, 50, 25)])
def test_rows_in_order_of_their_cluster(orc, prec, nr, ns, d, k, centres):
    from gpu_util import assert_topk_equal, dev
    rng = np.random.default_rng(centres)
    mu = rng.standard_normal((centres, d)).astype(np.float32)
    mu /= np.linalg.norm(mu, axis=1, keepdims=True)
    R = mixture(rng, mu, rng.integers(centres, size=nr))
    S = mixture(rng, mu, np.arange(ns) * centres // ns)
    Rd = dev(R)
    _, shuffled = passes(lambda: ops.join_topk(Rd, dev(S[rng.permutation(ns)]), k, prec=prec))
    got, ordered = passes(lambda: ops.join_topk(Rd, dev(S), k, prec=prec))
    assert ordered == shuffled
    rows = rng.choice(nr, size=40, replace=False)
    j, _, dist = orc.topk(np.ascontiguousarray(R[rows]), S, k)
    sub = ops.TopkResult(got.j[dev(rows)], got.dist[dev(rows)], 0, 0)
    assert_topk_equal(sub, j, dist, d, "%s rows in order" % prec)


@pytest.mark.parametrize("prec,d", [("bf16", 64), ("fp16", 128), ("fp8", 300), ("bf16", 256)])
def test_sample_sizes(orc, prec, d):
    """S around whole octets, strips and slots of the sample, its strides one
    and more, k from one to the most: rows equal the oracle's."""
    from gpu_util import assert_topk_equal, dev
    for nr, ns, k in [(3, 513, 1), (20, 519, 32), (33, 1031, 16), (65, 4111, 256), (17, 12007, 1), (1030, 13001, 10),
                      (40, 40009, 10)]:
        R = synth.gaussian_mixture_unit(nr, d, 5, 0.05, seed=d, stream=0)
        S = synth.gaussian_mixture_unit(ns, d, 5, 0.05, seed=d, stream=1)
        S = S[np.argsort(S[:, 0])]
        j, _, dist = orc.topk(R, S, k)
        assert_topk_equal(ops.join_topk(dev(R), dev(S), k, prec=prec), j, dist, d, "%s %dx%d k=%d" % (prec, nr, ns, k))
