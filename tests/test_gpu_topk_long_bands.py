"""Top-k of rows whose bands hold more entries than the selection's list: they
are selected over memory, with the band refined by the distances of the
entries of largest P~.  S lies in shells about each query, thinner than the
candidates' margin, so that nearly all of it is in every band; rows equal the
oracle's, also where the selection runs again for rows with more contenders
than it holds (copies of one row)."""
import numpy as np
import pytest

from paper_1812_07607_amd import ops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,d,thick", [("bf16", 64, 1e-3), ("fp16", 128, 1e-4), ("fp8", 128, 2e-2), ("fp8", 200, 1e-2)])
@pytest.mark.parametrize("k,copies", [(1, 0), (10, 0), (100, 0), (256, 0), (10, 300), (200, 700)])
def test_shells(orc, prec, d, thick, k, copies):
    from gpu_util import assert_topk_equal, dev
    rng = np.random.default_rng(d + k)
    n = 4099

    def unit(m):
        u = rng.standard_normal((m, d))
        return u / np.linalg.norm(u, axis=1, keepdims=True)

    q = unit(1)
    S = (q + unit(n) * rng.uniform(0.9, 0.9 + thick, size=(n, 1))).astype(np.float32)
    R = (q + 1e-5 * unit(9)).astype(np.float32)
    if copies:
        S[rng.choice(n, size=copies, replace=False)] = (q + 0.9 * unit(1)).astype(np.float32)
    got = ops.join_topk(dev(R), dev(S), k, prec=prec)
    assert got.band_entries > 1024 * len(R)
    j, _, dist = orc.topk(R, S, k)
    assert_topk_equal(got, j, dist, d, "%s k=%d copies=%d" % (prec, k, copies))
