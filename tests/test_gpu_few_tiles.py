"""eps-joins either side of the sizes whose few tiles the tile form takes in
place of the streaming pass (three eighths of the CUs' number of tiles to as
many as CUs; self-joins five eighths; R at most four times as long as S): pairs
equal the oracle's, and a call that finds nothing finds nothing."""
import numpy as np
import pytest

from paper_1812_07607_amd import ops, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,d", [("bf16", 20), ("fp16", 100), ("fp8", 64)])
@pytest.mark.parametrize("nr,ns", [(2048, 3072), (2048, 3073), (4096, 4096), (4096, 4097), (5120, 1280), (5121, 1280),
                                   (1, 24576), (1, 24577), (3328, None), (3329, None), (4352, None), (4353, None)])
def test_either_side(orc, prec, d, nr, ns):
    from gpu_util import assert_eps_equal, dev
    R = synth.gaussian_mixture_unit(nr, d, 8, 0.05, seed=nr, stream=0)
    S = None if ns is None else synth.gaussian_mixture_unit(ns, d, 8, 0.05, seed=nr, stream=1)
    to = R if S is None else S
    i, j = np.arange(nr) if nr > 1 else np.zeros(len(to), int), np.arange(nr if nr > 1 else len(to)) * 7 % len(to)
    eps = float(np.sqrt(np.sort(orc.pair_d2(R, to, i[i != j], j[i != j]))[len(i) // 200]))
    for e in (1e-6, eps):
        got = ops.join_eps(dev(R), None if S is None else dev(S), e, prec)
        assert_eps_equal(got, orc.eps_join(R, S, e), d, "%s %s x %s eps %g" % (prec, nr, ns, e))
