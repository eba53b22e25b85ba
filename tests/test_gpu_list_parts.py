"""The streaming eps pass's candidate list, counted in eight parts: lists that
hold the candidates exactly, so that parts fill up and flushes go on in the
next one, few rows (one counter), and lists that are too small."""
import pytest
import torch

from paper_1812_07607_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,ns", [(280, 700), (300, 517), (1100, 900), (5000, 300)])
@pytest.mark.parametrize("prec", ["bf16", "fp8"])
def test_full_lists(orc, nr, ns, prec):
    from gpu_util import assert_eps_equal, dev
    from paper_1812_07607_amd import ops
    R = synth.uniform_rows(nr, 40, seed=3, stream=0)
    S = synth.uniform_rows(ns, 40, seed=3, stream=1)
    S[ns // 2:] += 8.0  # half of S is far: which workgroups find candidates is uneven
    eps = 4.0
    ref = orc.eps_join(R, S, eps)
    free = ops.join_eps(dev(R), dev(S), eps, prec)
    assert_eps_equal(free, ref, 40, "free")
    for room in (free.candidates, free.candidates + 1, 2 * free.candidates, free.candidates // 3, 1):
        got = ops.join_eps(dev(R), dev(S), eps, prec, max_candidates=room, workspace=ops.Workspace(dev(R).device))
        assert got.candidates == free.candidates
        assert_eps_equal(got, ref, 40, "room %d" % room)
