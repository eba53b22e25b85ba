"""The buffers of the streaming top-k: rows of R go in blocks where one
buffer per row would be too small, and rows of S that no sample tells of fill
a buffer all the same, after which the tile form answers.  Rows equal the
oracle's; the candidate passes say which way a call went."""
import numpy as np
import pytest

from paper_1812_07607_amd import ops, synth

pytestmark = pytest.mark.gpu


def passes(f):
    """f's result and the candidate passes it ran"""
    c = ops.context()
    c.set_timing(True)
    c.timing(reset=True)
    r = f()
    n = c.timing(reset=True)["contract"][1]
    c.set_timing(False)
    return r, n


def check_rows(orc, got, R, S, k, rows, what):
    """the given rows against the oracle; S None: R's own rows, the row itself left out"""
    from gpu_util import assert_topk_equal, dev
    if S is None:
        j, _, dist = orc.topk(np.ascontiguousarray(R[rows]), R, k + 1)
        at = np.array([np.append(np.nonzero(a != i)[0], k)[:k] for a, i in zip(j, rows)])  # (k + 1 entries, less the row's own)
        j, dist = np.take_along_axis(j, at, 1), np.take_along_axis(dist, at, 1)
    else:
        j, _, dist = orc.topk(np.ascontiguousarray(R[rows]), S, k)
    sub = ops.TopkResult(got.j[dev(rows)], got.dist[dev(rows)], 0, 0)
    assert_topk_equal(sub, j, dist, R.shape[1], what)


@pytest.mark.parametrize("prec,k,exclude", [("bf16", 32, False), ("fp16", 50, True), ("fp8", 32, False), ("fp8", 20, True),
                                            ("bf16", 200, False)])
def test_rows_in_blocks(orc, prec, k, exclude):
    """65,536 rows of R: one split, a buffer of 1,024 entries if R went whole."""
    from gpu_util import dev
    rng = np.random.default_rng(k)
    n = 65536
    R = synth.gaussian_mixture_unit(n, 64, 40, 0.05, seed=k, stream=0)
    if exclude:
        # more copies of one row than a selection in LDS holds, in every block
        R[rng.choice(n, size=700, replace=False)] = R[9]
        got, runs = passes(lambda: ops.join_topk(dev(R), None, k, exclude_self=True, prec=prec))
        S = None
    else:
        S = synth.gaussian_mixture_unit(200000, 64, 40, 0.05, seed=k, stream=1)
        got, runs = passes(lambda: ops.join_topk(dev(R), dev(S), k, prec=prec))
    assert runs > 1
    rows = np.unique(np.concatenate([[0, 9, n - 1], np.arange(1, 64) * 1024, np.arange(1, 64) * 1024 - 1]))
    check_rows(orc, got, R, S, k, rows, prec)


@pytest.mark.parametrize("prec", ["bf16", "fp8"])
def test_all_of_s_fits_a_block(orc, prec):
    """S shorter than the rows that need no threshold, a small explicit band
    capacity: no buffer overflows, the tile form is not asked."""
    from gpu_util import dev
    R = synth.gaussian_mixture_unit(65536, 48, 10, 0.05, seed=3, stream=0)
    S = synth.gaussian_mixture_unit(500, 48, 10, 0.05, seed=3, stream=1)
    got, runs = passes(lambda: ops.join_topk(dev(R), dev(S), 10, prec=prec, band_cap=320))
    c = ops.context()
    full, once = passes(lambda: ops.join_topk(dev(R), dev(S), 10, prec=prec, band_cap=512))
    assert (runs, once) == (2, 1)
    assert bool((got.j == full.j).all()) and bool((got.dist == full.dist).all())
    check_rows(orc, got, R, S, 10, np.arange(0, 65536, 1111), prec)


def sampled_octets(nS, k):
    """The octets (8 rows each) of S whose maxima bound a row (1,024 rows of R and more)."""
    few = many = 1
    while (few + 1) ** 2 * 100 * (k + 90) <= nS:
        few += 1
    while many < 8 and (many + 1) ** 2 * (240 * k + 600) <= nS:
        many += 1
    octets = nS // 8
    stride = max(few, many)
    strips = -(-octets // stride) // 4
    slots = max(64, -(-4 * k // 64) * 64) // 4
    strips -= min(strips % n for n in range(slots // 2, slots + 1))
    step = (octets << 32) // (4 * strips)
    return np.array([n * step >> 32 for n in range(4 * strips)])


@pytest.mark.parametrize("prec,d,exclude", [("bf16", 64, False), ("fp16", 128, True), ("fp8", 256, False), ("fp8", 100, True)])
def test_buffers_overflow(orc, prec, d, exclude):
    """12,000 rows of S nearer than all others, none of them sampled, against
    buffers of about 8,192: they overflow (candidate passes are counted), and the
    tile form, for E4M3 seeded by its bf16 pilot, gives the oracle's rows.  The
    near rows are at spread-out distances, so that its own buffers hold."""
    from gpu_util import dev
    rng = np.random.default_rng(d)
    n, k = 70000, 10

    def unit(x):
        return (x / np.linalg.norm(x, axis=1, keepdims=True)).astype(np.float32)

    a = unit(rng.standard_normal((1, d)))

    def near(m, lo, hi):  # unit rows at angles to a of cosine lo to hi
        u = rng.standard_normal((m, d))
        u -= (u @ a.T) * a
        cos = rng.uniform(lo, hi, size=(m, 1))
        return unit(cos * a + np.sqrt(1 - cos * cos) * unit(u))

    S = unit(rng.standard_normal((n, d)))
    free = np.ones(n // 8, bool)
    free[sampled_octets(n, k + exclude)] = False
    spots = np.nonzero(np.repeat(free, 8))[0]
    spots = rng.choice(spots, size=12000, replace=False)
    S[spots] = near(12000, 0.3, 0.98)
    if exclude:
        R = S
        call = lambda x: ops.join_topk(dev(x), None, k, exclude_self=True, prec=prec, band_cap=2048)
    else:
        R = near(n, 0.98, 1.0)
        call = lambda x: ops.join_topk(dev(R), dev(x), k, prec=prec, band_cap=2048)
    _, runs = passes(lambda: call(S[rng.permutation(n)]))  # the sample sees the near rows
    assert runs == 1
    got, runs = passes(lambda: call(S))
    if prec != "fp8":
        assert runs == 2
    else:  # the pilot's own passes, or another attempt with larger buffers where there is no pilot
        assert runs >= (2 if exclude else 3)
    rows = np.concatenate([rng.choice(n, size=30, replace=False), spots[:30]])
    check_rows(orc, got, R, None if exclude else S, k, np.unique(rows), prec)
