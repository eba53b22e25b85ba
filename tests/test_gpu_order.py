"""The ordering of an eps-join's pairs: row counts and offsets at the edges of
the scan's chunks (one launch, two, three), calls that keep no pair or lose
candidates, bad input, a fresh output after each.  Pairs equal a direct
construction exactly."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 4094, 4095, 4096, 8191, 8192, 100001, 4096 * 4096 + 5])
def test_offsets_at_scan_chunks(n):
    from paper_1812_07607_amd import ops
    i = torch.arange(n, device="cuda")
    R = ((i * 7919) % 64).to(torch.float32).reshape(n, 1)
    S = torch.tensor([[0.0], [3.0], [3.25], [63.0]], device="cuda")
    out = ops.join_eps(R, S, 0.25, "bf16")
    v = R[:, 0]
    want = torch.cat([torch.stack([torch.nonzero(v == x)[:, 0], torch.full_like(torch.nonzero(v == x)[:, 0], j)], 1)
                      for j, x in ((0, 0.0), (1, 3.0), (2, 3.0), (3, 63.0))])
    want = want[torch.argsort(want[:, 0] * 4 + want[:, 1])]
    assert torch.equal(out.i.to(torch.int64), want[:, 0])
    assert torch.equal(out.j.to(torch.int64), want[:, 1])
    assert torch.equal(out.dist, torch.where(out.j == 2, 0.25, 0.0).to(torch.float32))


def test_calls_without_pairs_between_others():
    """No pairs, non-finite input, too few candidates at first: each call
    leaves the next one's result alone."""
    from paper_1812_07607_amd import ops
    R = torch.arange(300, device="cuda", dtype=torch.float32).reshape(-1, 1).repeat(1, 3)
    bad = R.clone()
    bad[17, 1] = float("nan")
    for prec in ("bf16", "fp32"):
        for _ in range(3):
            assert len(ops.join_eps(R, R + 0.5, 0.25, prec).i) == 0
            with pytest.raises(Exception):
                ops.join_eps(bad, R, 0.25, prec)
            out = ops.join_eps(R, R, 0.0, prec)
            assert torch.equal(out.i.to(torch.int64), torch.arange(300, device="cuda"))
            assert torch.equal(out.j, out.i)
            out = ops.join_eps(R, None, float("inf"), prec)
            iu = np.triu_indices(300, 1)
            assert np.array_equal(out.i.cpu().numpy(), iu[0]) and np.array_equal(out.j.cpu().numpy(), iu[1])


@pytest.mark.parametrize("n", [40, 17000])
def test_row_lengths(n):
    """Rows of every ordering path at its edges: a few lanes, a wave, LDS
    ranks, buckets (in LDS and in memory), windows, and pairs bunched so that
    a bucket would hold too many; rows few (a wave each) and many."""
    from paper_1812_07607_amd import ops
    lens = [0, 1, 7, 8, 9, 63, 64, 65, 255, 256, 257, 1000, 1024, 1025, 9000, 700, 40000]
    ns = 300000
    rng = np.random.default_rng(n)
    cls = np.full(ns, 999, np.int64)
    cls[5000:5000 + lens[15] - 2] = 15  # bunched, with two far away
    free = rng.permutation(np.flatnonzero(cls == 999))
    cls[free[:2]] = 15
    free = free[2:]
    for c, m in enumerate(lens):
        if c != 15:
            cls[free[:m]] = c
            free = free[m:]
    own = np.full(n, 500, np.int64)  # no partner
    own[rng.permutation(n)[:2 * len(lens)]] = np.tile(np.arange(len(lens)), 2)
    R = torch.tensor(own, device="cuda").to(torch.float32).reshape(-1, 1)
    S = torch.tensor(cls, device="cuda").to(torch.float32).reshape(-1, 1)
    out = ops.join_eps(R, S, 0.25, "bf16")
    members = [np.flatnonzero(cls == c) for c in range(len(lens))]
    want_i = np.concatenate([np.full(len(members[c]), i) for i, c in enumerate(own) if c < len(lens)])
    want_j = np.concatenate([members[c] for c in own if c < len(lens)])
    assert np.array_equal(out.i.cpu().numpy(), want_i) and np.array_equal(out.j.cpu().numpy(), want_j)
    assert not out.dist.any()
