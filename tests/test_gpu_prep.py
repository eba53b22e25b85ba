"""The operand prep of a store's rows: copies and norms of rows of every
length class (eight or sixteen lanes a row, a wave), aligned or not, many rows
and few, against torch's own conversions; the statistics bound what the copy
leaves out."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
TILE = 256


def fields(store, n, qld):
    """The store's arrays, in the order the library lays them out."""
    mem, npad, at, out = store.mem, (n + TILE - 1) // TILE * TILE, 256, {}
    for name, dt, size in (("q", torch.uint8, qld), ("nrm2", torch.float64, 8), ("h", torch.float32, 4),
                           ("qnorm", torch.float32, 4), ("rho", torch.float32, 4), ("dh", torch.float32, 4),
                           ("xnorm", torch.float32, 4)):
        out[name] = mem[at:at + npad * size].view(dt)[:npad * size // (1 if name == "q" else size)]
        at += (npad * size + 255) // 256 * 256
    return out


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16", "fp8"])
@pytest.mark.parametrize("n", [300, 33000])
def test_rows(prec, n):
    from paper_1812_07607_amd import ops
    size, chunk = {"fp32": (4, 32), "bf16": (2, 64), "fp16": (2, 64), "fp8": (1, 128)}[prec]
    for d, ld in [(1, 1), (3, 3), (33, 36), (64, 64), (65, 65), (100, 101), (128, 128), (256, 257), (257, 260),
                  (500, 500), (512, 512), (520, 520), (1024, 1024)]:
        g = torch.Generator(device="cuda").manual_seed(d)
        X = torch.randn(n, ld, device="cuda", generator=g)[:, :d]
        X[n // 2] = 0.0
        dpad = (d + chunk - 1) // chunk * chunk
        f = fields(ops.Store(X, prec), n, dpad * size)
        what = "%s n=%d d=%d" % (prec, n, d)
        x2 = X.double().pow(2).sum(1)
        nrm2 = f["nrm2"][:n]
        assert torch.all((nrm2 - x2).abs() <= 2.3e-16 * (d + 2) * x2), what  # gamma_d of a float64 sum
        assert torch.all(f["xnorm"][:n].double() >= x2.sqrt() * (1 - 1e-15)), what
        assert torch.all(f["xnorm"][:n].double() <= x2.sqrt() * (1 + 1e-6)), what
        q = f["q"].view(-1, dpad * size)
        assert not q[n:].any(), what
        if prec == "fp8":
            continue
        dt = {"fp32": torch.float32, "bf16": torch.bfloat16, "fp16": torch.float16}[prec]
        v = q[:n].contiguous().view(dt)
        want = X.to(dt)
        want = torch.where(want.abs() < torch.finfo(dt).tiny, torch.zeros_like(want), want)  # subnormals flush
        assert torch.equal(v[:, :d], want), what
        assert not v[:, d:].any(), what
        r2 = (X.double() - want.double()).pow(2).sum(1)
        assert torch.all(f["rho"][:n].double() >= r2.sqrt() * (1 - 1e-15)), what
        assert torch.all(f["rho"][:n].double() <= r2.sqrt() * (1 + 1e-6)), what


@pytest.mark.parametrize("n,d", [(33000, 64), (300, 100), (300, 600)])
def test_bad_values_are_counted_in_any_lane(n, d):
    from paper_1812_07607_amd import ops
    for row, col in ((0, 0), (n - 1, d - 1), (n // 3, d // 2)):
        X = torch.zeros(n, d, device="cuda")
        X[row, col] = float("inf")
        with pytest.raises(Exception, match="non-finite values in R \\(1\\)"):
            ops.Store(X, "bf16")
