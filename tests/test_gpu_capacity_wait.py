"""An eps-join that reports more pairs than the output holds returns with its
stream idle: the caller frees or reuses the workspace and the outputs at once
(the server hands them to another stream), so no ordering may still run."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1812_07607_amd import _lib, ops, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("indexed", [False, True])
def test_capacity_error_leaves_nothing_in_flight(orc, indexed):
    from gpu_util import dev, host
    # every pair of 3,000 x 4,000 rows: the ordering of 12M pairs takes longer
    # than the return to the test
    R = synth.uniform_rows(3000, 16, seed=1)
    S = synth.uniform_rows(4000, 16, seed=1, stream=1)
    eps, cap = 1e3, 1000
    c = ops.context()
    Rd, Sd = dev(R), dev(S)
    p = _lib.PREC["bf16"]
    out = [torch.full((cap,), -1, dtype=t, device="cuda") for t in (torch.int32, torch.int32, torch.float32)]
    pr = _lib.dl_pairs(*(t.data_ptr() for t in out), cap, 0, 0, 0)
    st = torch.cuda.Stream()
    need = (c.L.dl_join_eps_indexed_workspace(3000, 4000, 16, p, 0, 13_000_000, 0) if indexed
            else c.L.dl_join_eps_workspace(3000, 4000, 16, p, 0, 13_000_000))
    ws = torch.empty(int(need), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    args = [c.h, ops._mat(Rd), ops._mat(Sd), 0, eps, p]
    tail = [ctypes.c_void_p(ws.data_ptr()), ws.numel(), ctypes.byref(pr)]
    if indexed:
        rc = c.L.dl_join_eps_indexed(*args, 0, *tail, ctypes.byref(_lib.dl_index_info()), ctypes.c_void_p(st.cuda_stream))
    else:
        rc = c.L.dl_join_eps(*args, *tail, ctypes.c_void_p(st.cuda_stream))
    idle = st.query()
    assert rc == _lib.DL_ERR_CAPACITY and pr.count == 12_000_000
    assert idle
    # the first `capacity` pairs are there: row 0's columns in order
    assert np.array_equal(host(out[0]), np.zeros(cap, np.int32))
    assert np.array_equal(host(out[1]), np.arange(cap, dtype=np.int32))
