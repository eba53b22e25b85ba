"""An eps-join without pairs: nothing is ordered, the stream is idle on return,
and what the call leaves in its workspace does not reach the next one; offsets
of rows either side of the chunks a workgroup adds up for itself."""
import numpy as np
import pytest
import torch

from paper_1812_07607_amd import ops, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["bf16", "fp8", "fp32"])
@pytest.mark.parametrize("nr", [1, 300, 4095, 4096, 16382, 16383, 16384, 20481])
def test_none_then_some(orc, prec, nr):
    from gpu_util import assert_eps_equal, dev
    R = synth.gaussian_mixture_unit(nr, 32, 5, 0.05, seed=1, stream=0)
    S = synth.gaussian_mixture_unit(70, 32, 5, 0.05, seed=1, stream=1)
    Rd, Sd, ws = dev(R), dev(S), ops.Workspace("cuda")
    some = float(np.sqrt(np.sort(orc.pair_d2(R, S, np.arange(nr) % nr, np.arange(nr) % 70))[nr // 3]))
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    for eps in (1e-6, some, 1e-6, 0.5 * some):
        got = ops.join_eps(Rd, Sd, eps, prec, workspace=ws, stream=st)
        if eps == 1e-6:
            assert st.query() and got.count == 0
        st.synchronize()
        assert_eps_equal(got, orc.eps_join(R, S, eps), 32, "%s %d eps %g" % (prec, nr, eps))
