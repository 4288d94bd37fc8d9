"""The Python side of a call: the workspace that grows when the library says so, the stream it goes to, errors as before."""
import pytest
import torch

import paper_2507_01663_amd as ra
import workload
from gpu_util import DeviceProblem, context

pytestmark = pytest.mark.gpu


def results(dp):
    torch.cuda.synchronize()
    return dp.out.view(torch.int16).clone(), dp.lse.clone()


def test_workspace_grows_with_the_problems():
    small, large = (DeviceProblem(workload.make_problem(n, seed=3)) for n in ("tiny", "mid7b"))
    want = []
    for dp in (small, large):
        d = context()
        d.decode(dp.c)
        want.append(results(dp))
        d.close()
    d = context()
    for dp, w in ((small, want[0]), (large, want[1]), (small, want[0]), (large, want[1])):
        dp.out.fill_(float("nan"))
        d.decode(dp.c)
        got = results(dp)
        assert torch.equal(got[0], w[0]) and torch.equal(got[1], w[1])
        assert d.workspace(dp.c) is d._ws and d._ws.data_ptr() == d._ws_at[0] and d._ws.numel() >= ra.rollout_attn_workspace_size(d.ctx, dp.c)
    assert len(d._retired) == 1                      # the one that was too small, and nothing since
    large.c.D = 96
    for _ in range(2):
        with pytest.raises(ra.RolloutAttnError, match="RA_ERR_UNSUPPORTED"):
            d.decode(large.c)
    d.close()


def test_current_stream():
    d = context()
    dp = DeviceProblem(workload.make_problem("tiny", seed=4))
    d.decode(dp.c)
    want = results(dp)
    s = torch.cuda.Stream()
    assert d._hip_stream(None) == torch.cuda.current_stream(0).cuda_stream and d._hip_stream(s) == s.cuda_stream
    with torch.cuda.stream(s):
        assert d._hip_stream(None) == s.cuda_stream
        dp.out.zero_()
        d.decode(dp.c)
    got = results(dp)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    d.close()
