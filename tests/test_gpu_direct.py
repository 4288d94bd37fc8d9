"""Decode steps that go without a schedule, a workgroup per (sequence, kv head): against the oracle around the edges of the
rules that send them there (waves of a workgroup, the order of the sequences, the longest item, the shared pages' bytes)."""
import numpy as np
import pytest
import torch

import oracle
import workload
from gpu_util import DeviceProblem, compare, context

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dec():
    d = context()
    yield d
    d.close()


def lens(n, top, seed):
    """n lengths up to top: one of them top, some 0 and 1, the others anything between."""
    r = np.random.default_rng(seed).integers(0, top + 1, size=n)
    r[n // 2], r[0], r[-1] = top, 0, 1
    return [int(x) for x in r]


@pytest.mark.parametrize("kvd", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("Hq,Hkv,D,prompts,R,resp,whole", [
    (8, 4, 128, [0] * 40, 1, lens(40, 1536, 1), (True, True)),          # side by side: four waves (bf16), eight (e4m3); longest item
    (8, 4, 128, [0] * 40, 1, lens(40, 1537, 2), (False, True)),         # ... and a page past it
    (7, 1, 128, [0] * 200, 1, lens(200, 3073, 3), (False, False)),
    (8, 4, 128, [0] * 77, 1, lens(77, 900, 4), (True, True)),           # more items than compute units, not a multiple of eight: in order (bf16)
    (2, 1, 128, [0] * 360, 1, lens(360, 1601, 5), (False, True)),       # in order, eight waves (e4m3)
    (8, 2, 64, [0] * 100, 1, lens(100, 2560, 6), (True, True)),         # eight waves, ten stages each
    (8, 2, 64, [0] * 100, 1, lens(100, 2561, 7), (False, False)),
    (8, 4, 128, [0] * 30, 1, lens(30, 2048, 10), (False, False)),               # two or three workgroups to an item and the merge
    (8, 4, 128, [0] * 30, 1, lens(30, 2049, 11), (False, False)),       # ... and a page past it (bf16)
    (4, 2, 64, [0] * 60, 1, lens(60, 4096, 12), (False, False)),
    (2, 1, 64, [0] * 512, 1, [0] * 9 + [700] * 495 + [32 * 64 // 2] * 8, (True, True)),  # as many as are put in order, levels full of equals
    (2, 1, 64, [0] * 517, 1, lens(517, 1024, 8), (True, True)),         # more than that
    (4, 1, 64, [0] * 2049, 1, [33, 0, 17] * 683, (True, True)),
    (4, 2, 64, [100, 0, 333], 100, lens(300, 300, 9), (True, True)),    # groups: a member reads all its pages; some shorter than the prompt
])
def test_a_workgroup_per_item(dec, kvd, Hq, Hkv, D, prompts, R, resp, whole):
    p = workload.build_problem("direct", Hq, Hkv, D, prompts, R, resp, kv_dtype=kvd, seed=41)
    dp = DeviceProblem(p, use_hint=any(prompts))
    ws = dec.workspace(dp.c)
    ws.fill_(0xA5)
    print("case", Hq, Hkv, D, p.B, p.block_table.shape[1], kvd, flush=True)
    dec.decode(dp.c)
    out, lse = dp.results()
    # a step of one workgroup per item leaves the workspace alone: no schedule, no partials
    assert bool((ws == 0xA5).all()) == whole[kvd != "bf16"]
    # (outputs of one to three tokens are as large as single V entries: rounding them to bf16 alone is 2^-9 of that)
    compare(out, lse, *oracle.decode(p), "direct", abs_rel=2.0 ** -8)
    first = dp.out.clone()
    dec.decode(dp.c)
    torch.cuda.synchronize()
    assert torch.equal(first.view(torch.int16), dp.out.view(torch.int16))
