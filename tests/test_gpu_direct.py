"""Decode steps that go without a schedule, a workgroup per (sequence, kv head): against the oracle around the edges of the
rules that send them there (waves of a workgroup, the order of the sequences, the longest item, the shared pages' bytes)."""
import numpy as np
import pytest
import torch

import oracle
import workload
from gpu_util import DeviceProblem, compare, context, plan_of

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


S = (0, 0, 0, 0)             # has a schedule; otherwise workgroups per item, their waves, longest first, turned about


@pytest.mark.parametrize("kvd", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("Hq,Hkv,D,prompts,R,resp,plans", [
    (8, 4, 128, [0] * 40, 1, lens(40, 1536, 1), ((1, 4, 0, 1), (1, 8, 0, 1))),   # side by side: four waves (bf16), eight (e4m3); longest item
    (16, 4, 128, [0] * 40, 1, lens(40, 1537, 2), (S, (1, 8, 0, 1))),              # ... and a page past it
    (16, 4, 128, [0] * 40, 1, lens(40, 2561, 3), (S, S)),
    (8, 4, 128, [0] * 90, 1, lens(90, 900, 4), ((1, 4, 1, 1), (1, 4, 0, 1))),    # more items than compute units, in order (bf16)
    (8, 4, 128, [0] * 131, 1, lens(131, 900, 13), (S, (1, 4, 1, 1))),            # ... e4m3; not a multiple of eight
    (4, 1, 128, [0] * 360, 1, lens(360, 1601, 5), (S, (1, 8, 1, 1))),            # in order, eight waves (e4m3)
    (8, 2, 64, [0] * 100, 1, lens(100, 2048, 6), ((1, 8, 0, 1), (1, 8, 0, 1))),  # eight waves, eight stages each
    (8, 2, 64, [0] * 100, 1, lens(100, 2049, 7), (S, S)),
    (8, 2, 64, [0] * 180, 1, lens(180, 1700, 14), ((1, 8, 1, 1), (1, 8, 0, 1))),  # ... in order (bf16)
    (4, 2, 64, [0] * 512, 1, lens(512, 1760, 15), (S, (1, 8, 1, 1))),            # as many as are put in order, eight waves
    (2, 2, 64, [0] * 512, 1, lens(512, 1000, 16), ((1, 4, 1, 1), (1, 4, 0, 1))),  # ... four waves (bf16)
    (4, 4, 64, [0] * 300, 1, lens(300, 1000, 18), ((1, 4, 1, 1), (1, 4, 1, 1))),            # ... e4m3
    (2, 2, 64, [0] * 512, 1, [0] * 9 + [700] * 487 + [1000] * 16, ((1, 4, 1, 1), (1, 4, 0, 1))),  # levels full of equals
    (4, 4, 64, [0] * 300, 1, [800] * 300, ((1, 4, 1, 1), (1, 4, 1, 1))),                    # ... one level for all, of a width that is no power of two
    (8, 4, 128, [0] * 30, 1, lens(30, 1536, 10), ((2, 4, 0, 0), (2, 8, 0, 0))),  # two or three workgroups to an item and the merge
    (8, 4, 128, [0] * 30, 1, lens(30, 1537, 11), (S, (2, 8, 0, 0))),             # ... and a page past it (bf16)
    (4, 2, 64, [0] * 60, 1, lens(60, 2560, 12), ((2, 8, 0, 0), (2, 8, 0, 0))),
    (2, 1, 64, [0] * 512, 1, [0] * 9 + [700] * 495 + [32 * 64 // 2] * 8, ((1, 4, 0, 1), (1, 4, 0, 1))),  # no more than run side by side: as they come
    (2, 1, 64, [0] * 517, 1, lens(517, 768, 8), ((1, 4, 0, 1), (1, 4, 0, 1))),   # more sequences than are put in order
    (4, 1, 64, [0] * 1789, 1, [33, 0, 17] * 596 + [33], ((1, 4, 0, 1), (1, 4, 0, 1))),
    (4, 2, 64, [100, 0, 333], 100, lens(300, 300, 9), ((1, 4, 0, 0), (1, 4, 0, 0))),  # groups: a member reads all its pages; some shorter than the prompt
])
def test_a_workgroup_per_item(dec, kvd, Hq, Hkv, D, prompts, R, resp, plans):
    p = workload.build_problem("direct", Hq, Hkv, D, prompts, R, resp, kv_dtype=kvd, seed=41)
    dp = DeviceProblem(p, use_hint=any(prompts))
    plan = plan_of(dec, p, use_hint=any(prompts))
    assert (tuple(plan) if plan.splits else S) == plans[kvd != "bf16"]
    ws = dec.workspace(dp.c)
    ws.fill_(0xA5)
    print("case", Hq, Hkv, D, p.B, p.block_table.shape[1], kvd, flush=True)
    dec.decode(dp.c)
    out, lse = dp.results()
    # a step of one workgroup per item leaves the workspace alone: no schedule, no partials
    assert bool((ws == 0xA5).all()) == (plan.splits == 1)
    # (outputs of one to three tokens are as large as single V entries: rounding them to bf16 alone is 2^-9 of that)
    compare(out, lse, *oracle.decode(p), "direct", abs_rel=2.0 ** -8)
    first = dp.out.clone()
    dec.decode(dp.c)
    torch.cuda.synchronize()
    assert torch.equal(first.view(torch.int16), dp.out.view(torch.int16))


@pytest.mark.parametrize("kvd", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("Hq,Hkv,D,B,top,plans", [
    (4, 2, 64, 70, 1500, ((1, 8, 0, 1), (1, 8, 0, 0))),
    (16, 4, 128, 40, 1537, (S, (1, 8, 0, 1))),
    (4, 2, 64, 300, 1600, (S, (1, 8, 1, 1))),
    (8, 2, 64, 180, 1700, ((1, 8, 1, 1), (1, 8, 0, 1))),
    (8, 4, 128, 90, 900, ((1, 4, 1, 1), (1, 4, 0, 1))),
])
def test_strided_pools(dec, kvd, Hq, Hkv, D, B, top, plans):
    """K and V interleaved page by page and a row of slack behind every slot's: every stride is used as given."""
    p = workload.build_problem("strided", Hq, Hkv, D, [0] * B, 1, lens(B, top, 17), kv_dtype=kvd, seed=43)
    dp = DeviceProblem(p, use_hint=False)
    plan = plan_of(dec, p, use_hint=False)
    assert (tuple(plan) if plan.splits else S) == plans[kvd != "bf16"]
    n, slack = p.num_pages, 16 // dp.k_pool.element_size()
    both = torch.zeros((n, 2, Hkv, 16, D + slack), dtype=dp.k_pool.dtype, device="cuda:0")
    both[:, 0, :, :, :D], both[:, 1, :, :, :D] = dp.k_pool, dp.v_pool
    dp.k_pool, dp.v_pool = both[:, 0, :, :, :D], both[:, 1, :, :, :D]
    dp.set(use_hint=False)
    assert dp.c.kv_stride_token == D + slack and dp.c.kv_stride_page == 2 * Hkv * 16 * (D + slack)
    print("case", Hq, Hkv, D, B, top, kvd, flush=True)
    dec.decode(dp.c)
    compare(*dp.results(), *oracle.decode(p), "strided", abs_rel=2.0 ** -8)


@pytest.mark.parametrize("kvd,Hq,Hkv,D", [("bf16", 28, 4, 128), ("fp8_e4m3", 8, 2, 64)])
@pytest.mark.parametrize("pages", [1, 2, 63, 64, 65, 127, 128, 129, 193])
def test_widths_of_the_table(dec, kvd, Hq, Hkv, D, pages):
    """One sequence fills its row, others end anywhere; of wide tables several workgroups share an item and the merge adds them up."""
    top = 16 * pages
    p = workload.build_problem("width", Hq, Hkv, D, [0] * 4, 1, [top - 3, 0, 1, top // 2 + 1], kv_dtype=kvd, seed=47)
    plan = plan_of(dec, p, use_hint=False)
    assert plan.splits == 1 if pages < 63 else plan.splits > 1
    dp = DeviceProblem(p, use_hint=False)
    dec.workspace(dp.c).fill_(0xA5)
    print("case", kvd, Hq, Hkv, D, pages, flush=True)
    dec.decode(dp.c)
    compare(*dp.results(), *oracle.decode(p), "width", abs_rel=2.0 ** -8)
