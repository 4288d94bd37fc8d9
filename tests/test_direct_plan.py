"""Which decode batches go without a schedule, and how: the library's host rule at its edges (256 compute units, 1024 resident
attention waves for bf16 pools and 2048 for e4m3 ones; nothing runs on a GPU here)."""
import pytest

from gpu_util import direct_plan

SCHEDULED = (0, 0, 0, 0)


def plan(B, Hkv, G, D, fp8, tokens, share=0):
    p = direct_plan(B, Hkv, G, D, fp8, (tokens + 15) // 16, share, 256, 2048 if fp8 else 1024)
    return (p.splits, p.waves, p.sorted, p.turned)


# (splits, waves, the longest first, turned about over the dies)
@pytest.mark.parametrize("shape,want", [
    # small batches: as they come
    ((4, 2, 2, 64, 0, 256), (1, 4, 0, 0)),
    ((10, 8, 8, 128, 0, 349), (1, 4, 0, 0)),
    ((8, 4, 7, 128, 0, 2001, 1), (8, 4, 0, 0)),
    # ... eight waves at head dim 64 only, bf16 only unsplit
    ((10, 8, 1, 128, 1, 1498), (3, 4, 0, 0)),
    ((80, 2, 4, 64, 1, 1504), (1, 8, 0, 0)),
    ((10, 8, 2, 64, 0, 1441), (3, 4, 0, 0)),
    ((69, 2, 2, 64, 0, 831), (1, 8, 0, 0)),
    # the bytes of the table: 32 MB, or 96 with a quarter as many items as compute units
    ((25, 4, 2, 128, 0, 640), (2, 4, 0, 0)),
    ((25, 4, 2, 128, 0, 640, 1), (2, 4, 0, 0)),
    ((25, 4, 2, 128, 0, 641), (2, 4, 0, 0)),              # (past it, but several workgroups to an item ...
    ((25, 4, 2, 128, 0, 641, 1), SCHEDULED),              # ... keep the schedule where prompts are shared)
    ((4, 2, 1, 128, 0, 24576, 1), (32, 4, 0, 0)),
    ((4, 2, 1, 128, 0, 24577, 1), SCHEDULED),
    # nothing to do
    ((0, 4, 7, 128, 0, 1024), SCHEDULED),
    ((4, 4, 7, 128, 0, 0), SCHEDULED),
])
def test_plan(shape, want):
    got = plan(*shape)
    assert (got if got[0] else SCHEDULED) == want
