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
    # an item's stages: twelve a wave at head dim 128 (ten of e4m3 with shared prompts), eight at 64 (twelve)
    ((64, 4, 7, 128, 0, 1536), (1, 4, 0, 1)),
    ((64, 4, 7, 128, 0, 1537), SCHEDULED),
    ((64, 4, 7, 128, 0, 1536, 1), (1, 4, 0, 0)),
    ((100, 4, 7, 128, 1, 1536), (1, 4, 0, 1)),
    ((100, 8, 7, 128, 1, 1280, 1), (1, 4, 0, 0)),
    ((100, 8, 7, 128, 1, 1281, 1), SCHEDULED),
    ((300, 2, 4, 64, 0, 1024), (1, 4, 1, 1)),
    ((300, 2, 4, 64, 0, 1025), SCHEDULED),
    ((240, 2, 4, 64, 0, 1152), (1, 4, 0, 1)),             # (nine in one round)
    ((240, 2, 4, 64, 0, 1153), SCHEDULED),
    ((300, 4, 1, 64, 1, 1024), (1, 4, 1, 1)),
    ((300, 4, 1, 64, 1, 1025), SCHEDULED),
    ((520, 2, 4, 64, 1, 1536, 1), (1, 4, 0, 0)),
    ((520, 2, 4, 64, 1, 1537, 1), SCHEDULED),
    # ... eight of eight waves
    ((29, 16, 1, 64, 1, 2048), (1, 8, 0, 1)),
    ((29, 16, 1, 64, 1, 2049), SCHEDULED),
    ((300, 2, 1, 64, 1, 2560), (1, 8, 1, 1)),             # (ten in order)
    ((300, 2, 1, 64, 1, 2561), SCHEDULED),
    ((45, 8, 8, 128, 1, 2560), (1, 8, 1, 1)),             # (ten at 128)
    ((45, 8, 8, 128, 1, 2561), SCHEDULED),
    ((32, 8, 2, 128, 1, 1536), (1, 8, 0, 1)),             # ... six with few query heads to a page of 128
    ((32, 8, 2, 128, 1, 1537), SCHEDULED),
    # ... six where several workgroups share it
    ((30, 4, 7, 128, 0, 1536), (2, 4, 0, 0)),
    ((30, 4, 7, 128, 0, 1537), SCHEDULED),
    ((43, 2, 2, 64, 0, 2560), (2, 8, 0, 0)),
    ((43, 2, 2, 64, 0, 2561), SCHEDULED),                 # ... five of bf16 at head dim 64
    ((43, 2, 2, 64, 1, 3072), (2, 8, 0, 0)),
    ((43, 2, 2, 64, 1, 3073), SCHEDULED),
    # rounds of workgroups: of bf16 pages of 128, ...
    ((160, 4, 7, 128, 0, 1024), (1, 4, 1, 1)),
    ((161, 4, 7, 128, 0, 1024), SCHEDULED),
    ((256, 4, 7, 128, 0, 64), (1, 4, 0, 0)),              # (a small batch: as many as there are)
    ((240, 4, 7, 128, 0, 512), (1, 4, 0, 1)),
    ((241, 4, 7, 128, 0, 512), SCHEDULED),
    ((144, 4, 7, 128, 0, 560, 1), (1, 4, 0, 0)),
    ((145, 4, 7, 128, 0, 560, 1), SCHEDULED),
    ((256, 4, 7, 128, 0, 1024), SCHEDULED),               # one of them long, the others short: 21.5 us scheduled, 23.1 not
    ((256, 4, 7, 128, 0, 1536), SCHEDULED),
    # ... e4m3 ones of 128, ...
    ((448, 4, 7, 128, 1, 1471), (1, 4, 1, 1)),
    ((449, 4, 7, 128, 1, 1471), SCHEDULED),
    ((704, 4, 7, 128, 1, 512), (1, 4, 0, 1)),
    ((705, 4, 7, 128, 1, 512), SCHEDULED),
    ((448, 4, 3, 128, 1, 512), (1, 4, 0, 1)),
    ((449, 4, 3, 128, 1, 512), SCHEDULED),
    ((320, 4, 3, 128, 1, 513), (1, 4, 0, 1)),
    ((321, 4, 3, 128, 1, 513), SCHEDULED),
    # ... bf16 at head dim 64, ...
    ((704, 4, 2, 64, 0, 512), (1, 4, 0, 1)),
    ((705, 4, 2, 64, 0, 512), SCHEDULED),
    ((512, 4, 2, 64, 0, 513), (1, 4, 0, 1)),
    ((513, 4, 2, 64, 0, 513), SCHEDULED),
    ((320, 4, 2, 64, 0, 800), (1, 4, 1, 1)),
    ((321, 4, 2, 64, 0, 800), SCHEDULED),
    # ... e4m3 at 64
    ((1024, 4, 2, 64, 1, 512), (1, 4, 0, 1)),
    ((1025, 4, 2, 64, 1, 512), SCHEDULED),
    ((512, 8, 2, 64, 1, 1000), (1, 4, 1, 1)),
    ((513, 8, 2, 64, 1, 1000), SCHEDULED),
    ((2048, 2, 4, 64, 1, 600, 1), (1, 4, 0, 0)),
    ((2049, 2, 4, 64, 1, 600, 1), SCHEDULED),
    # a last round that is nearly empty, of long items
    ((64, 4, 7, 128, 0, 1191), (1, 4, 0, 1)),
    ((35, 8, 1, 128, 0, 1191), SCHEDULED),
    ((10, 32, 1, 128, 0, 1369), SCHEDULED),
    ((10, 32, 4, 128, 0, 1369), (1, 4, 1, 1)),
    ((77, 4, 7, 128, 0, 1191), (1, 4, 1, 1)),
    ((129, 4, 16, 128, 0, 1311), SCHEDULED),
    ((154, 4, 16, 128, 0, 1311), (1, 4, 1, 1)),
    ((35, 8, 1, 128, 0, 700), (1, 4, 0, 1)),              # short ones: as many as there are
    ((35, 8, 2, 64, 0, 2000), SCHEDULED),                 # eight waves: two fifths full
    ((45, 8, 2, 64, 0, 2000), (1, 8, 1, 1)),
    # shared pages: what the caches take, less where a page has few query heads
    ((64, 4, 7, 128, 0, 1500, 1), (1, 4, 0, 0)),
    ((1024, 2, 4, 64, 1, 1280, 1), (1, 4, 0, 0)),
    ((128, 4, 7, 128, 0, 1280, 1), (1, 4, 0, 0)),
    ((128, 4, 7, 128, 0, 1281, 1), SCHEDULED),
    ((128, 32, 1, 128, 1, 257, 1), SCHEDULED),
    ((32, 8, 1, 128, 0, 1026, 1), (1, 4, 0, 0)),
    ((40, 8, 1, 128, 0, 592, 1), (1, 4, 0, 0)),           # (beyond one round)
    ((40, 8, 1, 128, 0, 624, 1), SCHEDULED),
    ((200, 2, 4, 64, 0, 1546, 1), SCHEDULED),             # eight waves, bf16, beyond one round
    ((128, 2, 4, 64, 0, 1546, 1), (1, 8, 0, 0)),
    ((200, 2, 16, 64, 0, 1800, 1), (1, 8, 0, 0)),
    ((400, 2, 4, 64, 1, 1600, 1), (1, 8, 0, 0)),
    ((116, 4, 7, 128, 1, 2048, 1), (1, 8, 0, 0)),
    ((160, 8, 5, 128, 1, 1518, 1), SCHEDULED),
    # nothing to do
    ((0, 4, 7, 128, 0, 1024), SCHEDULED),
    ((4, 4, 7, 128, 0, 0), SCHEDULED),
])
def test_plan(shape, want):
    got = plan(*shape)
    assert (got if got[0] else SCHEDULED) == want
