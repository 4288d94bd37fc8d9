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
    # an item's stages: twelve a wave, sixteen at head dim 64
    ((64, 4, 7, 128, 0, 1536), (1, 4, 0, 1)),
    ((64, 4, 7, 128, 0, 1537), SCHEDULED),
    ((300, 4, 1, 64, 1, 2048), (1, 4, 1, 1)),
    ((300, 4, 1, 64, 1, 2049), SCHEDULED),
    # ... ten of eight waves in no order, sixteen in order
    ((29, 16, 1, 64, 1, 2560), (1, 8, 0, 1)),
    ((29, 16, 1, 64, 1, 2561), SCHEDULED),
    ((100, 2, 4, 64, 0, 2560), (1, 8, 0, 1)),
    ((100, 2, 4, 64, 0, 2561), SCHEDULED),
    ((45, 8, 8, 128, 1, 2560), (1, 8, 1, 1)),
    ((45, 8, 8, 128, 1, 2561), SCHEDULED),
    ((300, 2, 1, 64, 1, 4096), (1, 8, 1, 1)),
    ((300, 2, 1, 64, 1, 4097), SCHEDULED),
    # ... twelve of bf16 beyond one round in no order
    ((849, 2, 4, 64, 0, 1536), (1, 4, 0, 1)),
    ((849, 2, 4, 64, 0, 1537), SCHEDULED),
    ((849, 2, 4, 64, 1, 1958), (1, 4, 0, 1)),
    # ... eight where several workgroups share it
    ((30, 4, 7, 128, 0, 2048), (2, 4, 0, 0)),
    ((30, 4, 7, 128, 0, 2049), SCHEDULED),
    # rounds of workgroups
    ((192, 4, 7, 128, 0, 1024), (1, 4, 1, 1)),
    ((193, 4, 7, 128, 0, 1024), SCHEDULED),
    ((80, 8, 1, 128, 0, 679), (1, 4, 0, 1)),
    ((81, 8, 1, 128, 0, 679), SCHEDULED),                 # ... with few query heads to a page
    ((256, 4, 7, 128, 0, 1024), SCHEDULED),               # one of them long, the others short: 21.5 us scheduled, 23.1 not
    ((256, 4, 7, 128, 0, 1536), SCHEDULED),
    ((1000, 8, 1, 128, 0, 64), SCHEDULED),
    ((448, 4, 7, 128, 1, 1471), (1, 4, 1, 1)),
    ((449, 4, 7, 128, 1, 1471), SCHEDULED),
    ((1024, 4, 7, 128, 1, 308), (1, 4, 0, 1)),
    ((1025, 4, 7, 128, 1, 308), SCHEDULED),
    ((474, 8, 1, 128, 1, 481), SCHEDULED),                # few query heads to a page
    ((224, 8, 2, 64, 0, 2000), (1, 4, 1, 1)),
    ((225, 8, 2, 64, 0, 2000), SCHEDULED),
    ((1024, 4, 4, 64, 0, 500), (1, 4, 0, 1)),
    ((1024, 4, 2, 64, 0, 500), SCHEDULED),
    ((478, 8, 5, 128, 1, 740), SCHEDULED),
    ((512, 8, 2, 64, 1, 2000), (1, 4, 1, 1)),
    ((513, 8, 2, 64, 1, 2000), SCHEDULED),
    # a last round that is nearly empty, of long items
    ((64, 4, 7, 128, 0, 1191), (1, 4, 0, 1)),
    ((35, 8, 1, 128, 0, 1191), SCHEDULED),
    ((10, 32, 1, 128, 0, 1369), SCHEDULED),
    ((10, 32, 4, 128, 0, 1369), (1, 4, 1, 1)),
    ((77, 4, 7, 128, 0, 1191), (1, 4, 1, 1)),
    ((129, 4, 16, 128, 0, 1311), SCHEDULED),
    ((154, 4, 16, 128, 0, 1311), (1, 4, 1, 1)),
    ((35, 8, 1, 128, 0, 700), (1, 4, 0, 1)),              # short ones: as many as there are
    ((35, 8, 2, 64, 0, 2300), SCHEDULED),                 # eight waves: two fifths full
    ((45, 8, 2, 64, 0, 2300), (1, 8, 1, 1)),
    # shared pages: what the caches take, less where a page has few query heads
    ((64, 4, 7, 128, 0, 1500, 1), (1, 4, 0, 0)),
    ((1024, 2, 4, 64, 1, 1280, 1), (1, 4, 0, 0)),
    ((175, 4, 7, 128, 0, 927, 1), (1, 4, 0, 0)),
    ((182, 4, 7, 128, 0, 944, 1), SCHEDULED),
    ((128, 32, 1, 128, 1, 257, 1), SCHEDULED),
    ((32, 8, 1, 128, 0, 1024, 1), (1, 4, 0, 0)),
    ((32, 8, 1, 128, 0, 1040, 1), SCHEDULED),
    ((200, 2, 4, 64, 0, 1546, 1), SCHEDULED),             # eight waves, bf16, beyond one round
    ((128, 2, 4, 64, 0, 1546, 1), (1, 8, 0, 0)),
    ((400, 2, 4, 64, 1, 1600, 1), (1, 8, 0, 0)),
    ((116, 4, 7, 128, 1, 2048, 1), (1, 8, 0, 0)),
    ((116, 4, 7, 128, 1, 2049, 1), SCHEDULED),
    ((160, 8, 5, 128, 1, 1518, 1), SCHEDULED),
    # nothing to do
    ((0, 4, 7, 128, 0, 1024), SCHEDULED),
    ((4, 4, 7, 128, 0, 0), SCHEDULED),
])
def test_plan(shape, want):
    got = plan(*shape)
    assert (got if got[0] else SCHEDULED) == want
