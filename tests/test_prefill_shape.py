"""Which launch shape a prefill call takes (CPU: the rule is a function of the sizes): its edges, and that what it says is
consistent over drawn calls."""
import ctypes
import random

import pytest

import paper_2507_01663_amd as ra

CUS = 256
AUTO = -1


class Shape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("waves", "parts", "levels", "per_die")]


def shape(lens, Hq, Hkv, D, bound=None, stay=AUTO, cus=CUS):
    """The library's own rule; it is no entry point of the C ABI, so it is called by the name the compiler gave it."""
    f = ra.load_library()._ZN2ra13prefill_shapeEiiiiiiii
    f.restype = Shape
    return f(len(lens), sum(lens), max(lens) if bound is None else bound, Hkv, Hq // Hkv, D, cus, stay)


def kind(*a, **k):
    s = shape(*a, **k)
    return {(8, 1): "stay", (4, 1): "four", (8, 2): "halves"}[s.waves, s.parts]


@pytest.mark.parametrize("lens,Hq,Hkv,D,bound,want", [
    ([256], 28, 4, 128, None, "four"),            # short: four waves, also with a compute unit to each block
    ([257], 28, 4, 128, None, "halves"),
    ([224], 8, 2, 64, None, "four"),
    ([225], 8, 2, 64, None, "halves"),
    ([701], 28, 4, 128, None, "halves"),
    ([1100], 28, 4, 128, None, "halves"),         # 247 blocks
    ([1200], 28, 4, 128, None, "four"),           # 269
    ([128] * 8, 28, 4, 128, None, "four"),
    ([368] * 6, 28, 4, 128, None, "four"),        # 487 blocks by the tokens: two to a compute unit
    ([368] * 8, 28, 4, 128, None, "stay"),
    ([60] * 37, 32, 2, 64, None, "four"),         # three to a compute unit at head dim 64
    ([60] * 119, 32, 2, 64, None, "four"),        # ... and up to four rounds of them
    ([60] * 120, 32, 2, 64, None, "stay"),
    ([1024] * 12, 32, 2, 64, None, "four"),
    ([1024] * 13, 32, 2, 64, None, "stay"),
    ([60] * 62, 28, 4, 128, None, "four"),        # short prompts at head dim 128: three rounds
    ([60] * 63, 28, 4, 128, None, "stay"),
    ([65] * 20 + [1] * 5, 28, 4, 128, None, "four"),
    ([128] * 12, 64, 8, 128, None, "four"),       # ... and two and a half
    ([129] * 17, 28, 4, 128, None, "stay"),       # longer ones: those that run side by side
    ([4] * 5, 64, 8, 128, None, "four"),          # one tile of the eight that the bound is rounded up to
    ([9] * 38, 8, 8, 128, None, "four"),
    ([10] * 8, 28, 4, 128, 512, "four"),
    ([10] * 8, 28, 4, 128, 513, "stay"),
    ([512] * 16, 28, 4, 128, 2560, "stay"),       # a bound that makes like lengths look unlike
    ([100, 300, 500, 700] * 3, 28, 4, 128, None, "four"),   # long prompts of unlike lengths
    ([20, 100, 200, 500] * 3, 28, 4, 128, None, "four"),    # shorter ones too
    ([20, 100, 200, 500] * 8, 28, 4, 128, None, "four"),    # 3.2 blocks of eight units to a compute unit
    ([20, 100, 200, 500] * 10, 28, 4, 128, None, "stay"),   # 4.0
    ([20, 100, 200, 500] * 12, 32, 2, 64, None, "four"),    # head dim 64
    ([350, 390, 400, 500] * 3, 28, 4, 128, None, "stay"),   # nearly alike
    ([200, 500, 900, 1500] * 12, 28, 4, 128, None, "stay"), # ... and many blocks
    ([512] * 32, 28, 4, 128, None, "stay"),
    ([2048] * 16, 64, 8, 128, None, "stay"),
    ([16] * 4096, 4, 1, 64, None, "stay"),
    ([10] * 8, 28, 4, 128, 4096, "stay"),         # a bound far above the lengths
    ([21] * 63, 8, 2, 64, None, "four"),          # ... nearer, though the bound is rounded up to 256 rows
    ([20, 60, 100] * 120, 16, 2, 64, None, "stay"),  # many short prompts: 38 trips past them, over all rounds of workgroups
    ([20, 60, 100] * 60, 16, 2, 64, None, "four"),   # 9.5
    ([20, 40, 60] * 300, 4, 2, 64, None, "four"),    # ... few query heads to a kv head: 102
    ([20, 40, 60] * 500, 4, 2, 64, None, "stay"),    # 285
    ([40] * 6000, 1, 1, 64, None, "stay"),
])
def test_edges(lens, Hq, Hkv, D, bound, want):
    assert kind(lens, Hq, Hkv, D, bound) == want


def test_what_was_asked_for():
    lens = [512] * 32
    assert kind(lens, 28, 4, 128, stay=0) == "four"
    assert shape(lens, 28, 4, 128, stay=2).per_die == 2 and kind(lens, 28, 4, 128, stay=2) == "stay"
    assert shape(lens, 28, 4, 128, stay=64).per_die == CUS // 8
    # workgroups that stay also where a workgroup per block would have been the library's choice, and no more than asked for
    for lens, Hq, Hkv in (([257], 8, 8), ([600], 28, 4), ([1], 8, 8), ([100, 300, 500, 700] * 3, 28, 4), ([20, 100, 200, 500] * 3, 28, 4)):
        assert kind(lens, Hq, Hkv, 128) != "stay"
        for stay in (1, 2, 64):
            s = shape(lens, Hq, Hkv, 128, stay=stay)
            assert (s.waves, s.parts) == (8, 1) and s.per_die == min(stay, CUS // 8)


def test_every_block_has_a_workgroup():
    """With a workgroup per block a die has as many as it can have blocks: units of 32 rows and a head, four to a block, the
    blocks of a (prompt, kv head) dealt to the dies that share its heads in turn."""
    r = random.Random(5)
    for _ in range(3000):
        Hkv, G = r.choice([1, 2, 3, 4, 8, 6, 16]), r.choice([1, 2, 3, 4, 5, 7, 8, 16])
        n, longest = int(2 ** r.uniform(0, 6)), int(2 ** r.uniform(0, 11))
        lens = [r.randint(0, longest) for _ in range(n)]
        bound = longest + r.choice([0, 0, 1, 100])
        s = shape(lens, Hkv * G, Hkv, r.choice([64, 128]), bound, r.choice([AUTO, AUTO, 0]))
        assert s.per_die >= 1 and s.levels >= 1
        units = 8 if (s.waves, s.parts) == (8, 1) else 4
        gg = next(g for g in (8, 4, 2, 1) if Hkv % g == 0)
        share = 8 // gg
        most = 0
        for die in range(share):
            blocks = 0
            for g, L in enumerate(lens):
                nb, first = -(-(-(-L // 32) * G) // units), (die + g) % share
                mine = max(0, -(-(nb - first) // share))
                assert mine <= s.levels
                blocks += mine * (Hkv // gg)
            most = max(most, blocks)
        if units == 4:
            assert most <= s.per_die


def test_no_more_workgroups_than_the_tokens_can_fill():
    """A prompt has at most 31 tokens more than fill its tiles, a pair's last block three units fewer than four, and of a pair's
    blocks the dies that share it take one more than their share: beyond that, and beyond those that run side by side anyway, no
    workgroup is launched, however far the bound on the lengths lies above them."""
    r = random.Random(9)
    for _ in range(2000):
        Hkv, G = r.choice([1, 2, 3, 4, 8, 6, 16]), r.choice([1, 2, 3, 4, 5, 7, 8, 16])
        n, longest = int(2 ** r.uniform(0, 10)), int(2 ** r.uniform(0, 9))
        lens = [r.randint(1, longest) for _ in range(n)]
        D = r.choice([64, 128])
        s = shape(lens, Hkv * G, Hkv, D, longest, r.choice([AUTO, 0]))
        if (s.waves, s.parts) == (8, 1):
            continue
        tiles, share = (sum(lens) + 31 * n) / 32, 8 // next(g for g in (8, 4, 2, 1) if Hkv % g == 0)
        assert 8 * s.per_die <= (3 if D == 64 else 2) * CUS or 8 * s.per_die <= Hkv * ((tiles * G + 3 * n) / 4 + n * (share - 1) / 2 + share * (share - 1) / 2)
