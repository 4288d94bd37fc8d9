"""Prefill calls of few blocks: workgroups of four waves, and two waves to a unit's keys, against the oracle at the edges of
tiles and stages, with cache writes bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2507_01663_amd as ra
import workload
from test_gpu_prefill import DevicePrefill, check_minus_infinity, compare, expected_pools
from test_prefill_shape import kind
from workload.gen import bf16_bits_to_f32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dec():
    d = ra.Decoder(0)
    yield d
    d.close()


def check(dec, b, want, kv_dtype=None, what="", bound=None):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert kind([int(x) for x in b.lens], b.Hq, b.Hkv, b.D, bound, cus=cus) == want
    d = DevicePrefill(b, kv_dtype, max_len=bound)
    print("case", what, b.Hq, b.Hkv, b.D, list(b.lens), kv_dtype, flush=True)
    dec.prefill(d.c)
    out, lse = d.results()
    compare(out, lse, *oracle.prefill(b.q, b.k, b.v, b.cu_seqlens, b.softmax_scale), what)
    first = d.out.clone()
    dec.prefill(d.c)
    torch.cuda.synchronize()
    assert torch.equal(first.view(torch.int16), d.out.view(torch.int16))
    return d


@pytest.mark.parametrize("Hq,Hkv,D", [(28, 4, 128), (4, 2, 64), (3, 1, 128), (8, 8, 64), (16, 1, 128), (10, 2, 128)])
@pytest.mark.parametrize("lens,want", [
    ([1], "four"), ([31, 0, 33], "four"), ([64, 65], "four"), ([224], "four"), ([256], {64: "halves", 128: "four"}),
    ([257], "halves"), ([288], "halves"), ([289], "halves"), ([320, 31], "halves"), ([33, 415], "halves"), ([640], "halves"),
])
def test_edges_of_tiles_and_stages(dec, Hq, Hkv, D, lens, want):
    check(dec, workload.build_prefill("few", Hq, Hkv, D, lens, seed=21), want if isinstance(want, str) else want[D], what="few")


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("Hq,Hkv,D,lens,want", [
    (28, 4, 128, [300, 17], "halves"), (8, 2, 64, [17, 290, 16, 1], "halves"), (28, 4, 128, [100, 31, 0, 50], "four"), (16, 2, 64, [47, 128], "four"),
    (28, 4, 128, [600, 30, 333, 80, 200, 513, 47], "four"),
    (8, 8, 128, [290], "halves"), (6, 2, 64, [300, 31], "halves"), (4, 2, 64, [600, 30, 333, 80, 200], "halves"),  # few heads to a kv head:
    (8, 8, 128, [33, 250, 0, 16], "four"), (6, 2, 64, [129, 1], "four"),                                            # up to four stages a block
    (8, 8, 64, [33, 200, 0, 16], "four"), (8, 8, 128, [96, 5], "four"), (8, 8, 128, [97, 5], "four"), (16, 16, 128, [140, 97, 111, 30, 99, 100, 128], "four"),
    (64, 8, 128, [33, 5, 64, 31, 0, 17, 48] * 4, "four"), (28, 4, 128, [60] * 62, "four"), (28, 4, 128, [60] * 63, "stay"),   # more blocks than
    (40, 8, 128, [128, 97, 65] * 4, "four"), (8, 8, 128, [9, 1, 4] * 13, "four"), (4, 4, 64, [37, 2] * 40, "four"),           # run side by side,
    (32, 2, 64, [200, 3, 129, 256] * 5, "four"), (16, 1, 64, [700, 20, 20, 64, 1] * 4, "four"),                               # or short prompts
])
def test_cache_writes(dec, kv_dtype, Hq, Hkv, D, lens, want):
    b = workload.build_prefill("few", Hq, Hkv, D, lens, seed=23)
    d = check(dec, b, want, kv_dtype, "write")
    k, v, ks, vs = expected_pools(b, kv_dtype)
    for got, ref in ((d.k_pool, k), (d.v_pool, v)):
        got = got.view(torch.int16).cpu().numpy().view(np.uint16) if kv_dtype == "bf16" else got.cpu().numpy()
        assert np.array_equal(got, ref)
    if ks is not None:
        assert np.array_equal(d.k_scale.cpu().numpy(), ks, equal_nan=True) and np.array_equal(d.v_scale.cpu().numpy(), vs, equal_nan=True)


@pytest.mark.parametrize("D", [64, 128])
def test_keys_of_one_part_that_dwarf_the_other_parts(dec, D):
    """The parts' reference points lie far apart: the one with the small scores has to vanish, whichever it is."""
    for t in (5, 40, 70, 299):
        b = workload.build_prefill("few", 8, 2, D, [300], seed=25)
        k = bf16_bits_to_f32(b.k).copy()
        k[t] *= 1000.0
        b.k = workload.f32_to_bf16_bits(k)
        check(dec, b, "halves", what="dominant key %d" % t)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("stages", [0, 1])
def test_scores_of_minus_infinity_in_one_part(dec, D, stages):
    """All keys of one of the two waves score -inf: their weights are zero and the results those of the other wave's keys alone."""
    assert kind([300], 4, 1, D, cus=torch.cuda.get_device_properties(0).multi_processor_count) == "halves"
    check_minus_infinity(dec, D, stages, 300)
