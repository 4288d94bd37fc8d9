"""Prompt prefill on the GPU through the C ABI against the fp64 oracle: causal attention of packed prompts
(element by element at reduced sizes, whole prompts and sampled heads at the benchmark's sizes), the cache
write (bit-exact), and the hand-over to the decode step."""
import numpy as np
import pytest
import torch

import oracle
import paper_2507_01663_amd as ra
import workload
from gpu_util import ABS_TOL, LSE_TOL, REL_TOL, bits_to_bf16
from gpu_util import compare as compare_decode
from workload.gen import PAGE, bf16_bits_to_f32

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
OUT_ULP = 2.0 ** -8      # one bf16 unit in the last place, relative: the allowance for outputs that are not small


def compare(out, lse, ref_out, ref_lse, what=""):
    """The decode tolerances, with the element-wise bound widened by one bf16 ulp of the reference's magnitude."""
    return compare_decode(out, lse, ref_out, ref_lse, what, abs_rel=OUT_ULP)


@pytest.fixture(scope="module", params=["the library's choice", "one workgroup per block", "two workgroups per die that stay",
                                        "one per compute unit that stays"])
def dec(request):
    """Every test runs in the launch shape the library picks and in each of those it can be told to use: the results must
    not depend on how the blocks of query rows are dealt to workgroups (the setting is read when the context is made)."""
    import os
    value = {"the library's choice": None, "one workgroup per block": "0", "two workgroups per die that stay": "2",
             "one per compute unit that stays": "64"}[request.param]
    old = os.environ.get("ROLLOUT_ATTN_PREFILL_WGS_PER_DIE")
    if value is None:
        os.environ.pop("ROLLOUT_ATTN_PREFILL_WGS_PER_DIE", None)
    else:
        os.environ["ROLLOUT_ATTN_PREFILL_WGS_PER_DIE"] = value
    try:
        d = ra.Decoder(0)
    finally:
        if old is None:
            os.environ.pop("ROLLOUT_ATTN_PREFILL_WGS_PER_DIE", None)
        else:
            os.environ["ROLLOUT_ATTN_PREFILL_WGS_PER_DIE"] = old
    yield d
    d.close()


class DevicePrefill:
    def __init__(self, b, kv_dtype=None, max_len=None, poison=True):
        self.b = b
        self.q, self.k, self.v = bits_to_bf16(b.q, DEV), bits_to_bf16(b.k, DEV), bits_to_bf16(b.v, DEV)
        self.cu = torch.from_numpy(b.cu_seqlens).to(DEV)
        T = b.q.shape[0]
        self.out = torch.full((T, b.Hq, b.D), float("nan"), dtype=torch.bfloat16, device=DEV)
        self.lse = torch.full((T, b.Hq), float("nan"), dtype=torch.float32, device=DEV)
        pools = {}
        if kv_dtype is not None:
            shape = (b.num_pages, b.Hkv, PAGE, b.D)
            if kv_dtype == "bf16":
                self.k_pool = torch.full(shape, float("nan"), dtype=torch.bfloat16, device=DEV)
                self.v_pool = torch.full(shape, float("nan"), dtype=torch.bfloat16, device=DEV)
                self.k_scale = self.v_scale = None
            else:
                self.k_pool = torch.full(shape, 0x7F, dtype=torch.uint8, device=DEV)
                self.v_pool = torch.full(shape, 0x7F, dtype=torch.uint8, device=DEV)
                self.k_scale = torch.full((b.num_pages, b.Hkv), float("nan"), dtype=torch.float32, device=DEV)
                self.v_scale = torch.full((b.num_pages, b.Hkv), float("nan"), dtype=torch.float32, device=DEV)
            self.page_off = torch.from_numpy(b.page_offsets).to(DEV)
            self.pages = torch.from_numpy(b.pages).to(DEV) if b.pages.size else torch.zeros(1, dtype=torch.int32, device=DEV)
            pools = dict(k_pool=self.k_pool, v_pool=self.v_pool, k_scale=self.k_scale, v_scale=self.v_scale,
                         page_offsets=self.page_off, pages=self.pages)
        lens = b.lens
        self.c = ra.prefill_from_tensors(self.q, self.k, self.v, self.cu, int(lens.max()) if max_len is None and lens.size else (max_len or 0),
                                         self.out, self.lse, float(b.softmax_scale), **pools)

    def results(self):
        torch.cuda.synchronize()
        return self.out.float().cpu().numpy().astype(np.float64), self.lse.cpu().numpy().astype(np.float64)


def check_all(dec, b, what):
    d = DevicePrefill(b)
    dec.prefill(d.c)
    out, lse = d.results()
    ref_out, ref_lse = oracle.prefill(b.q, b.k, b.v, b.cu_seqlens, b.softmax_scale)
    return compare(out, lse, ref_out, ref_lse, what)


@pytest.mark.parametrize("Hq,Hkv,D,lens", [
    (28, 4, 128, [1, 15, 16, 17, 33, 255, 256, 257, 300, 0, 700]),     # around every tile, stage and block edge
    (8, 2, 64, [5, 64, 513, 31, 32]),
    (4, 4, 128, [129, 2, 511]),                                          # one query head per kv head
    (32, 2, 64, [100, 260]),                                             # sixteen
    (40, 8, 128, [48, 1024]),
])
def test_every_element_against_the_oracle(dec, Hq, Hkv, D, lens):
    b = workload.build_prefill("pf", Hq, Hkv, D, lens, seed=3)
    errs = check_all(dec, b, "prefill Hq=%d Hkv=%d D=%d lens=%s" % (Hq, Hkv, D, lens))
    print("errors (abs, row-rel, lse):", errs)


def test_large_scores_and_an_outlier_key(dec):
    # scores far from zero exercise the running maximum: a key early in the prompt that dominates, then is overtaken
    b = workload.build_prefill("pf", 8, 2, 128, [400], seed=5)
    k = bf16_bits_to_f32(b.k).copy()
    k[7] *= 6.0
    k[300] *= 9.0
    b.k = workload.f32_to_bf16_bits(k)
    check_all(dec, b, "outlier keys")


@pytest.mark.parametrize("D", [64, 128])
def test_keys_a_thousand_times_larger_than_the_rest(dec, D):
    # A key whose scores dwarf all others makes any disagreement between the reference point of the exponent and the
    # scores it is applied to overflow at once (the reference point comes from a maximum over fresh MFMA results; the
    # weights from the same results a little later).  One such key in the first stage, one at a stage edge, one in the
    # middle of a later block.
    b = workload.build_prefill("pf", 8, 2, D, [100, 700], seed=11)
    k = bf16_bits_to_f32(b.k).copy()
    for t in (6, 100 + 31, 100 + 32, 100 + 300, 100 + 511):
        k[t] *= 1000.0
    b.k = workload.f32_to_bf16_bits(k)
    check_all(dec, b, "dominant keys, D=%d" % D)


def test_no_prompts_and_empty_prompts(dec):
    b = workload.build_prefill("pf", 8, 2, 64, [0, 0], seed=1)
    d = DevicePrefill(b, max_len=0)
    dec.prefill(d.c)            # nothing to do, nothing touched
    torch.cuda.synchronize()
    b = workload.build_prefill("pf", 8, 2, 64, [0, 40, 0], seed=1)
    check_all(dec, b, "empty prompts around one")


def test_bound_on_the_prompt_length_sizes_the_launch(dec):
    # a bound above the real lengths costs nothing but idle workgroups; one below them leaves the tail of a prompt
    # untouched (whole blocks of 256 query rows), and what is computed is still right
    b = workload.build_prefill("pf", 8, 2, 128, [300, 40], seed=2)
    ref_out, ref_lse = oracle.prefill(b.q, b.k, b.v, b.cu_seqlens, b.softmax_scale)
    d = DevicePrefill(b, max_len=2000)
    dec.prefill(d.c)
    compare(*d.results(), ref_out, ref_lse, "generous bound")
    d = DevicePrefill(b, max_len=200)
    dec.prefill(d.c)
    out, lse = d.results()
    compare(out[:256], lse[:256], ref_out[:256], ref_lse[:256], "first block of the long prompt")
    compare(out[300:], lse[300:], ref_out[300:], ref_lse[300:], "the short prompt")
    assert np.isnan(out[256:300]).all() and np.isnan(lse[256:300]).all()


def test_benchmark_size_whole_prompts(dec):
    # the launch bench.py times (32 prompts of 512, 7B head shape); three prompts in full against the oracle
    b = workload.make_prefill("grpo7b", seed=0)
    d = DevicePrefill(b)
    dec.prefill(d.c)
    out, lse = d.results()
    assert np.isfinite(out).all() and np.isfinite(lse).all()
    for g in (0, 13, 31):
        a, e = int(b.cu_seqlens[g]), int(b.cu_seqlens[g + 1])
        cu = np.array([0, e - a], dtype=np.int32)
        ref_out, ref_lse = oracle.prefill(b.q[a:e], b.k[a:e], b.v[a:e], cu, b.softmax_scale)
        compare(out[a:e], lse[a:e], ref_out, ref_lse, "grpo7b prompt %d" % g)


@pytest.mark.parametrize("config,groups", [("tail32b", 64), ("stream72b", 16)])
def test_benchmark_size_sampled_heads(dec, config, groups):
    # full launch; the oracle takes two prompts with two query heads each (and the kv heads they use)
    b = workload.make_prefill(config, seed=0, groups=groups)
    d = DevicePrefill(b)
    dec.prefill(d.c)
    out, lse = d.results()
    assert np.isfinite(out).all() and np.isfinite(lse).all()
    G = b.Hq // b.Hkv
    for g, heads in ((1, (0, b.Hq - 1)), (groups - 1, (G, 2 * G + 1))):
        a, e = int(b.cu_seqlens[g]), int(b.cu_seqlens[g + 1])
        cu = np.array([0, e - a], dtype=np.int32)
        for h in heads:
            kv = h // G
            ref_out, ref_lse = oracle.prefill(b.q[a:e, h:h + 1], b.k[a:e, kv:kv + 1], b.v[a:e, kv:kv + 1], cu, b.softmax_scale)
            compare(out[a:e, h:h + 1], lse[a:e, h:h + 1], ref_out, ref_lse, "%s prompt %d head %d" % (config, g, h))


def expected_pools(b, kv_dtype):
    """What the cache write must leave in pools that started out as poison: the oracle's cache write
    (oracle.prefill_write, pinned on the CPU in tests/test_prefill_oracle_pins.py)."""
    shape = (b.num_pages, b.Hkv, PAGE, b.D)
    if kv_dtype == "bf16":
        kp, vp = np.full(shape, 0x7FC0, dtype=np.uint16), np.full(shape, 0x7FC0, dtype=np.uint16)
        ks = vs = None
    else:
        kp, vp = np.full(shape, 0x7F, dtype=np.uint8), np.full(shape, 0x7F, dtype=np.uint8)
        ks, vs = np.full(shape[:2], np.nan, dtype=np.float32), np.full(shape[:2], np.nan, dtype=np.float32)
    oracle.prefill_write(b.k, b.v, b.cu_seqlens, b.page_offsets, b.pages, kp, vp, ks, vs)
    return kp, vp, ks, vs


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("D", [64, 128])
def test_cache_write_is_bit_exact(dec, kv_dtype, D):
    b = workload.build_prefill("pf", 8, 2, D, [1, 16, 17, 100, 0, 260], seed=7)
    k = bf16_bits_to_f32(b.k).copy()
    k[20:36] = 0.0                    # a page of zeros: scale 1
    k[40] *= 1000.0                   # and one with a large row
    b.k = workload.f32_to_bf16_bits(k)
    d = DevicePrefill(b, kv_dtype=kv_dtype)
    dec.prefill(d.c)
    torch.cuda.synchronize()
    kp, vp, ks, vs = expected_pools(b, kv_dtype)
    view = (lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)) if kv_dtype == "bf16" else (lambda t: t.cpu().numpy())
    np.testing.assert_array_equal(view(d.k_pool), kp)
    np.testing.assert_array_equal(view(d.v_pool), vp)
    if kv_dtype != "bf16":
        np.testing.assert_array_equal(d.k_scale.cpu().numpy().view(np.uint32), ks.view(np.uint32))
        np.testing.assert_array_equal(d.v_scale.cpu().numpy().view(np.uint32), vs.view(np.uint32))
    # and the attention was computed as well
    out, lse = d.results()
    ref_out, ref_lse = oracle.prefill(b.q, b.k, b.v, b.cu_seqlens, b.softmax_scale)
    compare(out, lse, ref_out, ref_lse, "prefill with cache write")


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
def test_cache_write_into_pools_that_are_views(dec, kv_dtype):
    # K and V interleaved per page in one allocation, with room between the token rows: the write goes through the strides
    b = workload.build_prefill("pf", 8, 2, 128, [70, 33], seed=13)
    d = DevicePrefill(b, kv_dtype=kv_dtype)
    pad = 32 if kv_dtype == "bf16" else 64
    both = torch.zeros((b.num_pages, 2, b.Hkv, PAGE, b.D + pad), dtype=d.k_pool.dtype, device=DEV)
    both[..., :b.D] = torch.stack([d.k_pool, d.v_pool], dim=1)
    kp, vp = both[:, 0, :, :, :b.D], both[:, 1, :, :, :b.D]
    d.c = ra.prefill_from_tensors(d.q, d.k, d.v, d.cu, int(b.lens.max()), d.out, d.lse, float(b.softmax_scale), k_pool=kp, v_pool=vp,
                                  k_scale=d.k_scale, v_scale=d.v_scale, page_offsets=d.page_off, pages=d.pages)
    assert d.c.kv_stride_token == b.D + pad and d.c.kv_stride_page == 2 * b.Hkv * PAGE * (b.D + pad)
    dec.prefill(d.c)
    torch.cuda.synchronize()
    ek, ev, eks, evs = expected_pools(b, kv_dtype)
    view = (lambda t: t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)) if kv_dtype == "bf16" else (lambda t: t.contiguous().cpu().numpy())
    np.testing.assert_array_equal(view(kp), ek)
    np.testing.assert_array_equal(view(vp), ev)
    assert (both[..., b.D:] == 0).all()          # nothing landed between the rows
    if kv_dtype != "bf16":
        np.testing.assert_array_equal(d.k_scale.cpu().numpy().view(np.uint32), eks.view(np.uint32))
        np.testing.assert_array_equal(d.v_scale.cpu().numpy().view(np.uint32), evs.view(np.uint32))


def test_cache_write_skips_missing_and_invalid_pages(dec):
    b = workload.build_prefill("pf", 4, 2, 64, [50, 50], seed=9)
    # prompt 0 keeps only two of its four pages; prompt 1 has one page id out of range
    keep = np.concatenate([b.pages[0:2], b.pages[4:8]]).astype(np.int32)
    keep[3] = b.num_pages + 5
    b.pages = keep
    b.page_offsets = np.array([0, 2, 6], dtype=np.int32)
    d = DevicePrefill(b, kv_dtype="bf16")
    dec.prefill(d.c)
    torch.cuda.synchronize()
    kp, vp, _, _ = expected_pools(b, "bf16")
    np.testing.assert_array_equal(d.k_pool.view(torch.int16).cpu().numpy().view(np.uint16), kp)
    np.testing.assert_array_equal(d.v_pool.view(torch.int16).cpu().numpy().view(np.uint16), vp)


def test_decode_of_the_last_prompt_token_over_the_written_pages(dec):
    # prefill writes the prompts' pages; a decode step whose query is each prompt's last token over exactly those
    # pages must give that token's prefill output (both are checked against their own oracles elsewhere; here
    # the two kernels meet through the cache)
    b = workload.build_prefill("pf", 28, 4, 128, [512, 100, 333], seed=4)
    d = DevicePrefill(b, kv_dtype="bf16")
    dec.prefill(d.c)
    out, lse = d.results()
    lens = b.lens
    last = (b.cu_seqlens[1:] - 1).astype(np.int64)
    n = lens.size
    width = int(((lens + PAGE - 1) // PAGE).max())
    bt = np.full((n, width), -1, dtype=np.int32)
    for g in range(n):
        ids = b.pages[b.page_offsets[g]:b.page_offsets[g + 1]]
        bt[g, :ids.size] = ids
    q = d.q[torch.from_numpy(last).to(DEV)].contiguous()
    o2 = torch.full((n, b.Hq, b.D), float("nan"), dtype=torch.bfloat16, device=DEV)
    l2 = torch.full((n, b.Hq), float("nan"), dtype=torch.float32, device=DEV)
    prob = ra.problem_from_tensors(q, d.k_pool, d.v_pool, torch.from_numpy(bt).to(DEV), torch.from_numpy(lens.astype(np.int32)).to(DEV),
                                   o2, l2, float(b.softmax_scale))
    dec.decode(prob)
    torch.cuda.synchronize()
    dout = o2.float().cpu().numpy().astype(np.float64)
    dlse = l2.cpu().numpy().astype(np.float64)
    assert np.abs(dout - out[last]).max() <= 2 * ABS_TOL
    assert np.abs(dlse - lse[last]).max() <= 2 * LSE_TOL
    num = np.sqrt(((dout - out[last]) ** 2).sum(-1))
    den = np.sqrt((out[last] ** 2).sum(-1))
    assert (num / den).max() <= 2 * REL_TOL


def test_rejected_arguments(dec):
    b = workload.build_prefill("pf", 8, 2, 64, [40], seed=1)
    d = DevicePrefill(b)
    for field, value, status in (("Hq", 7, ra.RA_ERR_INVALID_ARG), ("D", 96, ra.RA_ERR_UNSUPPORTED), ("q", None, ra.RA_ERR_INVALID_ARG),
                                 ("softmax_scale", float("nan"), ra.RA_ERR_INVALID_ARG), ("num_prompts", -1, ra.RA_ERR_INVALID_ARG)):
        old = getattr(d.c, field)
        setattr(d.c, field, value)
        with pytest.raises(ra.RolloutAttnError) as e:
            dec.prefill(d.c)
        assert e.value.status == status, field
        setattr(d.c, field, old)
    dec.prefill(d.c)
    torch.cuda.synchronize()


def test_bounds_far_above_the_lengths_and_very_many_heads(dec):
    # the bound on the prompt length is the caller's and may be generous; heads without end share one kv head.  What the
    # launch refuses is a grid that cannot be: blocks of 256 rows (of a die), or pages of the cache, past 2^31
    b = workload.build_prefill("pf", 256, 1, 64, [70, 3], seed=4)
    ref = oracle.prefill(b.q, b.k, b.v, b.cu_seqlens, b.softmax_scale)
    d = DevicePrefill(b, max_len=1 << 20)
    dec.prefill(d.c)
    compare(*d.results(), *ref, "256 heads, a bound of a million")
    Hq = 1 << 18
    q = torch.ones((1, Hq, 128), dtype=torch.bfloat16, device=DEV)
    k, v = (torch.randn((1, 1, 128), device=DEV).to(torch.bfloat16) for _ in range(2))
    out, lse = torch.zeros_like(q), torch.zeros((1, Hq), device=DEV)
    dec.prefill(ra.prefill_from_tensors(q, k, v, torch.tensor([0, 1], dtype=torch.int32, device=DEV), 1, out, lse, 1.0))
    assert torch.equal(out, v.expand_as(out))               # one key: the weight is 1
    assert float((lse - k.double().sum()).abs().max()) < 1e-4
    d = DevicePrefill(b, max_len=(1 << 31) - 1)
    with pytest.raises(ra.RolloutAttnError):
        dec.prefill(d.c)
    b = workload.build_prefill("pf", 16, 4, 64, [3] * 8, seed=4)
    d = DevicePrefill(b, kv_dtype="bf16", max_len=1 << 30)  # 2^26 pages of each of 32 (prompt, kv head) pairs
    with pytest.raises(ra.RolloutAttnError):
        dec.prefill(d.c)
    torch.cuda.synchronize()
    assert torch.isnan(d.out.float()).all() and torch.isnan(d.k_pool.float()).all()


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("Hq,Hkv,D", [(3, 3, 128), (8, 4, 64), (12, 4, 128), (8, 2, 128), (10, 2, 64), (21, 3, 128), (16, 1, 64), (48, 6, 128)])
def test_cache_write_of_every_head_ratio(dec, kv_dtype, Hq, Hkv, D):
    # written by the attention kernel (four query heads per kv head and more, and most calls of one workgroup per block) or by the
    # copy kernel: the same bits.  Values
    # that a quantiser may treat apart: a page of zeros, signed zeros, scales far below and above the usual range,
    # magnitudes that differ by 2^40 inside a page, NaN.  (Only the pools are looked at: no output is finite here.)
    b = workload.build_prefill("pf", Hq, Hkv, D, [1, 31, 32, 33, 0, 300, 47, 129], seed=Hq + D)
    k, v = bf16_bits_to_f32(b.k).copy(), bf16_bits_to_f32(b.v).copy()
    c = b.cu_seqlens
    k[c[5]:c[5] + 16] = 0.0
    v[c[5] + 16:c[5] + 32] *= np.float32(1e-30)
    k[c[5] + 32:c[5] + 48] *= np.float32(1e33)
    v[c[5] + 48:c[5] + 64, :, ::3] *= np.float32(2.0 ** -40)
    k[c[5] + 64:c[5] + 80, :, 1::2] = -0.0
    v[c[5] + 81, :, 5] = np.nan
    v[c[6] + 46, :, 3] = 7.0
    b.k, b.v = workload.f32_to_bf16_bits(k), workload.f32_to_bf16_bits(v)
    d = DevicePrefill(b, kv_dtype=kv_dtype)
    dec.prefill(d.c)
    torch.cuda.synchronize()
    kp, vp, ks, vs = expected_pools(b, kv_dtype)
    view = (lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)) if kv_dtype == "bf16" else (lambda t: t.cpu().numpy())
    np.testing.assert_array_equal(view(d.k_pool), kp)
    np.testing.assert_array_equal(view(d.v_pool), vp)
    if kv_dtype != "bf16":
        np.testing.assert_array_equal(d.k_scale.cpu().numpy().view(np.uint32), ks.view(np.uint32))
        np.testing.assert_array_equal(d.v_scale.cpu().numpy().view(np.uint32), vs.view(np.uint32))


@pytest.mark.parametrize("Hq,Hkv,D,n,longest", [(14, 2, 64, 150, 70), (6, 3, 128, 70, 40), (16, 1, 64, 3, 700), (5, 1, 128, 1, 1000), (12, 12, 64, 17, 90),
                                                  (8, 8, 64, 70, 1100), (32, 8, 64, 16, 100), (32, 8, 64, 15, 100)])
def test_deal_of_many_and_of_few_prompts(dec, Hq, Hkv, D, n, longest):
    # every block of every prompt is taken once: more prompts than a wave has lanes, kv heads that share dies or not,
    # fewer blocks than workgroups, long prompts of unlike lengths, levels found by votes (eight of sixteen prompts) or by sums
    lens = np.random.default_rng(n).integers(0, longest + 1, size=n).tolist()
    lens[0], lens[-1] = longest, max(1, lens[-1])
    b = workload.build_prefill("pf", Hq, Hkv, D, lens, seed=n)
    check_all(dec, b, "%d prompts, Hq=%d Hkv=%d" % (n, Hq, Hkv))


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("Hq,Hkv,D,lens", [(28, 4, 128, [1]), (28, 4, 128, [33, 95]), (8, 2, 64, [31, 0, 129]), (16, 1, 64, [200]),
                                           (64, 8, 128, [100]), (4, 4, 64, [97, 5]), (5, 1, 128, [257])])
def test_calls_of_few_blocks(dec, kv_dtype, Hq, Hkv, D, lens):
    # so few that a block takes four (tile, head) units instead of eight where the library chooses, by four waves or by eight, two
    # to a unit's keys; a last block has one to three; the cache is written from the ring whatever the head ratio, and not with
    # the settings that make workgroups stay where a kv head has fewer than four query heads
    b = workload.build_prefill("pf", Hq, Hkv, D, lens, seed=Hq + len(lens))
    d = DevicePrefill(b, kv_dtype=kv_dtype)
    dec.prefill(d.c)
    compare(*d.results(), *oracle.prefill(b.q, b.k, b.v, b.cu_seqlens, b.softmax_scale), "few blocks, %s" % lens)
    kp, vp, ks, vs = expected_pools(b, kv_dtype)
    view = (lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)) if kv_dtype == "bf16" else (lambda t: t.cpu().numpy())
    np.testing.assert_array_equal(view(d.k_pool), kp)
    np.testing.assert_array_equal(view(d.v_pool), vp)
    if kv_dtype != "bf16":
        np.testing.assert_array_equal(d.k_scale.cpu().numpy().view(np.uint32), ks.view(np.uint32))
        np.testing.assert_array_equal(d.v_scale.cpu().numpy().view(np.uint32), vs.view(np.uint32))


def check_minus_infinity(dec, D, stages, n):
    """Keys of the even (0) or the odd (1) stages of 32 score -inf: they weigh nothing.  Rows with no other key, the first 32 if it
    is the even stages, have lse -inf and no finite output."""
    b = workload.build_prefill("few", 4, 1, D, [n], seed=27)
    d = DevicePrefill(b)
    off = (torch.arange(n, device=DEV) // 32) % 2 == stages
    d.q[..., 0] = 1.0
    d.k[off] = 0.0
    d.k[off, :, 0] = float("-inf")
    dec.prefill(d.c)
    torch.cuda.synchronize()
    q, k, v = d.q.double().transpose(0, 1), d.k[:, 0].double(), d.v[:, 0].double()
    s = torch.where(off[None, None, :], float("-inf"), (q @ torch.where(off[:, None], 0.0, k).t().contiguous()) * float(b.softmax_scale))
    s = s.masked_fill(torch.ones((n, n), dtype=torch.bool, device=DEV).triu(1), float("-inf"))
    ref, ref_lse = (s.softmax(-1) @ v).transpose(0, 1), torch.logsumexp(s, -1).t()
    first = 0 if stages else 32
    assert torch.isfinite(d.out[first:]).all()
    assert float((d.out[first:].double() - ref[first:]).norm() / ref[first:].norm()) < 1e-2
    assert float((d.lse[first:].double() - ref_lse[first:]).abs().max()) < 1e-3
    assert torch.isnan(d.out[:first]).all() and bool((d.lse[:first] == float("-inf")).all())


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("stages", [0, 1])
@pytest.mark.parametrize("n", [220, 300])    # where the library chooses: four waves, and two to a unit
def test_keys_that_score_minus_infinity(dec, D, stages, n):
    check_minus_infinity(dec, D, stages, n)


def test_a_row_maximum_that_keeps_growing(dec):
    # the exponent's reference point follows the row maximum from a distance: keys whose scores grow by several powers of two
    # from stage to stage, past the float range of exp if the point stayed
    b = workload.build_prefill("pf", 14, 2, 128, [640], seed=3)
    k, q = bf16_bits_to_f32(b.k).copy(), bf16_bits_to_f32(b.q).copy()
    k[:] = np.abs(k[:1]) * np.exp2(np.arange(640, dtype=np.float32) / 80.0)[:, None, None]
    q[:, ::2] = np.abs(q[:, ::2])
    b.k, b.q = workload.f32_to_bf16_bits(k), workload.f32_to_bf16_bits(q)
    check_all(dec, b, "growing scores")


def test_very_many_short_prompts_take_no_longer_than_their_data_warrants():
    """Which blocks a workgroup takes is worked out on the device from the prompts' lengths.  With 4096 prompts of a tile
    each there is next to nothing to do for a block, so a search that walks the prompts shows: 870 us against 10 for a copy
    of the queries when it did, 66 without (156 for a launch of 256-row blocks whose numbers are divided out).  The
    bound of 20 copies lies a factor of three from either."""
    n, Hq, D = 4096, 4, 64
    T = 16 * n
    q = torch.randn((T, Hq, D), device=DEV).to(torch.bfloat16)
    k, v = (torch.randn((T, 1, D), device=DEV).to(torch.bfloat16) for _ in range(2))
    out, lse = torch.empty_like(q), torch.empty((T, Hq), device=DEV)
    cu = 16 * torch.arange(n + 1, dtype=torch.int32, device=DEV)
    c = ra.prefill_from_tensors(q, k, v, cu, 16, out, lse, D ** -0.5)
    d = ra.Decoder(0)

    def us(fn, reps=20):
        best = float("inf")
        for _ in range(5):
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            fn()
            e0.record()
            for _ in range(reps):
                fn()
            e1.record()
            torch.cuda.synchronize()
            best = min(best, 1e3 * e0.elapsed_time(e1) / reps)
        return best

    copy = torch.empty_like(q)
    t, tc = us(lambda: d.prefill(c)), us(lambda: copy.copy_(q))
    print("prefill %.1f us, copy of the queries %.1f us" % (t, tc), flush=True)
    for g in (0, 1, 1000, n - 1):                      # the answer, at the ends and in between
        a = slice(16 * g, 16 * g + 16)
        s = (q[a].double().transpose(0, 1) @ k[a, 0].double().t()) * D ** -0.5
        s = s.masked_fill(torch.ones((16, 16), dtype=torch.bool, device=DEV).triu(1), float("-inf"))
        ref = (s.softmax(-1) @ v[a, 0].double()).transpose(0, 1)
        assert float((out[a].double() - ref).norm() / ref.norm()) < REL_TOL
    assert t < 20 * tc, (t, tc)
    d.close()
