"""Measured cases of the library: what a rollout worker asks of it, through the binding's public calls.

A rollout worker prefills each prompt once and writes its K and V rows into pages, appends one token per sequence and
layer in every decode iteration, and runs the decode attention of that iteration, layer after layer.  The cases below are
those calls at the sizes of this repository's workloads (workload/gen.py: "tiny", "grpo7b", "tail32b", "stream72b" and
their head shapes) and at generic ones between and beside them: a handful of short sequences, the stragglers that a long
tailed batch ends with, ragged prompts, a large batch of a small model.

Lengths belong to the case (they come from its "length_seed"); values, page placement and queries come from the seed.
"""
import math
import random

import numpy as np
import torch

import paper_2507_01663_amd as ra

PAGE = 16
DEV = "cuda:0"
SLACK = 1.25                 # pages of a pool per page in use, as a serving cache has spare pages

_decoder = None


def decoder():
    """The process's one decoder (a context and its workspace), as a worker keeps it."""
    global _decoder
    if _decoder is None:
        _decoder = ra.Decoder(0)
    return _decoder


# ---- the cases ----------------------------------------------------------------------------------------

def _decode(name, Hq, Hkv, D, prompts, samples, prompt, law, resp, kv, layers=1, length_seed=0):
    return {"name": name, "kind": "decode", "Hq": Hq, "Hkv": Hkv, "D": D, "prompts": prompts, "samples": samples, "prompt": prompt,
            "law": law, "resp": resp, "kv": kv, "layers": layers, "length_seed": length_seed}


def _prefill(name, Hq, Hkv, D, prompts, shortest, longest, kv, length_seed=0):
    return {"name": name, "kind": "prefill", "Hq": Hq, "Hkv": Hkv, "D": D, "prompts": prompts, "shortest": shortest, "longest": longest,
            "kv": kv, "length_seed": length_seed}


def listed():
    return [
        # one prompt, four short responses of a small model: a smoke run, an evaluation prompt; all latency
        _decode("decode_tiny", 4, 2, 64, 1, 4, 16, "uniform", 240, "bf16"),
        # one GRPO group in flight on its own: the first prompt of a batch, or an interactive session (prompt not a
        # multiple of a page)
        _decode("decode_one_group", 28, 4, 128, 1, 8, 501, "uniform", 1500, "bf16"),
        # what is left of a long-tailed batch when all but a few sequences have finished: every one long
        _decode("decode_stragglers", 40, 8, 128, 3, 2, 1024, "late", 15000, "bf16"),
        # the 7B-shaped GRPO batch in full flight, the headline workload, with either cache type
        _decode("decode_grpo7b", 28, 4, 128, 32, 8, 512, "uniform", 3584, "bf16"),
        _decode("decode_grpo7b_e4m3", 28, 4, 128, 32, 8, 512, "uniform", 3584, "e4m3"),
        # the 32B-shaped long-tailed batch: the largest decode step of the usual run
        _decode("decode_tail32b", 40, 8, 128, 64, 8, 1024, "lognormal", 16384, "bf16"),
        # a large batch of a small model: more sequences than the attention waves schedule by themselves
        _decode("decode_wide_d64_e4m3", 8, 2, 64, 128, 8, 250, "uniform", 1030, "e4m3"),
        # four consecutive layers of one decode iteration of a mid-sized batch: one schedule, reused by the other layers
        _decode("decode_layers", 28, 4, 128, 8, 8, 300, "uniform", 1200, "bf16", layers=4),
        # the cache write of a decode iteration with a quantised cache
        {"name": "append_e4m3", "kind": "append", "Hq": 40, "Hkv": 8, "D": 128, "batch": 512, "longest": 60, "kv": "e4m3", "length_seed": 0},
        # a few prompts of all lengths arriving together
        _prefill("prefill_ragged", 28, 4, 128, 8, 37, 701, "bf16"),
        # the prompts of the 7B-shaped GRPO batch
        _prefill("prefill_grpo7b", 28, 4, 128, 32, 512, 512, "bf16"),
        # the prompts of the 72B-shaped batch, into a quantised cache: the largest prefill
        _prefill("prefill_stream72b_e4m3", 64, 8, 128, 16, 2048, 2048, "e4m3"),
    ]


HEADS = [(4, 2, 64), (8, 2, 64), (32, 2, 64), (28, 4, 128), (40, 8, 128), (64, 8, 128), (8, 8, 128)]


def _spread(rng, lo, hi):
    """An integer of lo .. hi, spread evenly over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "decode", "prefill", "prefill", "prefill", "append"])
    while True:
        Hq, Hkv, D = rng.choice(HEADS)
        kv = rng.choice(["bf16", "e4m3"])
        length_seed = rng.randrange(1 << 30)
        if kind == "decode":
            c = _decode("", Hq, Hkv, D, _spread(rng, 1, 160), rng.choice([1, 2, 4, 5, 8, 16]), rng.choice([0, _spread(rng, 8, 2048)]),
                        rng.choice(["uniform", "uniform", "late", "lognormal"]), _spread(rng, 16, 16384), kv,
                        layers=rng.choice([1, 1, 1, 2, 3]), length_seed=length_seed)
            ok = c["prompts"] * c["samples"] <= 1100 and work(c)["bytes"] <= 5.5e9
        elif kind == "prefill":
            longest = _spread(rng, 8, 2048)
            c = _prefill("", Hq, Hkv, D, _spread(rng, 1, 64), rng.randint(1, longest), longest, kv, length_seed=length_seed)
            ok = work(c)["flops"] <= 1.0e12 and work(c)["bytes"] <= 2.0e9
        else:
            c = {"name": "", "kind": "append", "Hq": Hq, "Hkv": Hkv, "D": D, "batch": _spread(rng, 1, 1000), "longest": _spread(rng, 4, 400),
                 "kv": kv, "length_seed": length_seed}
            ok = c["batch"] * c["longest"] * Hkv * D <= 1 << 27
        if ok:
            del c["name"]
            return c


# ---- lengths ------------------------------------------------------------------------------------------

def _response_lengths(case):
    r, n, top = random.Random(case["length_seed"]), case["prompts"] * case["samples"], case["resp"]
    if case["law"] == "uniform":
        return [r.randint(0, top) for _ in range(n)]
    if case["law"] == "late":           # all of them far along
        return [r.randint(top // 2, top) for _ in range(n)]
    # long-tailed: the median an eighth of the cap
    return [min(top, int(round(math.exp(r.gauss(math.log(max(1.0, top / 8)), 0.8))))) for _ in range(n)]


def _prompt_lengths(case):
    r = random.Random(case["length_seed"])
    return [r.randint(case["shortest"], case["longest"]) for _ in range(case["prompts"])]


def _append_lengths(case):
    r = random.Random(case["length_seed"])
    return [r.randint(0, case["longest"]) for _ in range(case["batch"])]


def _pages(n):
    return (n + PAGE - 1) // PAGE


# ---- what the path cannot do without ------------------------------------------------------------------

def work(case):
    Hq, Hkv, D = case["Hq"], case["Hkv"], case["D"]
    e = 1 if case["kv"] == "e4m3" else 2
    if case["kind"] == "decode":
        resp = _response_lengths(case)
        shared = case["prompt"] // PAGE * PAGE if case["samples"] > 1 else 0
        lens = [case["prompt"] + x for x in resp]
        kv_tokens = (case["prompts"] * shared) + sum(n - shared for n in lens)
        step = 2 * kv_tokens * Hkv * D * e + 2 * len(lens) * Hq * D * 2 + 4 * len(lens) * Hq
        if e == 1:
            step += 8 * Hkv * (case["prompts"] * (shared // PAGE) + sum(_pages(n) - shared // PAGE for n in lens))
        tables = 4 * sum(_pages(n) for n in lens) + 4 * len(lens)
        return {"bytes": case["layers"] * step + tables, "flops": case["layers"] * 4 * D * Hq * sum(lens)}
    if case["kind"] == "prefill":
        lens = _prompt_lengths(case)
        T = sum(lens)
        size = 2 * T * Hq * D * 2 + 4 * T * Hq + 2 * T * Hkv * D * (2 + e) + 4 * sum(_pages(n) for n in lens)
        if e == 1:
            size += 8 * Hkv * sum(_pages(n) for n in lens)
        return {"bytes": size, "flops": 4 * D * Hq * sum(n * (n + 1) // 2 for n in lens)}
    n = case["batch"]
    return {"bytes": n * (2 * Hkv * D * (2 + e) + (16 * Hkv if e == 1 else 0) + 8), "flops": 0}


# ---- inputs -------------------------------------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _normal(shape, g):
    return torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(generator=g)


def _pool(pages, Hkv, D, kv, g):
    """A pool of normal values: bf16, or E4M3 codes with one scale per (page, kv head)."""
    if kv == "bf16":
        return _normal((pages, Hkv, PAGE, D), g), None
    codes = torch.empty((pages, Hkv, PAGE, D), dtype=torch.uint8, device=DEV)
    scale = torch.empty((pages, Hkv), dtype=torch.float32, device=DEV)
    for a in range(0, pages, 1 << 14):
        x = _normal((min(pages - a, 1 << 14), Hkv, PAGE, D), g).float()
        s = x.abs().amax(dim=(2, 3)) / 448.0
        codes[a:a + x.shape[0]] = (x / s[:, :, None, None]).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
        scale[a:a + x.shape[0]] = s
    return codes, scale


def _placement(pages_used, g):
    """(physical page of every logical one, pages in the pool)."""
    total = max(pages_used + 1, int(math.ceil(SLACK * pages_used)))
    return torch.randperm(total, generator=g, device=DEV)[:pages_used].to(torch.int32).cpu().numpy(), total


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _scale(D):
    return float(np.float32(1.0 / math.sqrt(D)))


def _prepare_decode(case, seed):
    g = _generator(seed)
    Hq, Hkv, D, R, n = case["Hq"], case["Hkv"], case["D"], case["samples"], case["prompts"]
    resp = _response_lengths(case)
    B = n * R
    lens = np.array([case["prompt"] + x for x in resp], dtype=np.int64)
    shared = case["prompt"] // PAGE if R > 1 else 0
    pages = (lens + PAGE - 1) // PAGE
    phys, total = _placement(int(n * shared + (pages - shared).sum()), g)
    prefix = phys[:n * shared].reshape(n, shared)
    table = np.full((B, max(1, int(pages.max()))), -1, dtype=np.int32)
    at = n * shared
    for b in range(B):
        own = int(pages[b]) - shared
        table[b, :shared] = prefix[b // R]
        table[b, shared:shared + own] = phys[at:at + own]
        at += own
    st = {"decoder": decoder(), "lens": lens, "table": _dev(table), "seq_lens": _dev(lens.astype(np.int32)), "layers": []}
    hint = {}
    if shared:
        hint = {"seq_group": _dev(np.repeat(np.arange(n, dtype=np.int32), R)),
                "prefix_page_offsets": _dev(np.arange(n + 1, dtype=np.int32) * shared), "prefix_pages": _dev(prefix.reshape(-1))}
    st["hint"] = hint
    for i in range(case["layers"]):
        kp, ks = _pool(total, Hkv, D, case["kv"], g)
        vp, vs = _pool(total, Hkv, D, case["kv"], g)
        y = {"k": kp, "v": vp, "ks": ks, "vs": vs, "q": _normal((B, Hq, D), g),
             "out": torch.empty((B, Hq, D), dtype=torch.bfloat16, device=DEV), "lse": torch.empty((B, Hq), dtype=torch.float32, device=DEV)}
        y["call"] = ra.problem_from_tensors(y["q"], kp, vp, st["table"], st["seq_lens"], y["out"], y["lse"], _scale(D), k_scale=ks, v_scale=vs,
                                            flags=ra.RA_FLAG_REUSE_SCHEDULE if i else 0, **hint)
        st["layers"].append(y)
    return st


def _prepare_prefill(case, seed):
    g = _generator(seed)
    Hq, Hkv, D = case["Hq"], case["Hkv"], case["D"]
    lens = np.array(_prompt_lengths(case), dtype=np.int64)
    T = int(lens.sum())
    npg = (lens + PAGE - 1) // PAGE
    phys, total = _placement(int(npg.sum()), g)
    cu, off = np.zeros(lens.size + 1, dtype=np.int32), np.zeros(lens.size + 1, dtype=np.int32)
    cu[1:], off[1:] = np.cumsum(lens), np.cumsum(npg)
    st = {"decoder": decoder(), "lens": lens, "cu": _dev(cu), "off": _dev(off), "pages": _dev(phys), "phys": phys,
          "q": _normal((T, Hq, D), g), "k": _normal((T, Hkv, D), g), "v": _normal((T, Hkv, D), g),
          "out": torch.empty((T, Hq, D), dtype=torch.bfloat16, device=DEV), "lse": torch.empty((T, Hq), dtype=torch.float32, device=DEV),
          "ks": None, "vs": None}
    kind = torch.bfloat16 if case["kv"] == "bf16" else torch.uint8
    st["kp"], st["vp"] = (torch.zeros((total, Hkv, PAGE, D), dtype=kind, device=DEV) for _ in range(2))
    if case["kv"] != "bf16":
        st["ks"], st["vs"] = (torch.zeros((total, Hkv), dtype=torch.float32, device=DEV) for _ in range(2))
    st["call"] = ra.prefill_from_tensors(st["q"], st["k"], st["v"], st["cu"], int(lens.max()), st["out"], st["lse"], _scale(D), k_pool=st["kp"],
                                         v_pool=st["vp"], k_scale=st["ks"], v_scale=st["vs"], page_offsets=st["off"], pages=st["pages"])
    return st


def _prepare_append(case, seed):
    g = _generator(seed)
    Hq, Hkv, D, B = case["Hq"], case["Hkv"], case["D"], case["batch"]
    lens = np.array(_append_lengths(case), dtype=np.int64)
    npg = lens // PAGE + 1                      # the new token's page is in the table
    phys, total = _placement(int(npg.sum()), g)
    table = np.full((B, int(npg.max())), -1, dtype=np.int32)
    at = 0
    for b in range(B):
        table[b, :npg[b]] = phys[at:at + npg[b]]
        at += int(npg[b])
    st = {"decoder": decoder(), "table": _dev(table), "seq_lens": _dev(lens.astype(np.int32))}
    st["k"], st["ks"] = _pool(total, Hkv, D, case["kv"], g)
    st["v"], st["vs"] = _pool(total, Hkv, D, case["kv"], g)
    st["k_new"], st["v_new"] = _normal((B, Hkv, D), g), _normal((B, Hkv, D), g)
    st["q"] = torch.zeros((B, Hq, D), dtype=torch.bfloat16, device=DEV)
    st["out"], st["lse"] = torch.empty_like(st["q"]), torch.empty((B, Hq), dtype=torch.float32, device=DEV)
    st["call"] = ra.problem_from_tensors(st["q"], st["k"], st["v"], st["table"], st["seq_lens"], st["out"], st["lse"], _scale(D),
                                         k_scale=st["ks"], v_scale=st["vs"])
    return st


def prepare(case, seed):
    st = {"decode": _prepare_decode, "prefill": _prepare_prefill, "append": _prepare_append}[case["kind"]](case, seed)
    st["kind"] = case["kind"]
    return st


# ---- one pass -----------------------------------------------------------------------------------------

def run(state):
    d = state["decoder"]
    if state["kind"] == "decode":
        for y in state["layers"]:
            d.decode(y["call"])
        return {"out": [y["out"] for y in state["layers"]], "lse": [y["lse"] for y in state["layers"]]}
    if state["kind"] == "prefill":
        d.prefill(state["call"])
        return {"out": state["out"], "lse": state["lse"], "k_pool": state["kp"], "v_pool": state["vp"], "k_scale": state["ks"],
                "v_scale": state["vs"]}
    d.append(state["call"], state["k_new"], state["v_new"])
    return {"k_pool": state["k"], "v_pool": state["v"], "k_scale": state["ks"], "v_scale": state["vs"]}


# ---- the same in 64 bits ------------------------------------------------------------------------------

def _attend(q, k, v, scale, causal):
    """q [T, Hq, D], k and v [S, Hkv, D] in 64 bits; causal: T == S.  (out [T, Hq, D], lse [T, Hq])"""
    T, Hq, D = q.shape
    S, Hkv, G = k.shape[0], k.shape[1], Hq // k.shape[1]
    out, lse = torch.empty_like(q), torch.empty((T, Hq), dtype=q.dtype, device=q.device)
    for h in range(Hkv):
        s = (q[:, h * G:(h + 1) * G].reshape(T * G, D) @ k[:, h].t().contiguous()).mul_(scale).view(T, G, S)
        if causal:
            s.masked_fill_(torch.ones((T, S), dtype=torch.bool, device=q.device).triu_(1)[:, None, :], float("-inf"))
        m = s.amax(dim=-1, keepdim=True)
        p = s.sub_(m).exp_()
        z = p.sum(dim=-1, keepdim=True)
        out[:, h * G:(h + 1) * G] = (p.view(T * G, S) @ v[:, h].contiguous()).view(T, G, D) / z
        lse[:, h * G:(h + 1) * G] = (m + z.log()).squeeze(-1)
    return out, lse


def _values(pool, scale, ids, n):
    """The first n tokens of the pages `ids`, [n, Hkv, D] in 64 bits."""
    x = pool[ids]
    if scale is None:
        x = x.double()
    else:
        x = x.view(torch.float8_e4m3fn).float().double() * scale[ids].double()[:, :, None, None]
    return x.transpose(1, 2).reshape(-1, x.shape[1], x.shape[3])[:n]


def exact(case, seed):
    if case["kind"] == "append":
        return None                     # codes and copied bits: compared byte for byte
    st = prepare(case, seed)
    scale = _scale(case["D"])
    if case["kind"] == "decode":
        outs, lses = [], []
        for y in st["layers"]:
            out, lse = y["q"].double(), torch.full(y["lse"].shape, float("-inf"), dtype=torch.float64, device=DEV)
            out.zero_()
            for b, n in enumerate(st["lens"].tolist()):
                if n:
                    ids = st["table"][b, :_pages(n)].long()
                    o, z = _attend(y["q"][b:b + 1].double(), _values(y["k"], y["ks"], ids, n), _values(y["v"], y["vs"], ids, n), scale, False)
                    out[b], lse[b] = o[0], z[0]
            outs.append(out)
            lses.append(lse)
        return {"out": outs, "lse": lses}
    out, lse = torch.empty(st["out"].shape, dtype=torch.float64, device=DEV), torch.empty(st["lse"].shape, dtype=torch.float64, device=DEV)
    a = 0
    for n in st["lens"].tolist():
        out[a:a + n], lse[a:a + n] = _attend(st["q"][a:a + n].double(), st["k"][a:a + n].double(), st["v"][a:a + n].double(), scale, True)
        a += n
    return {"out": out, "lse": lse, "k_pool": None, "v_pool": None, "k_scale": None, "v_scale": None}


def tolerance(case):
    if case["kind"] == "append":
        return "exact"
    # Inputs are exact in bf16 (or as codes and scales), scores and sums are fp32, the weights are rounded to bf16 before
    # the second product and the result once more.  Measured against exact(): relative errors of 1.5e-3 to 2.4e-3, largest
    # differences of up to 1.4e-2 (decode) and 4.0e-2 (prefill, whose outputs grow smaller along a prompt); four times that.
    return {"rel": 1e-2, "max": 0.16 if case["kind"] == "prefill" else 0.055}
