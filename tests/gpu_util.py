"""Helpers for the GPU tests: upload a workload.Problem, run the HIP library through its C ABI, compare."""
import ctypes
import os

import numpy as np

import paper_2507_01663_amd as ra
from paper_2507_01663_amd.torch_util import DeviceProblem, bits_to_bf16  # noqa: F401  (the tests import them from here)

ABS_TOL = 1e-2      # max |out_gpu - out_ref| over all elements
REL_TOL = 1e-2      # per (b, h) row: ||out_gpu - out_ref||_2 / ||out_ref||_2
LSE_TOL = 1e-3      # |lse_gpu - lse_ref|


def context(**env):
    """A Decoder made with these environment settings (they are read when the context is made, and nowhere else)."""
    names = {k: "ROLLOUT_ATTN_" + k for k in env}
    old = {k: os.environ.get(n) for k, n in names.items()}
    for k, n in names.items():
        os.environ[n] = str(env[k])
    try:
        d = ra.Decoder(0)
    finally:
        for k, n in names.items():
            if old[k] is None:
                os.environ.pop(n, None)
            else:
                os.environ[n] = old[k]
    d.settings = dict(env)
    return d


class DirectPlan(ctypes.Structure):
    """How a batch goes without a schedule: workgroups per (sequence, kv head) (0: it has a schedule), waves of a workgroup,
    whether the longest sequences come first, whether the workgroups are turned about over the dies."""
    _fields_ = [(n, ctypes.c_int32) for n in ("splits", "waves", "sorted", "turned")]

    def __iter__(self):
        return iter((self.splits, self.waves, self.sorted, self.turned))


def direct_plan(B, Hkv, G, D, fp8, max_pages, share, cus, waves):
    """The library's own rule; it is no entry point of the C ABI, so it is called by the name the compiler gave it."""
    f = ra.load_library()._ZN2ra11direct_planEiiiiiiiii
    f.restype = DirectPlan
    return f(B, Hkv, G, D, int(fp8), max_pages, int(share), cus, waves)


def plan_of(dec, p, use_hint=True):
    """What the library does with a decode step of this problem: a DirectPlan."""
    if str(getattr(dec, "settings", {}).get("DIRECT", 1)) == "0":
        return DirectPlan()
    import torch
    fp8 = p.kv_dtype != "bf16"
    waves = ra.rollout_attn_wave_count(dec.ctx, ra.RA_KV_FP8_E4M3 if fp8 else ra.RA_KV_BF16, p.D)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    share = use_hint and p.prefix_page_offsets.size > 1      # (a hint is used if it names groups, whatever they share)
    return direct_plan(p.B, p.Hkv, p.Hq // p.Hkv, p.D, fp8, p.block_table.shape[1], share, cus, waves)


def scheduled(dec, p, use_hint=True):
    """Whether a decode step of this problem has a schedule."""
    return plan_of(dec, p, use_hint).splits == 0


def compare(out, lse, ref_out, ref_lse, what="", abs_rel=0.0):
    """Asserts the three tolerances; returns the measured errors.  abs_rel widens the element-wise bound to
    ABS_TOL + abs_rel * |ref| for outputs that are not small: rounding the exact result to bf16 alone moves an
    element by up to 2**-9 of its magnitude, which passes ABS_TOL once |ref| > 5 (prompt prefill: the first tokens of a
    prompt average over few values; a decode step averages over hundreds and never gets there)."""
    assert np.isfinite(out).all(), what + ": non-finite output"
    empty = np.isneginf(ref_lse)
    assert (np.isneginf(lse) == empty).all(), what + ": -inf pattern of lse differs"
    d = out - ref_out
    abs_err = float(np.abs(d).max()) if d.size else 0.0
    num = np.sqrt((d * d).sum(axis=-1))
    den = np.sqrt((ref_out * ref_out).sum(axis=-1))
    rel = np.where(den > 0, num / np.maximum(den, 1e-300), num)
    rel_err = float(rel.max()) if rel.size else 0.0
    lse_err = float(np.abs(lse[~empty] - ref_lse[~empty]).max()) if (~empty).any() else 0.0
    excess = float((np.abs(d) - abs_rel * np.abs(ref_out)).max()) if d.size else 0.0
    assert excess <= ABS_TOL, "%s: max abs err %.3e (%.3e beyond the magnitude allowance)" % (what, abs_err, excess)
    assert rel_err <= REL_TOL, "%s: max row rel err %.3e" % (what, rel_err)
    assert lse_err <= LSE_TOL, "%s: max lse err %.3e" % (what, lse_err)
    return abs_err, rel_err, lse_err
