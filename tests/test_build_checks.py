"""Checks on the generated gfx950 code that the kernels' hand-managed pieces rely on (CPU only: hipcc
cross-compiles to assembly, nothing runs)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def isa(tmp_path_factory):
    from paper_2507_01663_amd import build
    out = tmp_path_factory.mktemp("isa") / "ra_kernels.s"
    flags = [f for f in build.flags_for("ra_kernels.hip") if f != "-fPIC"]
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["-S", "--cuda-device-only", "-o", str(out),
                                                                       os.path.join(build.CSRC, "ra_kernels.hip")]
    subprocess.run(cmd, check=True, stderr=subprocess.DEVNULL)
    return open(out).read()


def kernels(isa):
    """name -> body text of every attention kernel."""
    out = {}
    for m in re.finditer(r"^(_ZN2ra\d+attention_kernel\w+):.*?s_endpgm", isa, flags=re.S | re.M):
        out[m.group(1)] = m.group(0)
    return out


def descriptors(isa, prefix):
    """name -> (vector registers, scratch bytes) from each kernel's own descriptor."""
    out = {}
    for m in re.finditer(r"\.amdhsa_kernel (%s\w+)\n(.*?)\.end_amdhsa_kernel" % prefix, isa, flags=re.S):
        regs = int(re.search(r"\.amdhsa_next_free_vgpr (\d+)", m.group(2)).group(1))
        scratch = int(re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", m.group(2)).group(1))
        out[m.group(1)] = (regs, scratch)
    return out


def test_no_scratch_and_no_full_drain_in_the_page_loop(isa):
    desc = descriptors(isa, r"_ZN2ra\d+attention_kernel")
    bodies = kernels(isa)
    # bf16 and e4m3 pools, two ring depths, two head dims, with and without the planning pass
    assert len(bodies) == 16 and set(desc) == set(bodies)
    for name, body in bodies.items():
        regs, scratch = desc[name]
        assert scratch == 0 and regs <= 512, (name, regs, scratch)
        assert "scratch_" not in body, name
        # the LDS ring is paced by hand-written waits with a non-zero count; they must be there
        assert re.search(r"s_waitcnt vmcnt\([1-9][0-9]*\)", body), name


def test_streaming_probe_is_one_flat_kernel(isa):
    """The probe's figure is reported as the ceiling the attention kernel is judged against: its loads must be the ring's
    direct global-to-LDS loads, with nothing called and nothing on the stack."""
    m = re.search(r"^(_ZN2ra19stream_probe_kernel\w+):(.*?)s_endpgm", isa, flags=re.S | re.M)
    body = m.group(2)
    assert body.count("global_load_lds_dwordx4") >= 32 and "s_swappc" not in body and "scratch_" not in body
    assert descriptors(isa, r"_ZN2ra19stream_probe_kernel")[m.group(1)][1] == 0


def test_e4m3_kernels_fit_two_waves_per_simd(isa):
    """The e4m3 decode kernels are scheduled for two waves on a SIMD (six workgroups per compute unit at head dim
    128): that holds only while they stay within half of the 512 registers a lane has, without scratch."""
    desc = descriptors(isa, r"_ZN2ra\d+attention_kernel_fp8")
    assert len(desc) == 8    # two ring depths, two head dims, with and without the planning pass
    for name, (regs, scratch) in desc.items():
        assert regs <= 256 and scratch == 0, (name, regs, scratch)


def test_steps_without_a_schedule_look_up_pages_one_by_one(isa):
    """A table row may end with the sequence's last page in use: entries are looked up as the pages exist, by scalar loads behind the
    length, and never as a row of lanes.  The only vector loads into registers are those of the lengths that a wave sorts, 64 each."""
    found = re.findall(r"^_ZN2ra\d+direct_kernelILi\d+ELi\d+ELi\d+ELb([01])E\w+:(.*?)s_endpgm", isa, flags=re.S | re.M)
    assert len(found) == 14                                  # seven shapes, as they come and the longest first
    for order, body in found:
        before = body[:body.index("s_barrier")]              # (behind it the waves' partials)
        assert len(re.findall(r"(?:global|flat)_load_(?!lds)\w+ v", before)) == (8 if order == "1" else 0)


# Registers that the designed occupancy leaves a lane: workgroups of eight waves are two waves to a SIMD; of those of four, two share
# a compute unit at head dim 128 (two waves to a SIMD) and three at head dim 64, as their LDS lets in.
@pytest.mark.parametrize("source,kernels,unscratched,registers", [
    ("ra_prefill.hip", 4, 6, {64: 256, 128: 256}),           # workgroups that stay and two waves to a unit's keys, D = 64 and 128; the cache write
    ("ra_prefill_four.hip", 4, 4, {64: 168, 128: 256}),      # workgroups of four waves, levels by sums and by votes
])
def test_prefill_kernels_keep_their_accumulators_in_registers(source, kernels, unscratched, registers):
    import tempfile
    from paper_2507_01663_amd import build
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, source + ".s")
        flags = [f for f in build.flags_for(source) if f != "-fPIC"]
        subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["-S", "--cuda-device-only", "-o", out,
                                                                                  os.path.join(build.CSRC, source)],
                       check=True, stderr=subprocess.DEVNULL)
        text = open(out).read()
    found = re.findall(r"^(_ZN2ra14prefill_kernel\w+):.*?s_endpgm", text, flags=re.S | re.M)
    assert len(found) == kernels
    for m in re.finditer(r"^(_ZN2ra14prefill_kernel\w+):(.*?)s_endpgm", text, flags=re.S | re.M):
        assert "scratch_" not in m.group(2), m.group(1)
        assert "v_mfma_f32_32x32x16_bf16" in m.group(2), m.group(1)
        assert re.search(r"s_waitcnt vmcnt\([1-9][0-9]*\)", m.group(2)), m.group(1)
    assert text.count(".private_segment_fixed_size: 0") == unscratched
    desc = descriptors(text, r"_ZN2ra14prefill_kernel")
    assert len(desc) == kernels
    for name, (regs, scratch) in desc.items():
        assert scratch == 0 and regs <= registers[int(re.search(r"kernelILi(\d+)E", name).group(1))], (name, regs, scratch)
