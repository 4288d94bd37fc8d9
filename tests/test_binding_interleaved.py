"""The binding's workspace while it grows: a decode call that another one cuts into, at every bytecode of the first, never
gives the library an address of one workspace with the size of another.  The library and the device are stand-ins, so this
runs anywhere."""
import sys

import pytest
import torch

from paper_2507_01663_amd import binding


class Stream:
    cuda_stream = 7


class Library:
    """Notes what it is given; knows the size of every tensor that was made."""

    def __init__(self):
        self.sizes = {}
        self.calls = []

    def rollout_attn_create(self, out, device):
        return binding.RA_OK

    def rollout_attn_destroy(self, ctx):
        pass

    def rollout_attn_last_error(self, ctx):
        return b""

    def rollout_attn_workspace_size(self, ctx, problem, out):
        out._obj.value = problem._obj.B
        return binding.RA_OK

    def rollout_attn_decode(self, ctx, problem, workspace, size, stream):
        problem = getattr(problem, "_obj", problem)
        at = getattr(workspace, "value", workspace)
        self.calls.append((at, size))
        assert size <= self.sizes[at], "an address with the size of another workspace"
        return binding.RA_OK if problem.B <= size else binding.RA_ERR_WORKSPACE_TOO_SMALL


@pytest.fixture
def lib(monkeypatch):
    lib, empty, kept = Library(), torch.empty, []

    def make(n, dtype, device):
        t = empty(n, dtype=dtype)
        kept.append(t)                       # (no address comes twice)
        lib.sizes[t.data_ptr()] = n
        return t

    monkeypatch.setattr(binding, "load_library", lambda: lib)
    monkeypatch.setattr(torch, "empty", make)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    return lib


def problem(n):
    p = binding.ra_problem()
    p.B = n                                  # the stand-in's workspace: a byte per sequence
    return p


def cut_in(outer, inner, functions, at):
    """Runs outer(), and inner() before the at-th bytecode that outer executes in these functions; whether there is one."""
    codes, seen, busy = [f.__code__ for f in functions], [0], [False]

    def trace(frame, event, arg):
        if busy[0] or frame.f_code not in codes:
            return None
        frame.f_trace_opcodes = True
        if event == "opcode":
            if seen[0] == at:
                busy[0] = True
                inner()
                busy[0] = False
            seen[0] += 1
        return trace

    old = sys.gettrace()
    sys.settrace(trace)
    try:
        outer()
    finally:
        sys.settrace(old)
    return seen[0] > at


@pytest.mark.parametrize("first,outer,inner", [(100, 100, 5000), (100, 5000, 50), (None, 100, 5000)])
def test_no_mixed_workspace(lib, first, outer, inner):
    functions = [binding.Decoder.decode]
    if inner < outer:                        # (one that grows must not cut into another's growth: callers order those)
        functions.append(binding.Decoder.workspace)
    at = 0
    while True:
        d = binding.Decoder(0)
        if first is not None:
            d.decode(problem(first), Stream)
        if not cut_in(lambda: d.decode(problem(outer), Stream), lambda: d.decode(problem(inner), Stream), functions, at):
            break
        assert lib.calls[-1][1] >= min(outer, inner)
        d.close()
        at += 1
    assert at > 10
