"""The sampling entry points that return host results wait for the device the call ran on before they read its results: the
current device, which need not be the one that the tensors, and with them the stream of a copy to the host, belong to.  (The
tensors here are the CPU's, so another device than theirs is current.)"""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2503_00784_amd import binding


class _FakeLibrary:
    """Stands in for the compiled library: notes the call, touches nothing."""

    def __init__(self, events):
        self.events = events

    def duo_sample_workspace_bytes(self, vocab, n, k, out):
        C.cast(out, C.POINTER(C.c_size_t)).contents.value = 256
        return 0

    def duo_spec_sample(self, *a):
        self.events.append("call")
        return 0

    def duo_spec_sample_noalloc(self, *a):
        self.events.append("call")
        return 0

    def duo_deferred_sample(self, *a):
        self.events.append("call")
        return 0


@pytest.fixture()
def events(monkeypatch):
    seen = []
    fetch = binding._Results.fetch

    def noted(self, n):
        seen.append("fetch")
        return fetch(self, n)

    monkeypatch.setattr(binding, "load", lambda dtype="bf16": _FakeLibrary(seen))
    monkeypatch.setattr(binding, "_stream_ptr", lambda: 0)
    monkeypatch.setattr(binding._Results, "fetch", noted)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 1)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda device=None: seen.append("wait" if device is None else f"wait {device}"))
    return seen


def _inputs():
    V, n, k = 16, 2, 3
    return (torch.zeros(n * k, V), torch.zeros(V), torch.zeros((n, k), dtype=torch.int32), torch.full((n, k, V), 1.0 / V),
            torch.zeros((n, k + 1)))


def test_spec_sample_waits_for_the_current_device(events):
    got = binding.spec_sample(*_inputs())
    assert events == ["call", "wait", "fetch"]
    assert got["status"] == 0 and np.array_equal(got["accept_len"], [0, 0])


def test_deferred_sample_waits_for_the_current_device(events):
    rows, root, tok, q, u = _inputs()
    got = binding.deferred_sample(rows[:3], root, tok[0], q[0], u[0])
    assert events == ["call", "wait", "fetch"]
    assert got["accept_len"] == 0


@pytest.mark.parametrize("device,waits", [("cuda:1", False), ("cuda:0", True)])
def test_a_copy_on_the_stream_of_the_call_needs_no_other_wait(events, device, waits):
    binding._wait_for_call(torch.device(device))
    assert events == (["wait"] if waits else [])


def test_noalloc_sampler_waits_for_the_current_device(events):
    sampler = binding.NoAllocSampler(4, device="cpu")
    assert sampler.run(*_inputs()) == 0
    assert events == ["call"]  # enqueues only
    sampler.fetch(2)
    assert events == ["call", "wait", "fetch"]


class _WritingLibrary(_FakeLibrary):
    """Writes what the kernels write: n accepted lengths and tokens, the commit record, the status."""

    def duo_spec_sample_noalloc(self, logits, root, vocab, tokens, probs, uniforms, call, out, stream):
        n, res = call._obj.n, out._obj
        ints = lambda p: C.cast(p, C.POINTER(C.c_int32))
        for i in range(4):
            ints(res.commit)[i] = 100 + i
        ints(res.status)[0] = 0
        for i in range(n):
            ints(res.accept_len)[i] = 10 + i
            ints(res.next_token)[i] = 20 + i
        return 0


@pytest.mark.parametrize("max_n", [1, 2, 80])
def test_more_sequences_than_a_sampler_was_made_for_leave_the_commit_alone(events, monkeypatch, max_n):
    monkeypatch.setattr(binding, "load", lambda dtype="bf16": _WritingLibrary(events))
    sampler = binding.NoAllocSampler(max_n, device="cpu")
    assert sampler.accept_len.shape == sampler.next_token.shape == (max_n,)
    assert sampler.run(*_inputs()) == 0  # two sequences
    got = sampler.fetch(2)
    assert (got["selected"], got["commit_len"], got["commit_token"], got["new_prefix_len"], got["status"]) == (100, 101, 102, 103, 0)
    assert got["accept_len"][0] == 10 and got["next_token"][0] == 20
