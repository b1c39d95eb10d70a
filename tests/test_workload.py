"""Properties of the seeded input generators (harness only)."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_2310_08152_amd import workload as W


def _valid(spans, L_total):
    for (c, r), (c2, _) in zip(spans, spans[1:]):
        assert c < r < c2, (c, r, c2)
    for c, r in spans:
        assert 0 <= c < L_total and r > c


@pytest.mark.parametrize("name", list(W.WORKLOADS))
def test_workload_spans_are_valid_and_deterministic(name):
    w = W.get_workload(name)
    a = W.workload_spans(w)
    b = W.workload_spans(w)
    assert a == b
    assert len(a) == w.batch
    for s in a:
        _valid(s, w.meta_len)


def test_tiny_spans():
    s = W.workload_spans(W.get_workload("tiny-f32"))[0]
    assert s == [(32 * k + 8, 32 * k + 24) for k in range(8)]


def test_window_spans_ratio_and_jitter():
    w = W.get_workload("opt1.3b-prefill")
    for s in W.workload_spans(w):
        assert len(s) == 32
        assert W.span_coverage(s, w.seq_len) == w.seq_len // 2
        for k, (c, r) in enumerate(s):
            assert abs(c - (64 * k + 16)) <= 4 and r - c == 32


@pytest.mark.parametrize("name,ratio", [("opt1.3b-decode", 0.75), ("3b-rope", 0.5)])
def test_uniform_spans_exact_ratio(name, ratio):
    w = W.get_workload(name)
    for s in W.workload_spans(w):
        assert W.span_coverage(s, w.seq_len) == int(round(ratio * w.seq_len))
        assert all(r < w.seq_len for _, r in s)
        lengths = [r - c for c, r in s]
        assert max(lengths) <= 64


def test_streaming_schedule():
    w = W.get_workload("3b-rope-stream")
    s = W.workload_spans(w)[0]
    closed = [x for x in s if x[1] < w.meta_len]
    assert len(closed) == 21 and len(s) == 22
    assert all(r - c == 32 for c, r in s)
    assert s[0] == (1032, 1064)


def test_randn_rounds_to_bf16():
    import torch
    x = W.randn((4, 5), seed=3, dtype="bf16")
    assert x.dtype == torch.bfloat16
    y = W.randn((4, 5), seed=3, dtype="f32")
    assert torch.equal(x, y.to(torch.bfloat16))


POSITIONS = {
    "int32": lambda t: t,
    "int64": lambda t: t.long(),
    "column-major": lambda t: t.t().contiguous().t(),
    "row-slice": lambda t: torch.cat([t, t], 1)[:, :t.shape[1]],
    "one-for-all": lambda t: t[:1],
}


@pytest.mark.parametrize("form", list(POSITIONS))
@pytest.mark.parametrize("dev", ["cpu", pytest.param("cuda", marks=pytest.mark.gpu)])
def test_start_prompt_takes_any_positions(dev, form):
    """Whatever torch can copy into the bookkeeping: host caches, positions of
    another integer type, in views, or one sequence's for all."""
    if dev == "cuda" and not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2310_08152_amd import path as P
    cache = P.KVCache(1, 3, 1, 10, 64, torch.float32, dev)
    pos = POSITIONS[form](torch.arange(36, dtype=torch.int32).view(3, 12) % 7)
    for where in {dev, "cpu"}:
        cache.pos_ids.zero_()
        cache.start_prompt(5, SimpleNamespace(pos=pos.to(where)))
        want = torch.zeros(3, 10, dtype=torch.int32)
        want[:, :5] = pos[:, :5]
        assert torch.equal(cache.pos_ids.cpu(), want)
        assert cache.tok_idx[:, :5].tolist() == [[0, 1, 2, 3, 4]] * 3
        assert cache.kv_len.tolist() == cache.cur_tok.tolist() == [5] * 3


@pytest.mark.parametrize("current", [0, 1])
def test_start_prompt_on_another_gpu(monkeypatch, current):
    """The library launches on the current device: a cache on another GPU is
    filled by torch's copies, which go to the cache's.  (Stand-ins on the CPU
    for tensors on the second GPU.)"""
    from paper_2310_08152_amd import path as P
    gpu = torch.device("cuda:1")
    pos = torch.arange(24, dtype=torch.int32).view(2, 12)

    class OnGpu:
        is_cuda, device, dtype, shape = True, gpu, pos.dtype, pos.shape
        dim, is_contiguous = pos.dim, pos.is_contiguous

        def __getitem__(self, at):
            return pos[at]

    cache = P.KVCache(1, 2, 1, 10, 64, torch.float32, "cpu")
    length = cache.kv_len
    cache.kv_len = SimpleNamespace(device=gpu, fill_=length.fill_)
    launches = []
    monkeypatch.setattr(torch.cuda, "current_device", lambda: current)
    monkeypatch.setattr(P.B, "kv_start", lambda *a: launches.append(a))
    cache.start_prompt(5, SimpleNamespace(pos=OnGpu()))
    assert len(launches) == current
    if not current:
        assert torch.equal(cache.pos_ids[:, :5], pos[:, :5]) and length.tolist() == [5, 5]
