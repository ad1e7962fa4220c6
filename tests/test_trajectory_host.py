"""The decoding loop's order on streams, on a model of the device that runs on the CPU: work put
on a stream runs only when something waits for that stream, as late as the waits allow, so a
value read without a wait for the stream that writes it is seen to be stale."""
from __future__ import annotations

import contextlib
from types import SimpleNamespace

import pytest
import torch

from paper_2608_01784_amd import trajectory


class Stream:
    def __init__(self, handle):
        self.cuda_stream, self.queue, self.done = handle, [], 0

    def put(self, fn):
        self.queue.append(fn)

    def run_to(self, n):
        while self.done < n:
            self.done += 1
            self.queue[self.done - 1]()

    def wait_stream(self, other):
        n = len(other.queue)
        self.put(lambda: other.run_to(n))

    def synchronize(self):
        self.run_to(len(self.queue))


class Device:
    """Two streams, the layer's and the state update's launches, and copies to the host."""

    def __init__(self, monkeypatch):
        self.current = Stream(1)
        device = self

        class HostTensor(torch.Tensor):
            @classmethod
            def __torch_function__(cls, func, types, args=(), kwargs=None):
                if func is torch.Tensor.copy_ and device is not None:
                    dst, src = args[0].as_subclass(torch.Tensor), args[1]
                    device.current.put(lambda: dst.copy_(src))
                    return args[0]
                return super().__torch_function__(func, types, args, kwargs or {})

        plain_empty = torch.empty

        def empty(*args, pin_memory=False, device=None, **kw):
            t = plain_empty(*args, **kw).fill_(-77)      # (unwritten memory)
            return t.as_subclass(HostTensor) if pin_memory else t

        @contextlib.contextmanager
        def on(stream):
            was, self.current = self.current, stream
            yield
            self.current = was

        monkeypatch.setattr(torch, "empty", empty)
        monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: None)
        monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: self.current)
        monkeypatch.setattr(torch.cuda, "stream", on)
        monkeypatch.setattr(trajectory._lib, "reflex_advance_state", self.advance)

    def advance(self, conf_t, block_idx, seq_offsets, theta, min_commit, masked, hist_len, c1, c2,
                active_block, remaining, stream=None):
        def fn():     # every position whose confidence reaches theta is committed
            masked[conf_t >= theta] = 0
            for s in range(len(remaining)):
                remaining[s] = int(masked[seq_offsets[s]:seq_offsets[s + 1]].sum())
        (stream or self.current).put(fn)


def _run(monkeypatch, other, n_seq=3, per_seq=4):
    dev = Device(monkeypatch)
    T = n_seq * per_seq
    pairs, masked = torch.full((1,), -5, dtype=torch.int32), torch.zeros(T, dtype=torch.uint8)
    state = SimpleNamespace(block_idx=None, masked=masked, hist_len=None, conf_prev1=None, conf_prev2=None,
                            seq_offsets=torch.arange(0, T + 1, per_seq), active_block=torch.zeros(n_seq))
    dev.current.put(lambda: masked.fill_(1))                 # the prompt's state, made on this stream

    def forward(h, state, stream=None):
        (stream or dev.current).put(lambda: pairs.fill_(int(state.masked.sum()) * 10))

    seen = []

    def on_forward(t, state):                                # reads the forward's result and the state
        dev.current.put(lambda: seen.append((int(pairs), int(state.masked.sum()))))

    def confidence(t):                                       # a position of each sequence a forward
        conf = torch.zeros(T)
        dev.current.put(lambda: conf.copy_(torch.arange(T).remainder(per_seq).eq(t).float()))
        return conf

    layer = SimpleNamespace(forward=forward, pairs=pairs)
    stats = trajectory.run_trajectory(layer, None, state, confidence, 0.9, on_forward=on_forward,
                                      stream=Stream(2) if other else None)
    dev.current.synchronize()
    left = [n_seq * (per_seq - 1 - t) for t in range(per_seq)]
    assert stats.masked_left == left and stats.forwards == per_seq
    assert stats.pairs == [10 * (x + n_seq) for x in left]
    assert seen == [(10 * (x + n_seq), x + n_seq) for x in left]


@pytest.mark.parametrize("other", [False, True])
def test_results_come_from_the_stream_the_kernels_run_on(monkeypatch, other):
    _run(monkeypatch, other)


def test_many_sequences_are_added_up_without_a_python_list(monkeypatch):
    # (one element at a time, the host would take longer over many sequences than the forward)
    monkeypatch.setattr(torch.Tensor, "tolist", lambda t: pytest.fail("tolist of the counts"))
    _run(monkeypatch, False, n_seq=300)


def test_a_replaced_forward_is_called_every_time(monkeypatch):
    # a program may wrap the layer's forward, on the class or on one layer, also during the run
    from paper_2608_01784_amd.layer import MoELayer
    Device(monkeypatch)
    pairs, masked = torch.zeros(1, dtype=torch.int32), torch.ones(4, dtype=torch.uint8)
    state = SimpleNamespace(block_idx=None, masked=masked, hist_len=None, conf_prev1=None, conf_prev2=None,
                            seq_offsets=torch.tensor([0, 4]), active_block=torch.zeros(1))
    layer = MoELayer.__new__(MoELayer)
    layer.pairs, layer.ws, layer.out = pairs, None, None
    calls = []
    monkeypatch.setattr(MoELayer, "args", lambda self, *a: "arguments")
    monkeypatch.setattr(trajectory._lib, "reflex_moe_forward", lambda a, ws, stream=None: calls.append("plain"))
    confidence = lambda t: torch.arange(4).eq(t).float()      # noqa: E731

    def replace(t, state):
        if t == 1:
            layer.forward = lambda h, state, stream=None: calls.append("layer")

    with monkeypatch.context() as m:
        m.setattr(MoELayer, "forward", lambda self, h, state, stream=None: calls.append("class"))
        trajectory.run_trajectory(layer, None, state, confidence, 0.9)
    assert calls == ["class"] * 4
    calls.clear()
    masked.fill_(1)
    trajectory.run_trajectory(layer, None, state, confidence, 0.9, on_forward=replace)
    assert calls == ["plain"] * 2 + ["layer"] * 2
