"""A multi-forward decoding run on the GPU: each denoising forward runs the fused
variable-count MoE layer(s) on the current decoding state, then the state kernel
commits positions by the confidence threshold (Eq. (1)), shifts the confidence
history and advances blocks.  The confidences are inputs (in a real model they
come from the LM head of the same forward).

This is bookkeeping around the library's entry points; every step runs in HIP
kernels.
"""
from __future__ import annotations

from contextlib import nullcontext
from dataclasses import dataclass, field
from typing import Callable, List, Optional

from . import _lib
from .layer import PLAIN_FORWARD, MoELayer, TokenState


@dataclass
class TrajectoryStats:
    forwards: int = 0
    pairs: List[int] = field(default_factory=list)      # P of each forward
    masked_left: List[int] = field(default_factory=list)

    @property
    def total_pairs(self) -> int:
        return int(sum(self.pairs))


def run_trajectory(layer: MoELayer, h, state: TokenState, confidence: Callable[[int], object],
                   theta: float, min_commit: int = 0, max_forwards: int = 10_000,
                   on_forward: Optional[Callable[[int, TokenState], None]] = None,
                   stream=None) -> TrajectoryStats:
    """Run forwards until every target position is committed (or max_forwards).

    confidence(t) returns the [T] float32 device tensor of forward t's
    confidences.  on_forward(t, state), if given, is called after each layer
    forward and before the state update (the state still describes forward t).
    The forwards and state updates run on `stream` (default: the current one); both
    callbacks run on the current stream, which is ordered after the forward before them
    and before the state update after them."""
    import torch
    stats = TrajectoryStats()
    remaining = torch.empty(state.active_block.shape[0], dtype=torch.int32,
                            device=state.active_block.device)
    # The host needs P and the masked positions left of every forward before it can launch the
    # next one, and the GPU idles meanwhile.  Both come back behind one wait (two `item()` and a
    # reduction launch before), and the next forward's arguments are prepared ahead of it
    # (LLaDA-MoE layer, T = 1024: 307 us a forward before, 280 now).
    host = torch.empty(1 + remaining.shape[0], dtype=torch.int32, pin_memory=True)
    # Few sequences are added up as a list, many as an array (1 / 64 / 1024 sequences: 1.0 / 2.5 /
    # 16 us as a list, 2.8 / 2.8 / 2.1 as an array; 65536: a forward 0.3 ms longer).
    array = host.numpy() if remaining.shape[0] > 64 else None
    # The kernels' stream: the results are copied and waited for there.  Where it is not the
    # current stream, each waits for the other where one reads what the other has made.
    current = torch.cuda.current_stream()
    run = current if stream is None else stream
    apart = run.cuda_stream != current.cuda_stream
    if apart:
        if not hasattr(run, "wait_stream"):      # (any object with a stream handle)
            run = torch.cuda.ExternalStream(run.cuda_stream)
        run.wait_stream(current)
        remaining.record_stream(run)
    args = None
    for t in range(max_forwards):
        if args is None:
            layer.forward(h, state, stream=stream)
        else:
            _lib.reflex_moe_forward(args, layer.ws, stream)
        if apart:
            current.wait_stream(run)
        if on_forward is not None:
            on_forward(t, state)
        conf_t = confidence(t)
        if stream is None:
            run = torch.cuda.current_stream()
        elif apart:
            run.wait_stream(current)
        _lib.reflex_advance_state(conf_t, state.block_idx, state.seq_offsets, theta, min_commit,
                                  state.masked, state.hist_len, state.conf_prev1, state.conf_prev2,
                                  state.active_block, remaining, stream=stream)
        with torch.cuda.stream(run) if apart else nullcontext():
            host[:1].copy_(layer.pairs, non_blocking=True)
            host[1:].copy_(remaining, non_blocking=True)
        plain = getattr(layer.forward, "__func__", None) is PLAIN_FORWARD
        args = layer.args(h, state) if plain else None
        run.synchronize()
        stats.forwards += 1
        counts = host.tolist() if array is None else array
        stats.pairs.append(int(counts[0]))
        left = sum(counts[1:]) if array is None else int(counts[1:].sum())
        stats.masked_left.append(left)
        if left == 0:
            break
    return stats
