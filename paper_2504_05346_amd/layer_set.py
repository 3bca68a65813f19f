"""Layers that read the same input share the Hessian, hence the damped factor.

The q/k/v projections of an attention block, or the gate/up projections of an MLP, are pruned
against the same calibration input X (paper, Alg. 1: H depends on X only).  `prune_layer_set`
accumulates H once, factors it once and runs one sweep per weight matrix with `factor_in`
(include/thanos.h).  Sequencing and allocation only: every step runs in the library's kernels.
"""
import ctypes
from typing import Iterable, List, Sequence, Tuple

import torch

from .binding import (THANOS_NM, PruneOpts, _check, lib, thanos_factor, thanos_factor_workspace_bytes,
                      thanos_hessian_accumulate, thanos_prune_layer_shared,
                      thanos_prune_workspace_bytes)


# Sweeps of few rows leave most of the chip idle and run side by side, up to _LANES at a time: on the caller's
# stream and on helper streams of the library, each with a workspace of its own that its sweeps use in turn.  More
# than four streams share hardware queues.  In the unstructured mode the selections of concurrent sweeps wait for
# their own workgroups at grid barriers, at most one of which fits a compute unit: together they launch no more
# of them than the sweep with the most rows by itself (`sharers`; 3 x 768 x 768 0.76 -> 0.77 ms a call, 3 x 64 x 1024,
# where that is one workgroup per sweep, 0.94 -> 1.00).
# Whole calls on 2 b tokens, one, two, three, four at a time: at 50 % 3 x 768 x 768 1.42, 1.09, 0.93 ms, 4 x 512 x 2048
# 4.11, 2.62, 2.60, 2.22, 8 x 128 x 4096 14.6, 8.6, 7.1, 5.9, 3 x 1024 x 8192 17.5, 14.3, 11.3; n:m one and all:
# 3 x 768 x 768 0.82, 0.59, 3 x 1280 x 5120 6.7, 4.7, 60 x 64 x 8192 137, 100.  From about 15 rows per compute unit
# in all on, the sweeps fill the chip by themselves (2 x 2048 x 2048 2.86 and 2.84 ms, n:m 1.90 and 1.89).  The further
# workspaces (b x b values and more each, hence the limit on b) take no more than the factorisation's, which
# has just been freed, and 64 MiB.
# A sweep of one block is over before the next lane has been set up: 3 x 768 x 128 n:m 0.24 ms one after the other, 0.27
# side by side, 3 x 768 x 256 0.33 both ways.
_LANES = 4
_ROWS_PER_UNIT = 15
_SIDE_BY_SIDE_COLUMNS = 8192
_SPARE_BYTES = 64 << 20


def _lanes(rows, b, block, need, freed, units) -> int:
    """How many sweeps run at once, for matrices of `rows` rows that need workspaces of up to `need` bytes."""
    if len(rows) < 2 or not 2 * block <= b <= _SIDE_BY_SIDE_COLUMNS:
        return 1
    if sum(-(-c // 16) * 16 for c in rows) > _ROWS_PER_UNIT * units:
        return 1
    return min(_LANES, len(rows), 1 + (freed + _SPARE_BYTES) // need)


def prune_layer_set(weights: Sequence[torch.Tensor], x_chunks: Iterable[torch.Tensor], *, mode: int,
                    sparsity: float = 0.0, n: int = 0, m: int = 0, block_size: int = 128,
                    damping: float = 0.01, outlier_fraction: float = 0.0, cast: bool = False,
                    stream=None) -> Tuple[List[dict], torch.Tensor]:
    """Prune every matrix of `weights` (each c_i x b, same b, on the GPU) against the input given
    as token-major chunks [n_tok, b].  Returns ([{"W": fp32, "W_cast": dtype of the input or
    None, "mask": uint8, "info": int32[1]}, ...], H).  `info` follows thanos_prune_layer; the
    caller synchronises before reading it."""
    if not weights:
        raise ValueError("no weight matrix given")
    b = weights[0].shape[1]
    dev = weights[0].device
    H = torch.zeros((b, b), dtype=torch.float32, device=dev)
    for xc in x_chunks:
        thanos_hessian_accumulate(H, xc, 1.0, stream)
    U = torch.empty((b, b), dtype=torch.float32, device=dev)
    xnorm2 = torch.empty((b,), dtype=torch.float32, device=dev)
    finfo = torch.zeros((1,), dtype=torch.int32, device=dev)
    fws = torch.empty((thanos_factor_workspace_bytes(b),), dtype=torch.uint8, device=dev)
    thanos_factor(H, damping, U, xnorm2, fws, finfo, stream)
    freed = fws.numel()
    del fws
    for W in weights:
        assert W.shape[1] == b and W.device == dev
    rows = [W.shape[0] for W in weights]
    o = PruneOpts(mode=mode, sparsity=float(sparsity), n=n, m=m, block_size=block_size, damping=damping,
                  outlier_fraction=float(outlier_fraction))
    o.factor_in, o.xnorm2_in = U.data_ptr(), xnorm2.data_ptr()
    need = max(thanos_prune_workspace_bytes(c, b, o) for c in rows)
    if need == 0:
        raise ValueError("options rejected by thanos_prune_workspace_bytes")
    lanes = 1
    if stream is None and not torch.cuda.is_current_stream_capturing():  # in a graph: one stream
        units = torch.cuda.get_device_properties(dev).multi_processor_count
        lanes = _lanes(rows, b, block_size, need, freed, units)
    spaces = [torch.empty((need,), dtype=torch.uint8, device=dev)]

    def result(W):
        return {"W": torch.empty(W.shape, dtype=torch.float32, device=dev),
                "W_cast": torch.empty(W.shape, dtype=W.dtype, device=dev) if cast else None,
                "mask": torch.empty(W.shape, dtype=torch.uint8, device=dev),
                "info": torch.zeros((1,), dtype=torch.int32, device=dev)}

    def sweep(W, res, lane, on):
        # a failed factorisation shows in finfo; the sweeps then run on a meaningless factor
        thanos_prune_layer_shared(W, H, o, res["W"], res["W_cast"], res["mask"], spaces[lane], res["info"],
                                  len(spaces), on)

    results = []
    if lanes == 1:
        for W in weights:
            results.append(result(W))
            sweep(W, results[-1], 0, stream)
        return results, H
    # Everything is allocated (and cleared) on the caller's stream before the fork and joined into it again, so
    # that to the caller and its allocator the call is work on that stream.
    results = [result(W) for W in weights]
    try:
        while len(spaces) < lanes:
            spaces.append(torch.empty_like(spaces[0]))
    except torch.OutOfMemoryError:  # fewer lanes, same results
        pass
    main = torch.cuda.current_stream(dev)
    ready = main.record_event()
    streams, helpers, held = [main], [], []
    try:
        # all lanes before the first sweep: the pool lends what a sweep has handed back, with work still queued on
        # it, to the next that asks
        for _ in spaces[1:]:
            helper, side = _borrow(dev)
            helpers.append((helper, side))
            side.wait_event(ready)
            streams.append(side)
        for k, (W, res) in enumerate(zip(weights, results)):
            lane = k % len(spaces)
            sweep(W, res, lane, streams[lane])
            if mode == THANOS_NM and b > 16 * block_size and k < len(spaces) - 1:
                # the sweep has far updates (more than two super-blocks of eight blocks): keep the next lane's
                # from queueing behind them
                held.append(_borrow(dev))
    finally:
        for helper, side in helpers:
            main.wait_stream(side)
        for helper, _ in helpers + held:  # the sweeps have joined what they put on the held ones
            lib().thanos_helper_release(helper)
    return results, H


def _borrow(dev):
    """A helper stream of the library and its handle.  torch makes 32 streams for the first one asked for, and
    among so many the helpers of later calls no longer get hardware queues of their own: a factorisation
    after that call 5.57 instead of 4.94 ms (5120 columns beside the row losses)."""
    helper, stream = ctypes.c_void_p(), ctypes.c_void_p()
    with torch.cuda.device(dev):
        _check(lib().thanos_helper_acquire(ctypes.byref(helper), ctypes.byref(stream)), "thanos_helper_acquire")
    return helper, torch.cuda.ExternalStream(stream.value, device=dev)

