"""Framework-facing buffer over the C ABI (Sec. VI-A "Common Backend Architecture",
Table V "Buffer operations"): `dispatch`, `combine`, `get_tokens_per_expert_list`,
`get_comm_stream`, `capture`, `destroy_handle`, `combine_backward`, plus autograd wrappers that reuse one
handle for the forward and the backward pass (Sec. III-F training pattern, Sec. VI-B).

What it adds to the binding is resource plumbing only, as the paper describes it:
  - the group's allocations go through torch's caching allocator (allocator
    callbacks, pointers kept in a map; Sec. VI-A "Memory and streams");
  - a dedicated communication stream for calls that overlap: it waits for the event such a
    call is given, and the compute stream waits for the event it returns.  A call without
    an event would have either stream wait for the other (the paper's synchronous scheme):
    nothing could run beside it, so it runs on the compute stream itself, see `_start`;
  - per-expert counts land in pinned, device-mapped host memory, so reading them needs
    an event wait but no device-to-host copy (Sec. VI-A "Expert counts").
Every data-path step still runs in the library's kernels.
"""
from __future__ import annotations

import contextlib
import ctypes
import threading
from typing import List, Optional, Tuple

import torch

from . import binding as ep


class EPHandle:
    """One routing decision (Sec. III-C "MoE Handle"): the C handle plus what is needed to
    size outputs and to run the backward pass."""

    def __init__(self, raw, topk_idx: torch.Tensor, num_tokens: int):
        self.raw = raw
        self.topk_idx = topk_idx
        self.num_tokens = num_tokens
        self.alive = True


class EPBuffer:
    def __init__(self, num_ranks: int, num_experts: int, hidden: int, top_k: int,
                 max_tokens_per_rank: int, mode: str = "ht", my_rank: int = 0,
                 slots_per_subregion: int = 0, dispatch_path: str = "direct", max_handles: int = 4,
                 device: str = "cuda:0", dispatch_order: int = ep.EP_ORDER_TOKEN, quantize_ahead: bool = False):
        ep.load()
        self.device = torch.device(device)
        self.R, self.E, self.H, self.K, self.B = num_ranks, num_experts, hidden, top_k, max_tokens_per_rank
        self.ll = mode == "ll"
        self.C = (slots_per_subregion or max_tokens_per_rank) if self.ll else 0
        self._held = {}

        def _alloc(pp, nbytes):
            t = torch.empty(int(nbytes), dtype=torch.uint8, device=self.device)
            self._held[t.data_ptr()] = t
            pp[0] = t.data_ptr()
            return 0

        def _free(p):
            return 0 if self._held.pop(p, None) is not None else 1

        self._alloc_cb, self._free_cb = ep.ALLOC_FN(_alloc), ep.FREE_FN(_free)
        cfg = ep.make_config(num_ranks, num_experts, hidden, top_k, max_tokens_per_rank,
                             mode=ep.EP_MODE_LL if self.ll else ep.EP_MODE_HT, my_rank=my_rank,
                             slots_per_subregion=slots_per_subregion,
                             dispatch_path=ep.EP_PATH_RANK_DEDUP if dispatch_path == "once_per_rank" else ep.EP_PATH_DIRECT,
                             max_handles=max_handles, dispatch_order=dispatch_order, quantize_ahead=int(quantize_ahead))
        self._dedup = dispatch_path == "once_per_rank"
        with torch.cuda.device(self.device):
            self.group = ep.ep_group_create(cfg, alloc_fn=self._alloc_cb, free_fn=self._free_cb)
            self._comm = torch.cuda.Stream()
        self._comm_given = False  # somebody else may queue work on the communication stream
        # calls are ordered as they were made, whatever stream each runs on: the event of the last one made outside a
        # graph capture, and the streams that need not wait for it
        self._order_event: Optional[torch.cuda.Event] = None
        self._order_streams: Tuple[int, ...] = ()
        self._lock = threading.Lock()
        # pinned host memory, written by the dispatch kernel through its device mapping
        self.recv_expert_counter = torch.zeros(num_experts, dtype=torch.int32, pin_memory=True)
        self._counter_desc = ep.tensor_desc(self.recv_expert_counter, ep.EP_TAG_RECV_EXPERT_COUNTER_HOST)
        self._counter_desc.data = _device_pointer_of_pinned(self.recv_expert_counter)
        self._last_event: Optional[torch.cuda.Event] = None

    # ------------------------------------------------------------------ streams and events
    @property
    def comm_stream(self) -> torch.cuda.Stream:
        """The communication stream.  Once asked for, it takes every call: its owner may queue work between them.  It comes
        behind the calls made so far, but for one that is given out under graph capture: it may be part of the capture, which
        can't wait for work outside of it.  The next call or request outside the capture makes up for that."""
        with self._lock:
            if self._order_event is not None and self._comm.cuda_stream not in self._order_streams and not self._capturing():
                self._comm.wait_event(self._order_event)
                self._order_streams += (self._comm.cuda_stream,)
            self._comm_given = True
        return self._comm

    @comm_stream.setter
    def comm_stream(self, stream: torch.cuda.Stream) -> None:
        with self._lock:
            self._comm, self._comm_given = stream, True

    def _capturing(self) -> bool:
        """Whether the compute stream or the communication stream is under graph capture."""
        if torch.cuda.is_current_stream_capturing():
            return True
        with torch.cuda.stream(self._comm):
            return torch.cuda.is_current_stream_capturing()

    def get_comm_stream(self) -> torch.cuda.Stream:
        return self.comm_stream

    def capture(self) -> torch.cuda.Event:
        """An event on the compute stream, as the callers pass between layers."""
        ev = torch.cuda.Event()
        ev.record(torch.cuda.current_stream())
        return ev

    def _start(self, previous_event: Optional[torch.cuda.Event]) -> Tuple[torch.cuda.Stream, torch.cuda.Stream, bool]:
        """The compute stream, the stream the call runs on, which has been made to wait, and whether a graph is captured.

        The compute stream itself, where the communication stream would wait for all of it and it for the call in turn:
        two events and two waits across streams cost 22 us per call (a training step of five calls, 440 us of kernels: 588 us,
        this way 488; a decode step, 12 us of kernels: 130, this way 49).  Not under graph capture, whose calls are not ordered
        with those outside, not on another device's stream, and not on a stream that torch did not make and that its owner
        may destroy while the library still remembers it (its id is its address)."""
        compute = torch.cuda.current_stream()
        capturing = torch.cuda.is_current_stream_capturing()
        comm = self._comm
        sp = compute.cuda_stream
        if (previous_event is None and not self._comm_given and not capturing and compute.device_index == comm.device_index
                and (sp == 0 or compute.stream_id != sp)):
            run = compute
        else:
            run, sp = comm, comm.cuda_stream
            if previous_event is not None:
                comm.wait_event(previous_event)
            else:
                comm.wait_stream(compute)
        if not capturing and self._order_event is not None and sp not in self._order_streams:
            run.wait_event(self._order_event)
        return compute, run, capturing

    def _on(self, compute: torch.cuda.Stream, run: torch.cuda.Stream):
        return contextlib.nullcontext() if run is compute else torch.cuda.stream(run)

    def _leave(self, compute: torch.cuda.Stream, run: torch.cuda.Stream, capturing: bool,
               *outputs: Optional[torch.Tensor]) -> torch.cuda.Event:
        """Records the end of the call and makes the compute stream wait for it.  Outputs that were allocated on the
        communication stream are used on the compute stream: their memory must not come back to a later call, which may
        be told to wait for an earlier event only, before that use has ended."""
        ev = torch.cuda.Event()
        ev.record(run)
        if run is not compute:
            for t in outputs:
                if t is not None:
                    t.record_stream(compute)
            compute.wait_event(ev)
        self._last_event = ev
        if not capturing:
            self._order_event, self._order_streams = ev, (run.cuda_stream, compute.cuda_stream)
        return ev

    def _with_counter(self, outs) -> "ctypes.Array":
        """Descriptors of a dispatch's outputs and of the pinned per-expert counter (its device address)."""
        arr = (ep.ep_tensor_t * (len(outs) + 1))()
        ctypes.memmove(arr, ep._descs(outs), ctypes.sizeof(ep.ep_tensor_t) * len(outs))
        arr[len(outs)] = self._counter_desc
        return arr

    # ------------------------------------------------------------------ operations
    def dispatch(self, x: torch.Tensor, topk_idx: Optional[torch.Tensor] = None,
                 topk_weights: Optional[torch.Tensor] = None, handle: Optional[EPHandle] = None,
                 previous_event: Optional[torch.cuda.Event] = None, fp8: bool = False):
        """recv_x, recv_src, recv_w, handle, event = dispatch(x, topk_idx, topk_weights, handle).

        With `handle` given this is the cached dispatch of the backward pass: the routing of
        the forward pass is reused.  HT mode returns [T*K, H] storage (rows beyond the
        handle's count are unused); LL mode returns [E, C, H].  With fp8=True recv_x is a
        pair (codes float8_e4m3fn, scales float32 [rows, H/128])."""
        with self._lock:
            return self._dispatch(x, topk_idx, topk_weights, handle, previous_event, fp8)

    def _dispatch(self, x, topk_idx, topk_weights, handle, previous_event, fp8):
        T = x.shape[0]
        compute, run, capturing = self._start(previous_event)
        sp = run.cuda_stream
        with self._on(compute, run):
            rows = self.E * self.C if self.ll else T * self.K
            dt = torch.float8_e4m3fn if fp8 else torch.bfloat16
            store = torch.empty((rows, self.H), dtype=dt, device=self.device)
            recv_x = store.view(self.E, self.C, self.H) if self.ll else store
            recv_w = torch.empty(rows, dtype=torch.float32, device=self.device) if topk_weights is not None else None
            recv_src = torch.empty(rows, dtype=torch.int32, device=self.device)
            scales = torch.empty((rows, self.H // 128), dtype=torch.float32, device=self.device) if fp8 else None
            ids = topk_idx if handle is None else handle.topk_idx
            ins, outs = ep._dispatch_tensors(x, recv_x, topk_weights, recv_w, recv_src, None, ids if self._dedup else None, scales)
            outs = self._with_counter(outs)
            ins, n_in = ep._descs(ins), len(ins)
            if handle is None:
                assert topk_idx is not None
                # layout and dispatch in one call: one launch for small inputs, and for large ones the layout
                # knows which tokens it may read ahead
                raw = ctypes.c_void_p()
                td = ep.tensor_desc(topk_idx, ep.EP_TAG_TOPK_IDX)
                ep._check(ep.load().ep_layout_dispatch(ctypes.byref(raw), self.group, ctypes.byref(td), None, ins, n_in, outs,
                                                       len(outs), sp), "ep_layout_dispatch")
                handle = EPHandle(raw, topk_idx, T)
            else:
                ep._check(ep.load().ep_dispatch(handle.raw, ins, n_in, outs, len(outs), 0, sp), "ep_dispatch")
            for t in (x, ids, topk_weights):
                if t is not None:
                    t.record_stream(run)
        ev = self._leave(compute, run, capturing, store, recv_w, recv_src, scales)
        return ((recv_x, scales) if fp8 else recv_x), recv_src, recv_w, handle, ev

    def combine(self, y: torch.Tensor, handle: EPHandle, topk_weights: Optional[torch.Tensor] = None,
                previous_event: Optional[torch.cuda.Event] = None):
        """out, event = combine(y, handle, topk_weights)."""
        with self._lock:
            compute, run, capturing = self._start(previous_event)
            sp = run.cuda_stream
            with self._on(compute, run):
                out = torch.empty((handle.num_tokens, self.H), dtype=torch.bfloat16, device=self.device)
                ep.ep_combine(handle.raw, y, out, topk_weights=topk_weights, stream=sp)
                y.record_stream(run)
                if topk_weights is not None:
                    topk_weights.record_stream(run)
            return out, self._leave(compute, run, capturing, out)

    def combine_backward(self, grad_out: torch.Tensor, handle: EPHandle, topk_weights: Optional[torch.Tensor] = None,
                         y: Optional[torch.Tensor] = None, previous_event: Optional[torch.cuda.Event] = None):
        """grad_y, grad_w, event = combine_backward(grad_out, handle, topk_weights, y): the gradient of a
        weighted combine with respect to the expert outputs (windows like y, rows without an entry
        zero) and, when y is given, with respect to the gate weights [T, K]."""
        with self._lock:
            return self._combine_backward(grad_out, handle, topk_weights, y, previous_event)

    def _combine_backward(self, grad_out, handle, topk_weights, y, previous_event):
        compute, run, capturing = self._start(previous_event)
        sp = run.cuda_stream
        with self._on(compute, run):
            if y is not None:
                grad_y = torch.empty(y.shape, dtype=torch.bfloat16, device=self.device)
            else:
                rows = self.E * self.C if self.ll else handle.num_tokens * self.K
                store = torch.empty((rows, self.H), dtype=torch.bfloat16, device=self.device)
                grad_y = store.view(self.E, self.C, self.H) if self.ll else store
            grad_w = torch.empty((handle.num_tokens, self.K), dtype=torch.float32, device=self.device) if y is not None else None
            try:
                ep.ep_combine_backward_full(handle.raw, grad_out, grad_y, topk_weights=topk_weights, y=y, grad_w=grad_w, stream=sp)
            except ep.EpError as err:
                if err.code != ep.EP_ERR_UNSUPPORTED:
                    raise
                # a handle whose rows lie among another source's (expert_base): the whole window is cleared first
                grad_y.zero_()
                ep.ep_combine_backward(handle.raw, grad_out, grad_y, topk_weights=topk_weights, y=y, grad_w=grad_w, stream=sp)
            for t in (grad_out, topk_weights, y):
                if t is not None:
                    t.record_stream(run)
        return grad_y, grad_w, self._leave(compute, run, capturing, grad_y, grad_w)

    def get_tokens_per_expert_list(self) -> List[int]:
        """Rows placed per expert by the last dispatch, read from the pinned counter."""
        if self._last_event is not None:
            self._last_event.synchronize()
        return self.recv_expert_counter.tolist()

    def routing_rows(self, handle: EPHandle) -> torch.Tensor:
        """dst_row [T, K] of the handle as a device tensor (a copy; -1 = no row)."""
        info = ep.ep_handle_query(handle.raw, ok=(ep.EP_SUCCESS, ep.EP_ERR_INVALID_ROUTING, ep.EP_ERR_OVERFLOW))
        out = torch.empty((handle.num_tokens, self.K), dtype=torch.int32, device=self.device)
        if out.numel():
            hip = ep._hip_runtime()
            rc = hip.hipMemcpy(ctypes.c_void_p(out.data_ptr()), ctypes.c_void_p(info.dst_row),
                               ctypes.c_size_t(4 * out.numel()), ctypes.c_int(3))  # 3 = device to device
            if rc != 0:
                raise RuntimeError(f"hipMemcpy failed with {rc}")
        return out

    def get_num_recv_tokens(self, handle: EPHandle) -> int:
        return ep.ep_handle_get_num_recv_tokens(handle.raw)

    def destroy_handle(self, handle: EPHandle) -> None:
        """Deferred destruction (Sec. VI-B): wait for the last recorded event, then release."""
        if handle.alive:
            if self._last_event is not None:
                self._last_event.synchronize()
            ep.ep_handle_destroy(handle.raw)
            handle.alive = False

    def close(self) -> None:
        if self.group is not None:
            self._comm.synchronize()
            if self._order_event is not None:
                self._order_event.synchronize()  # every call made before it has ended too
            ep.ep_group_destroy(self.group, stream=self._comm.cuda_stream)
            self.group = None
            assert not self._held, "group did not return all its allocations"


def _device_pointer_of_pinned(t: torch.Tensor) -> int:
    """Device address of a pinned host tensor (hipHostGetDevicePointer)."""
    hip = ep._hip_runtime()
    dev = ctypes.c_void_p()
    hip.hipHostGetDevicePointer.restype = ctypes.c_int
    rc = hip.hipHostGetDevicePointer(ctypes.byref(dev), ctypes.c_void_p(t.data_ptr()), ctypes.c_uint(0))
    if rc != 0 or not dev.value:
        raise RuntimeError(f"hipHostGetDevicePointer failed with {rc}")
    return int(dev.value)


# ---------------------------------------------------------------------- autograd wrappers


class EPDispatchFn(torch.autograd.Function):
    """Forward: dispatch x.  Backward: the gradient of a row copy is the sum of the row
    gradients, i.e. an unweighted combine with the same handle."""

    @staticmethod
    def forward(ctx, x, buf: EPBuffer, handle: EPHandle):
        recv_x, _, _, _, _ = buf.dispatch(x, handle=handle)
        ctx.buf, ctx.handle = buf, handle
        return recv_x

    @staticmethod
    def backward(ctx, grad_recv):
        gx, _ = ctx.buf.combine(grad_recv.contiguous(), ctx.handle)
        return gx, None, None


class EPCombineFn(torch.autograd.Function):
    """Forward: weighted combine.  Backward: one call with the same handle -- the output gradient
    dispatched to the rows of y, each copy scaled by its gate weight, and the weight gradient as
    the dot product of every expert output row with the gradient of its token."""

    @staticmethod
    def forward(ctx, y, topk_weights, buf: EPBuffer, handle: EPHandle):
        out, _ = buf.combine(y, handle, topk_weights)
        ctx.buf, ctx.handle = buf, handle
        ctx.save_for_backward(y, topk_weights)
        return out

    @staticmethod
    def backward(ctx, grad_out):
        y, w = ctx.saved_tensors
        grad_y, grad_w, _ = ctx.buf.combine_backward(grad_out.contiguous(), ctx.handle, w, y)
        return grad_y, grad_w, None, None
