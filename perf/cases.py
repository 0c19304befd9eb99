"""The work this framework is measured on: whole steps through its public entry points.

A case is one step of a program that runs MoE layers with this library: routing layout, dispatch of
the tokens to the expert rows, combine of the expert outputs (and, in training, the backward pass).
Four kinds of program (`flow`):

  serve   the C ABI through the binding, descriptors built once: layout and dispatch in one call for
          small inputs (at most 8192 routed entries), ep_layout[_prefetch] + ep_dispatch for larger
          ones, then ep_combine.  Options: padded windows with a capacity, rows placed among another
          source's (expert_base), padding tokens (ids of -1), FP8 rows, once-per-rank dispatch,
          two-level summation, dispatch order.
  staged  the same step in its two-phase form (send_only + ep_complete), two buffer sets.
  buffer  the framework-facing EPBuffer: it allocates the outputs and runs on its own stream.
  train   EPBuffer again, forward and backward on one handle.

Expert networks are not part of the path: the expert outputs y are inputs of the combine.
"""
from __future__ import annotations

import math

import torch

from paper_2603_13606_amd import binding as ep
from paper_2603_13606_amd.buffer import EPBuffer

DEV = "cuda:0"

_DEFAULTS = dict(
    flow="serve",
    R=32, T=4096, H=7168, E=256, K=8,
    padded=False,      # [E, C, H] windows instead of concatenated rows
    C=0,               # slots per expert of padded windows
    order="token",     # walk of the direct dispatch: "token" (the default of the library) or "destination"
    prior="uniform",   # of the gate: "uniform", "zipf" (few hot experts), "hot_ranks" (hot destination ranks)
    padding=0.0,       # share of the tokens that are batch padding (not routed)
    base=False,        # rows start where another source's rows end (expert_base)
    sides=False,       # gate weight, source token and per-expert counts are delivered with the rows
    fp8="",            # "" bf16 rows; "walk" quantised in the dispatch; "ahead" quantised during the layout
    once=False,        # once-per-rank dispatch
    node=0,            # ranks per node of the two-level summation, 0 = flat
)


def _case(name, **kw):
    return dict(_DEFAULTS, **kw, name=name)


def listed():
    return [
        # the smallest call that makes sense: launches and host path only
        _case("tiny", R=2, T=64, H=256, E=8, K=2),
        # a decode step of 128 tokens into padded windows, the shape of the low-latency benchmark
        _case("decode_padded", T=128, padded=True, C=128),
        # a ragged decode batch in the two-phase form (overlap of two micro-batches, double buffering)
        _case("decode_two_phase", flow="staged", T=93, padded=True, C=128),
        # a decode step as a serving engine calls it: buffer object, outputs allocated per call
        _case("decode_buffer", flow="buffer", R=16, T=160, H=4096, E=128),
        # a chunk of a chunked prefill, odd token count, between the decode and the prefill regime
        _case("chunk_ragged", T=611, sides=True),
        # high-throughput prefill, the headline shape, in the configuration meant for it
        _case("prefill", order="destination"),
        # prefill in the default configuration with odd sizes: 3001 tokens, 12 ranks, top-6, a hidden size that
        # is no multiple of 1 KiB rows, padding tokens, rows that follow another source's, side outputs
        _case("prefill_ragged", R=12, T=3001, H=2880, E=96, K=6, padding=0.03, base=True, sides=True),
        # skewed routing into padded windows whose capacity cuts the hot experts
        _case("prefill_capacity", R=16, H=4096, E=128, padded=True, C=512, order="destination", prior="zipf"),
        # prefill with quantised rows
        _case("prefill_fp8", fp8="walk", sides=True),
        # prefill with one message per destination rank and expansion on arrival
        _case("prefill_once_per_rank", once=True),
        # one MoE layer of a training step: forward and backward on one handle
        _case("train", flow="train", order="destination"),
        # twice the prefill batch on 64 ranks, half of the traffic to 8 hot ranks, summed per node first
        _case("large_two_level", R=64, T=8192, order="destination", prior="hot_ranks", node=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    c = dict(_DEFAULTS)
    c["flow"] = rng.choice(["serve"] * 6 + ["staged", "buffer", "train"])
    train = c["flow"] == "train"
    c["R"] = rng.choice([2, 4, 8, 12, 16, 32, 64])
    c["E"] = c["R"] * rng.choice([n for n in (1, 2, 3, 4, 8, 16) if 8 <= c["R"] * n <= 256])
    c["K"] = min(c["E"], rng.choice([1, 2, 4, 6, 8, 8, 8]))
    c["H"] = 128 * _log_int(rng, 2, 56) if rng.random() < 0.6 else 8 * _log_int(rng, 32, 896)
    c["T"] = _log_int(rng, 1, 4096 if train else 8192)
    c["prior"] = rng.choice(["uniform", "uniform", "zipf", "hot_ranks"])
    c["order"] = rng.choice(["token", "destination"])
    if c["flow"] in ("serve", "staged"):
        c["sides"] = rng.random() < 0.5
        c["padding"] = rng.choice([0.0, 0.0, round(rng.uniform(0.01, 0.2), 3)])
        kind = rng.choice(["concat", "concat", "base", "padded"])
        if kind == "padded":
            # windows of at most 1 GiB; small capacities cut rows
            most = max(8, (1 << 30) // (2 * c["E"] * c["H"]))
            c["padded"], c["C"] = True, min(most, max(1, _log_int(rng, max(1, c["T"] * c["K"] // c["E"]), 4 * c["T"])))
        c["base"] = kind == "base" and c["flow"] == "serve"
    if c["flow"] == "serve":
        extra = rng.choice(["", "", "fp8", "once", "node"])
        if extra == "fp8" and c["H"] % 128 == 0:
            c["fp8"] = "ahead" if c["order"] == "destination" and rng.random() < 0.3 else "walk"
        elif extra == "once" and not c["base"]:
            c["once"], c["order"] = True, "token"
        elif extra == "node":
            c["node"] = max(1, c["R"] // rng.choice([2, 4, 8]))
    return c


def _log_prior(c, gen, device):
    E = c["E"]
    if c["prior"] == "zipf":
        rank = torch.randperm(E, generator=gen, device=device).float() + 1.0
        return -1.2 * rank.log()
    if c["prior"] == "hot_ranks":  # an eighth of the ranks takes half of the probability
        hot = max(1, c["R"] // 8)
        share = hot / c["R"]
        ranks = torch.randperm(c["R"], generator=gen, device=device) < hot
        p = torch.where(ranks, 0.5 / share, 0.5 / max(1e-9, 1.0 - share))
        return p.repeat_interleave(E // c["R"]).log()
    return torch.zeros(E, device=device)


def _routing(c, gen, device):
    """Expert ids [T, K] in descending gate probability and the gate weights renormalised over them."""
    logits = torch.randn((c["T"], c["E"]), generator=gen, device=device) + _log_prior(c, gen, device)
    top, idx = torch.topk(logits, c["K"], dim=1)
    w = torch.softmax(top, dim=1).contiguous()
    idx = idx.to(torch.int32)
    pad = int(c["T"] * c["padding"])
    if pad:
        idx[c["T"] - pad:] = -1
    return idx.contiguous(), w


def _counts(c, idx):
    e = idx.reshape(-1)
    return torch.bincount(e[e >= 0].long(), minlength=c["E"])


def _normal(shape, gen):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.bfloat16)


class _State:
    """What a program keeps between steps; gives the group back when it is dropped."""

    group = None
    buf = None

    def __del__(self):
        try:
            torch.cuda.synchronize()
            if self.buf is not None:
                self.buf.close()
            if self.group is not None:
                ep.ep_group_destroy(self.group)
        except Exception:
            pass


def prepare(case, seed):
    c = case
    gen = torch.Generator(DEV)
    gen.manual_seed(seed)
    s = _State()
    s.flow = c["flow"]
    T, H, K, E, R = c["T"], c["H"], c["K"], c["E"], c["R"]
    s.topk, s.w = _routing(c, gen, DEV)
    s.x = _normal((T, H), gen)
    order = ep.EP_ORDER_DESTINATION if c["order"] == "destination" else ep.EP_ORDER_TOKEN
    if s.flow in ("buffer", "train"):
        s.buf = EPBuffer(R, E, H, K, max_tokens_per_rank=T, mode="ht", dispatch_order=order)
        s.y = _normal((T * K, H), gen)
        s.g = _normal((T, H), gen) if s.flow == "train" else None
        return s
    cfg = ep.make_config(R, E, H, K, max(T, c["C"]), mode=ep.EP_MODE_LL if c["padded"] else ep.EP_MODE_HT,
                         slots_per_subregion=c["C"], dispatch_path=ep.EP_PATH_RANK_DEDUP if c["once"] else ep.EP_PATH_DIRECT,
                         max_handles=4, staged_buffers=2 if s.flow == "staged" else 0, ranks_per_node=c["node"],
                         dispatch_order=order, quantize_ahead=int(c["fp8"] == "ahead"))
    s.group = ep.ep_group_create(cfg)
    s.stream = torch.cuda.current_stream().cuda_stream
    rows = E * c["C"] if c["padded"] else T * K
    s.base = None
    if c["base"]:
        theirs = _counts(c, _routing(c, gen, DEV)[0])
        both = _counts(c, s.topk) + theirs
        s.base = (torch.cumsum(both, 0) - both + theirs).to(torch.int32)
        rows = 2 * T * K
    shape = (E, c["C"], H) if c["padded"] else (rows, H)
    # rows that the routing does not reach are never written: the windows start out as zeros
    s.recv = torch.zeros(shape, dtype=torch.float8_e4m3fn if c["fp8"] else torch.bfloat16, device=DEV)
    s.scales = torch.zeros((rows, H // 128), device=DEV) if c["fp8"] else None
    s.recv_w = torch.zeros(rows, device=DEV) if c["sides"] else None
    s.recv_src = torch.zeros(rows, dtype=torch.int32, device=DEV) if c["sides"] else None
    s.recv_count = torch.zeros(E, dtype=torch.int32, device=DEV) if c["sides"] else None
    s.y = _normal(shape, gen)
    s.out = torch.zeros((T, H), dtype=torch.bfloat16, device=DEV)
    s.outputs = [t for t in (s.recv, s.scales, s.recv_w, s.recv_src, s.recv_count, s.out) if t is not None]
    if s.flow == "staged":
        return s
    sides = dict(recv_w=s.recv_w, recv_src=s.recv_src, recv_count=s.recv_count)
    s.combine = ep.prepare_combine(s.y, s.out, topk_weights=s.w)
    s.one_call = T * K <= 8192 and not c["fp8"] and not c["once"]
    if s.one_call:
        s.layout_dispatch = ep.PreparedLayoutDispatch(s.group, s.topk, s.x, s.recv, topk_weights=s.w, expert_base=s.base, **sides)
    else:
        s.layout = ep.PreparedLayout(s.group, s.topk, expert_base=s.base, tokens=s.x if c["order"] == "destination" else None)
        s.dispatch = ep.prepare_dispatch(s.x, s.recv, topk_weights=s.w, recv_scales=s.scales,
                                         topk_idx=s.topk if c["once"] else None, **sides)
    return s


def run(s):
    if s.flow == "serve":
        if s.one_call:
            h = s.layout_dispatch(s.stream)
        else:
            h = s.layout(s.stream)
            s.dispatch(h, s.stream)
        s.combine(h, s.stream)
        ep.ep_handle_destroy(h)
        return s.outputs
    if s.flow == "staged":
        h = ep.ep_layout(s.group, s.topk, stream=s.stream)
        ep.ep_dispatch(h, s.x, s.recv, topk_weights=s.w, recv_w=s.recv_w, recv_src=s.recv_src, recv_count=s.recv_count,
                       send_only=1, stream=s.stream)
        ep.ep_complete(h, stream=s.stream)
        ep.ep_combine(h, s.y, s.out, topk_weights=s.w, send_only=1, stream=s.stream)
        ep.ep_complete(h, stream=s.stream)
        ep.ep_handle_destroy(h)
        return s.outputs
    recv_x, recv_src, recv_w, h, _ = s.buf.dispatch(s.x, s.topk, s.w)
    out, _ = s.buf.combine(s.y, h, s.w)
    res = [recv_x, recv_src, recv_w, out, s.buf.recv_expert_counter]
    if s.flow == "train":
        grad_y, grad_w, _ = s.buf.combine_backward(s.g, h, s.w, s.y)
        grad_x, _ = s.buf.combine(grad_y, h)
        res += [grad_y, grad_w, grad_x]
    s.buf.destroy_handle(h)
    return res


def _rows(c):
    """Routed entries that get a row (a typical routing, where a capacity cuts some)."""
    routed = (c["T"] - int(c["T"] * c["padding"])) * c["K"]
    if not c["padded"] or c["C"] >= c["T"]:
        return routed
    gen = torch.Generator()
    gen.manual_seed(1)
    return int(_counts(c, _routing(c, gen, "cpu")[0]).clamp(max=c["C"]).sum())


def work(case):
    """Bytes: what each call of the step has to read and write once (staging copies and index arrays of
    the implementation are not counted).  Flops: one multiply and one add per element summed."""
    c = case
    T, H, K = c["T"], c["H"], c["K"]
    n, m, token = T * K, _rows(c), 2 * H
    row_out = H + H // 32 if c["fp8"] else 2 * H
    sides = 8 * m + 4 * c["E"] if c["sides"] or c["flow"] in ("buffer", "train") else 0
    total = 4 * n + 4 * n                          # expert ids, gate weights
    total += T * token + m * row_out + sides       # dispatch
    total += m * token + T * token                 # combine
    flops = 2 * m * H
    if c["flow"] == "train":
        total += 4 * n + T * token + m * token     # gate weights, output gradient, expert outputs in
        total += m * token + 4 * n                 # their gradients and those of the weights out
        total += m * token + T * token             # row gradients back to token gradients
        flops += 3 * m * H + m * H
    return {"bytes": total, "flops": flops}


def tolerance(case):
    """Rows, codes, scales, counts and indices are copies and exact by construction.  Sums over the K
    expert rows are float32 rounded once to bf16: another order of the sums moves a result to the
    neighbouring bf16 value now and then (one step is at most 2^-7 of the value; against float64 sums
    5e-5 of the values moved, 1.7e-5 relative in the 2-norm).  Weight gradients stay in float32
    (1e-7 relative against float64)."""
    return {"rel": 7e-5, "max": 1e-2}
