"""The framework-facing buffer (dispatch / combine / counters / autograd reuse of one
handle) against the oracle and a dense float64 reference."""
import numpy as np
import pytest
import torch

from paper_2603_13606_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hx():
    import ep_harness
    ep_harness.ensure_built()
    assert torch.cuda.is_available()
    return ep_harness


def test_buffer_forward_matches_oracle_and_counts(hx, oracle_mod):
    from paper_2603_13606_amd.buffer import EPBuffer
    w = wl.make_workload("ll_decode", T=100, H=512)
    spec = w.spec
    lay = oracle_mod.layout(w.topk_idx, E=spec.E, R=spec.R, C_rank=128)
    buf = EPBuffer(spec.R, spec.E, spec.H, spec.K, max_tokens_per_rank=128, mode="ht")
    try:
        x = hx.bits_to_dev(w.x_bits)
        topk = torch.from_numpy(w.topk_idx).to(hx.DEV)
        gate = torch.from_numpy(w.topk_w).to(hx.DEV)
        recv_x, recv_src, recv_w, h, ev = buf.dispatch(x, topk, gate, previous_event=buf.capture())
        assert buf.get_tokens_per_expert_list() == lay.expert_count.tolist()
        rows = buf.get_num_recv_tokens(h)
        assert rows == lay.kept
        o_recv = np.zeros((rows, spec.H), np.uint16)
        o_w = np.zeros(rows, np.float32)
        o_src = np.zeros(rows, np.int32)
        oracle_mod.dispatch(w.x_bits, w.topk_w, lay, o_recv, o_w, o_src)
        assert np.array_equal(hx.dev_to_bits(recv_x[:rows]), o_recv)
        assert np.array_equal(recv_src[:rows].cpu().numpy(), o_src)
        assert np.array_equal(recv_w[:rows].cpu().numpy(), o_w)
        assert np.array_equal(buf.routing_rows(h).cpu().numpy(), lay.dst_row)
        out, _ = buf.combine(recv_x, h, gate)
        torch.cuda.synchronize()
        assert np.array_equal(hx.dev_to_bits(out), oracle_mod.combine(o_recv, w.topk_w, lay, spec.H, acc="f32"))
        # cached dispatch with the same handle (backward pass), FP8 output
        (q, sc), _, _, h2, _ = buf.dispatch(x, handle=h, fp8=True)
        assert h2 is h
        o_q = np.zeros((rows, spec.H), np.uint8)
        o_s = np.zeros((rows, spec.H // 128), np.float32)
        oracle_mod.dispatch_fp8(w.x_bits, lay, o_q, o_s)
        torch.cuda.synchronize()
        assert np.array_equal(q[:rows].view(torch.uint8).cpu().numpy(), o_q)
        assert np.array_equal(sc[:rows].cpu().numpy(), o_s)
        buf.destroy_handle(h)
    finally:
        buf.close()


@pytest.mark.parametrize("name,T,H,mode,C,order", [
    ("tiny", None, None, "ht", 0, 0), ("tiny", None, None, "ll", 6, 0),
    ("ll_decode", 100, 1000, "ht", 0, 0), ("skew", 700, 512, "ll", 30, 0),
    ("ht_prefill", 1500, 7168, "ht", 0, 0),
    # groups in destination order, inputs of 8192 entries and more: the backward kernel walks the rows as they lie
    ("ht_prefill", 1500, 7168, "ht", 0, 1),
    ("skew", 1100, 520, "ll", 30, 1),          # padded windows, most entries cut by the capacity, 65 units per row
    ("skew", 1100, 512, "ll", 1100, 2),        # padded, nothing cut
    ("ll_decode", 1030, 64, "ht", 0, 1),       # rows of 8 units: one wave, most lanes idle
    ("ll_decode", 300, 256, "ht", 0, 1),       # too small for the row order: token walk
])
def test_backward_calls_match_the_oracle_composition(hx, oracle_mod, name, T, H, mode, C, order):
    """The backward pass with the handle of the forward pass, piece by piece against oracle calls:
    grad_x (backward of dispatch) = unweighted oracle.combine of the row gradients, bit-exact;
    grad_y (backward of combine) = oracle.dispatch, entry by entry, of the output gradient scaled by
    the entry's gate weight -- bit-exact with the float32 product, within one bf16 ulp of the
    float64 one; grad_w = row dot products, within the float32 summation bound of the float64 sums
    (far inside 1e-3 relative wherever the terms do not cancel)."""
    import backward_compose as bc
    from paper_2603_13606_amd.buffer import EPBuffer
    w = wl.make_workload(name, T=T, **({"H": H} if H else {}))
    spec = w.spec
    T, K, Hh = spec.T, spec.K, spec.H
    ll = mode == "ll"
    Cc = (C if C else T) if ll else 0
    topk = w.topk_idx.copy()
    topk[::11, 0] = -1
    lay = oracle_mod.layout(topk, E=spec.E, R=spec.R, layout=int(ll), C=Cc, C_rank=T)
    rows = spec.E * Cc if ll else T * K
    buf = EPBuffer(spec.R, spec.E, Hh, K, max_tokens_per_rank=T, mode=mode, slots_per_subregion=C, dispatch_order=order)
    try:
        rng = np.random.default_rng(T + Hh)
        d_topk = torch.from_numpy(topk).to(hx.DEV)
        gate = torch.from_numpy(w.topk_w).to(hx.DEV)
        x = hx.bits_to_dev(w.x_bits)
        _, _, _, h, _ = buf.dispatch(x, d_topk)
        # stand-in expert outputs and an output gradient, both arbitrary bf16 data
        y_bits = wl.f32_to_bf16_bits(rng.standard_normal((rows, Hh)).astype(np.float32))
        g_bits = wl.f32_to_bf16_bits(rng.standard_normal((T, Hh)).astype(np.float32))
        y = hx.bits_to_dev(y_bits)
        y = y.view(spec.E, Cc, Hh) if ll else y
        g = hx.bits_to_dev(g_bits)
        grad_y, grad_w, _ = buf.combine_backward(g, h, gate, y)
        torch.cuda.synchronize()
        want32 = bc.grad_y_rows(oracle_mod, lay, w.topk_w, g_bits, rows)
        want64 = bc.grad_y_rows(oracle_mod, lay, w.topk_w, g_bits, rows, exact=True)
        got_gy = hx.dev_to_bits(grad_y.reshape(rows, Hh))
        assert np.array_equal(got_gy, want32), "grad_y differs from the dispatched, scaled gradient"
        assert hx.bf16_ulp_distance(got_gy, want64).max() <= 1
        ref_w, mag, valid = bc.grad_w_reference(y_bits, g_bits, lay)
        bound = mag * 64 * 2.0 ** -24 + 1e-30
        got_w = grad_w.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got_w - ref_w) <= np.where(valid, bound, 0.0)), "grad_w outside the float32 summation bound"
        big = valid & (np.abs(ref_w) > 0.05 * mag)
        assert np.all(np.abs(got_w - ref_w)[big] <= 1e-3 * np.abs(ref_w)[big])
        assert np.all(got_w[~valid] == 0.0)
        # backward of dispatch: the row gradients summed per token, no weights
        r_bits = wl.f32_to_bf16_bits(rng.standard_normal((rows, Hh)).astype(np.float32))
        gr = hx.bits_to_dev(r_bits)
        gx, _ = buf.combine(gr.view(spec.E, Cc, Hh) if ll else gr, h)
        torch.cuda.synchronize()
        assert np.array_equal(hx.dev_to_bits(gx), oracle_mod.combine(r_bits, None, lay, Hh, acc="f32"))
        # without the expert outputs only grad_y is produced; y without grad_w is refused
        gy2, gw2, _ = buf.combine_backward(g, h, gate)
        torch.cuda.synchronize()
        assert gw2 is None and np.array_equal(hx.dev_to_bits(gy2.reshape(rows, Hh)), want32)
        from paper_2603_13606_amd import binding as ep
        with pytest.raises(ep.EpError):
            ep.ep_combine_backward(h.raw, g, grad_y, topk_weights=gate, y=y)
        buf.destroy_handle(h)
    finally:
        buf.close()


@pytest.mark.parametrize("E,T,C,H,gap,extra", [
    (8, 40, 0, 136, 8, 3), (8, 40, 3, 136, 8, 0), (8, 40, 90, 136, 8, 0), (96, 7, 5, 136, 8, 0), (768, 30, 4, 136, 8, 0),
    (8, 0, 0, 136, 8, 3), (8, 0, 4, 136, 8, 0),
    # rows back to back: several pieces per window, rows that straddle them; rows of one unit; one piece per window
    (16, 3, 200, 2056, 0, 0), (16, 10, 700, 8, 0, 0), (16, 10, 700, 8, 8, 0), (304, 2, 3, 64, 0, 0),
    (8, 40, 0, 520, 0, 3000), (8, 900, 0, 2056, 8, 500), (8, 900, 1100, 512, 0, 0), (8, 900, 60, 512, 8, 0),
])
def test_backward_clears_exactly_the_rows_without_an_entry(hx, oracle_mod, E, T, C, H, gap, extra):
    """ep_combine_backward_full into poisoned windows: rows of entries as ep_combine_backward leaves them,
    every other row zero, nothing outside the rows (a strided window); C = 0 is the concatenated layout.  More
    experts than the clearing workgroups (768), a number that does not divide them (96), empty inputs."""
    from paper_2603_13606_amd import binding as ep
    K, B = 4, max(T, 1)
    gen = torch.Generator(hx.DEV).manual_seed(E + T)
    topk = torch.randint(0, E, (T, K), generator=gen, device=hx.DEV, dtype=torch.int32)
    topk[::5, 1] = -1
    lay = oracle_mod.layout(topk.cpu().numpy(), E=E, R=8, layout=int(C > 0), C=C or B, C_rank=B)
    cfg = ep.make_config(8, E, H, K, B, mode=ep.EP_MODE_LL if C else ep.EP_MODE_HT, slots_per_subregion=C)
    group = ep.ep_group_create(cfg)
    try:
        h = ep.ep_layout(group, topk)
        rows = E * C if C else B * K + extra
        g = torch.randn((T, H), generator=gen, device=hx.DEV).bfloat16()
        store = torch.full((rows, H + gap), 7.0, dtype=torch.bfloat16, device=hx.DEV)
        plain = store.clone()
        win = lambda s: (s.view(E, C, H + gap) if C else s)[..., :H]
        ep.ep_combine_backward_full(h, g, win(store))
        ep.ep_combine_backward(h, g, win(plain))
        torch.cuda.synchronize()
        reached = np.zeros(rows, bool)
        reached[lay.dst_row[lay.dst_row >= 0]] = True
        want = plain.cpu()
        want[torch.from_numpy(~reached), :H] = 0
        assert torch.equal(store.cpu(), want)
        assert np.all(want[torch.from_numpy(~reached), H:].float().numpy() == 7.0)
        ep.ep_handle_destroy(h)
        if not C:  # among another source's rows: refused
            h = ep.ep_layout(group, topk, expert_base=torch.zeros(E, dtype=torch.int32, device=hx.DEV))
            with pytest.raises(ep.EpError):
                ep.ep_combine_backward_full(h, g, win(store))
            ep.ep_handle_destroy(h)
    finally:
        torch.cuda.synchronize()
        ep.ep_group_destroy(group)


@pytest.mark.parametrize("C", [0, 100])
def test_large_backward_gives_the_gradients_of_its_halves(hx, C):
    """A call large enough for two launches (12 000 rows of 8 KiB, 98 MB) against the same tokens in two calls
    of half the size (one launch each): bit for bit, concatenated and padded with entries cut."""
    from paper_2603_13606_amd import binding as ep
    E, T, H, K = 128, 1500, 4096, 8
    gen = torch.Generator(hx.DEV).manual_seed(C)
    topk = torch.randint(0, E, (T, K), generator=gen, device=hx.DEV, dtype=torch.int32)
    topk[::7, 3] = -1
    w = torch.rand((T, K), generator=gen, device=hx.DEV)
    g = torch.randn((T, H), generator=gen, device=hx.DEV).bfloat16()
    cfg = ep.make_config(8, E, H, K, T, mode=ep.EP_MODE_LL if C else ep.EP_MODE_HT, slots_per_subregion=C)
    group = ep.ep_group_create(cfg)
    rows = E * C if C else T * K
    y = torch.randn((rows, H), generator=gen, device=hx.DEV).bfloat16()
    shape = (E, C, H) if C else (rows, H)
    try:
        def run(lo, hi, src):
            h = ep.ep_layout(group, topk[lo:hi])
            dst = ep.read_device_i32(ep.ep_handle_query(h).dst_row, (hi - lo) * K).view(-1, K).to(hx.DEV).long()
            ys = torch.zeros_like(y)
            ys[dst[dst >= 0]] = src(dst)
            gy, gw = torch.zeros_like(y), torch.empty((hi - lo, K), device=hx.DEV)
            ep.ep_combine_backward(h, g[lo:hi], gy.view(shape), topk_weights=w[lo:hi], y=ys.view(shape), grad_w=gw)
            torch.cuda.synchronize()
            ep.ep_handle_destroy(h)
            return dst, gy, gw
        dst, gy, gw = run(0, T, lambda d: y[d[d >= 0]])
        for lo, hi in ((0, T // 2), (T // 2, T)):
            whole = dst[lo:hi]

            def src(d):
                part = torch.zeros((hi - lo, K, H), dtype=torch.bfloat16, device=hx.DEV)
                part[whole >= 0] = y[whole[whole >= 0]]
                return part[d >= 0]
            d2, gy2, gw2 = run(lo, hi, src)
            both = (whole >= 0) & (d2 >= 0)   # a capacity cuts other entries of a half
            assert both.sum() >= (3000 if C else (topk[lo:hi] >= 0).sum())
            assert torch.equal(gw[lo:hi][both], gw2[both])
            assert torch.equal(gy[whole[both]], gy2[d2[both]])
    finally:
        torch.cuda.synchronize()
        ep.ep_group_destroy(group)


@pytest.mark.parametrize("full", [False, True])
def test_backward_without_any_row_gives_zero_weight_gradients(hx, full):
    """T tokens that are all padding and expert outputs of no rows at all ([0, H], null data): the weight
    gradients are zeros, not what their storage held."""
    from paper_2603_13606_amd import binding as ep
    R, E, H, K, T = 4, 16, 256, 4, 37
    group = ep.ep_group_create(ep.make_config(R, E, H, K, T, mode=ep.EP_MODE_HT))
    try:
        h = ep.ep_layout(group, torch.full((T, K), -1, dtype=torch.int32, device=hx.DEV))
        g = torch.randn((T, H), device=hx.DEV).bfloat16()
        w = torch.rand((T, K), device=hx.DEV)
        y, grad_y = (torch.empty((0, H), dtype=torch.bfloat16, device=hx.DEV) for _ in range(2))
        assert y.data_ptr() == 0
        grad_w = torch.full((T, K), 7.0, device=hx.DEV)
        call = ep.ep_combine_backward_full if full else ep.ep_combine_backward
        call(h, g, grad_y, topk_weights=w, y=y, grad_w=grad_w)
        torch.cuda.synchronize()
        assert torch.all(grad_w == 0.0)
        ep.ep_handle_destroy(h)
    finally:
        torch.cuda.synchronize()
        ep.ep_group_destroy(group)


@pytest.mark.parametrize("T,H", [(300, 512), (1500, 4096)])
def test_backward_in_place(hx, T, H):
    """Weight gradients written over the gate weights, row gradients over the expert outputs: as into tensors of
    their own, also where a call is large enough for two launches (12 000 rows of 8 KiB)."""
    from paper_2603_13606_amd import binding as ep
    E, K = 128, 8
    gen = torch.Generator(hx.DEV).manual_seed(T)
    topk = torch.randint(0, E, (T, K), generator=gen, device=hx.DEV, dtype=torch.int32)
    topk[::7, 3] = -1
    w = torch.rand((T, K + 2), generator=gen, device=hx.DEV)
    g = torch.randn((T, H), generator=gen, device=hx.DEV).bfloat16()
    y = torch.randn((T * K, H), generator=gen, device=hx.DEV).bfloat16()
    group = ep.ep_group_create(ep.make_config(8, E, H, K, T, mode=ep.EP_MODE_HT))
    try:
        h = ep.ep_layout(group, topk)
        want_y, want_w = y.clone(), torch.empty((T, K), device=hx.DEV)
        ep.ep_combine_backward(h, g, want_y, topk_weights=w[:, :K], y=y, grad_w=want_w)
        for over_w, over_y in ((True, False), (False, True), (True, True)):
            w2, y2 = w.clone(), y.clone()
            gw, gy = (w2[:, :K] if over_w else torch.empty((T, K), device=hx.DEV)), (y2 if over_y else y.clone())
            ep.ep_combine_backward(h, g, gy, topk_weights=w2[:, :K], y=y2, grad_w=gw)
            torch.cuda.synchronize()
            assert torch.equal(gw, want_w) and torch.equal(gy, want_y), (over_w, over_y)
            assert torch.equal(w2[:, K:], w[:, K:])
        ep.ep_handle_destroy(h)
    finally:
        torch.cuda.synchronize()
        ep.ep_group_destroy(group)


def test_buffer_backward_with_rows_among_another_source(hx):
    """A handle made with expert_base, wrapped for the buffer: combine_backward fills every row without an entry
    with zeros, as it does for the buffer's own handles."""
    from paper_2603_13606_amd import binding as ep
    from paper_2603_13606_amd.buffer import EPBuffer, EPHandle
    R, E, H, K, T = 4, 16, 256, 4, 60
    gen = torch.Generator(hx.DEV).manual_seed(4)
    topk = torch.randint(0, E, (T, K), generator=gen, device=hx.DEV, dtype=torch.int32)
    count = torch.bincount(topk.reshape(-1).long(), minlength=E)
    base = (torch.cumsum(count + 3, 0) - count).to(torch.int32)  # three rows of another source ahead of each expert's
    buf = EPBuffer(R, E, H, K, max_tokens_per_rank=T, mode="ht")
    try:
        raw = ep.ep_layout(buf.group, topk, expert_base=base)
        torch.cuda.synchronize()
        h = EPHandle(raw, topk, T)
        rows = T * K + 3 * E + 5
        g = torch.randn((T, H), generator=gen, device=hx.DEV).bfloat16()
        y = torch.randn((rows, H), generator=gen, device=hx.DEV).bfloat16()
        w = torch.rand((T, K), generator=gen, device=hx.DEV)
        poison = torch.full((rows, H), 7.0, dtype=torch.bfloat16, device=hx.DEV)  # what the allocator hands out next may hold
        del poison
        grad_y, grad_w, _ = buf.combine_backward(g, h, w, y)
        want_y, want_w = torch.zeros_like(y), torch.empty((T, K), device=hx.DEV)
        ep.ep_combine_backward(raw, g, want_y, topk_weights=w, y=y, grad_w=want_w)
        torch.cuda.synchronize()
        assert torch.equal(grad_y, want_y) and torch.equal(grad_w, want_w)
        buf.destroy_handle(h)
    finally:
        buf.close()


def test_outputs_dropped_while_compute_still_reads_them_are_not_handed_out_again(hx):
    """Work on the results of three calls is queued, the results are dropped, and the next calls wait for an
    earlier event only (overlap): they get other memory while that work is pending, and it reads what it was given."""
    from paper_2603_13606_amd.buffer import EPBuffer
    R, E, H, K, T = 4, 16, 512, 4, 256
    gen = torch.Generator(hx.DEV).manual_seed(8)
    topk = torch.randint(0, E, (T, K), generator=gen, device=hx.DEV, dtype=torch.int32)
    gate = torch.rand((T, K), generator=gen, device=hx.DEV)
    xs = [torch.randn((T, H), generator=gen, device=hx.DEV).bfloat16() for _ in range(2)]
    buf = EPBuffer(R, E, H, K, max_tokens_per_rank=T, mode="ht")
    try:
        torch.cuda.synchronize()
        early = buf.capture()
        y = torch.randn((T * K, H), generator=gen, device=hx.DEV).bfloat16()
        recv_x, recv_src, recv_w, h, _ = buf.dispatch(xs[0], topk, gate)
        out, _ = buf.combine(recv_x, h, gate)
        grad_y, grad_w, _ = buf.combine_backward(xs[1], h, gate, y)
        first = [recv_x, recv_src, recv_w, out, grad_y, grad_w]
        want, got = [t.clone() for t in first], [torch.empty_like(t) for t in first]
        spans = [(t.data_ptr(), t.data_ptr() + t.numel() * t.element_size()) for t in first]
        torch.cuda.synchronize()
        torch.cuda._sleep(100_000_000)  # the compute stream is behind from here on
        for a, b in zip(got, first):
            a.copy_(b)
        end = buf.capture()
        del recv_x, recv_src, recv_w, out, grad_y, grad_w, first, b
        second = buf.dispatch(xs[1], topk, gate, previous_event=early)
        h2 = second[3]
        again = [*second[:3], buf.combine(y, h, gate, previous_event=early)[0],
                 *buf.combine_backward(xs[0], h, gate, y, previous_event=early)[:2]]
        assert not end.query(), "the reads were over too early for this test to say anything"
        for t in again:
            lo, hi = t.data_ptr(), t.data_ptr() + t.numel() * t.element_size()
            assert all(hi <= a or b <= lo for a, b in spans)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        buf.destroy_handle(h)
        buf.destroy_handle(h2)
    finally:
        torch.cuda.synchronize()
        buf.close()


@pytest.mark.parametrize("call", ["dispatch", "combine", "combine_backward"])
def test_inputs_of_a_third_stream_dropped_behind_a_call_are_not_handed_out_again(hx, call):
    """Every input comes from a stream that is neither the compute nor the communication stream and is dropped once the
    call is queued: that stream gets other memory until the call has run, and the results are those of a call alone."""
    from paper_2603_13606_amd.buffer import EPBuffer
    R, E, H, K, T = 4, 16, 512, 4, 256
    side = torch.cuda.Stream()
    buf = EPBuffer(R, E, H, K, max_tokens_per_rank=T, mode="ht")

    def inputs():
        with torch.cuda.stream(side):
            gen = torch.Generator(hx.DEV).manual_seed(9)
            topk = torch.randint(0, E, (T, K), generator=gen, device=hx.DEV, dtype=torch.int32)
            w = torch.rand((T, K), generator=gen, device=hx.DEV)
            x, y = (torch.randn((n, H), generator=gen, device=hx.DEV).bfloat16() for n in (T, T * K))
        side.synchronize()
        return topk, w, x, y

    def run(topk, w, x, y, h):
        if call == "dispatch":
            r = buf.dispatch(x, topk, w)
            r[3].topk_idx = None  # the handle would keep the ids
            return r[:3], r[3]
        return (buf.combine(y, h, w)[:1] if call == "combine" else buf.combine_backward(x, h, w, y)[:2]), None

    try:
        made = inputs()
        h = buf.dispatch(made[2], made[0], made[1])[3]
        h.topk_idx = None
        alone, h1 = run(*made, h)
        want = [t.clone() for t in alone]
        torch.cuda.synchronize()
        del made
        made = inputs()
        used = {"dispatch": made[:3], "combine": (made[1], made[3]), "combine_backward": made[1:]}[call]
        spans = [(t.data_ptr(), t.data_ptr() + t.numel() * t.element_size()) for t in used]
        torch.cuda._sleep(100_000_000)
        end = buf.capture()
        got, h2 = run(*made, h)
        del used, made
        taken = inputs()
        assert not end.query(), "the call ran too early for this test to say anything"
        for t in taken:
            lo, hi = t.data_ptr(), t.data_ptr() + t.numel() * t.element_size()
            assert all(hi <= a or b <= lo for a, b in spans)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        for made in (h, h1, h2):
            if made is not None:
                buf.destroy_handle(made)
    finally:
        torch.cuda.synchronize()
        buf.close()


@pytest.mark.parametrize("path", ["direct", "once_per_rank"])
def test_calls_keep_their_order_on_whatever_stream_each_runs(hx, path):
    """Calls without an event run on the stream they are made on, one after the other: from two streams, behind an
    overlapping call, and, once the communication stream has been asked for, behind what is queued there.  On a stream that
    torch did not make, and under graph capture, the communication stream takes them."""
    from paper_2603_13606_amd.buffer import EPBuffer
    R, E, H, K, T = 4, 16, 512, 4, 256
    gen = torch.Generator(hx.DEV).manual_seed(12)
    topk = [torch.randint(0, E, (T, K), generator=gen, device=hx.DEV, dtype=torch.int32) for _ in range(3)]
    gate = torch.rand((T, K), generator=gen, device=hx.DEV)
    xs = [torch.randn((T, H), generator=gen, device=hx.DEV).bfloat16() for _ in range(3)]
    buf = EPBuffer(R, E, H, K, max_tokens_per_rank=T, mode="ht", dispatch_path=path)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    try:
        want = []
        for i in range(3):
            r = buf.dispatch(xs[i], topk[i], gate)
            want.append([t.clone() for t in r[:3]] + [buf.combine(r[0], r[3], gate)[0].clone()])
            buf.destroy_handle(r[3])
        torch.cuda.synchronize()
        early = buf.capture()
        with torch.cuda.stream(a):
            torch.cuda._sleep(50_000_000)
            r0 = buf.dispatch(xs[0], topk[0], gate)
        with torch.cuda.stream(b):
            r1 = buf.dispatch(xs[1], topk[1], gate)
            r2 = buf.dispatch(xs[2], topk[2], gate, previous_event=early)
            outs = [buf.combine(r[0], r[3], gate) for r in (r0, r1, r2)]
        assert not r0[4].query(), "the first call ran too early for this test to say anything"
        r1[4].synchronize()
        assert r0[4].query()
        r2[4].synchronize()
        outs[2][1].synchronize()
        for r, o, w in zip((r0, r1, r2), outs, want):
            assert all(torch.equal(x.view(torch.int16) if x.dtype == torch.bfloat16 else x, y.view(torch.int16) if y.dtype == torch.bfloat16 else y)
                       for x, y in zip([*r[:3], o[0]], w))
            buf.destroy_handle(r[3])
        outside = torch.cuda.ExternalStream(a.cuda_stream)
        with torch.cuda.stream(outside):
            assert buf._start(None)[1] is buf._comm
            r = buf.dispatch(xs[0], topk[0], gate)
        r[4].synchronize()
        assert torch.equal(r[0].view(torch.int16), want[0][0].view(torch.int16))
        buf.destroy_handle(r[3])
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            assert buf._start(None)[1] is buf._comm
            r = buf.dispatch(xs[1], topk[1], gate)
            out = buf.combine(r[0], r[3], gate)[0]
        for _ in range(3):
            r[0].zero_(), out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(r[0].view(torch.int16), want[1][0].view(torch.int16)) and torch.equal(out.view(torch.int16), want[1][3].view(torch.int16))
        h = r[3]
        r = buf.dispatch(xs[2], topk[2], gate)  # outside the capture again
        comm = buf.get_comm_stream()
        with torch.cuda.stream(comm):
            torch.cuda._sleep(50_000_000)
            queued = buf.capture()
        out, done = buf.combine(r[0], r[3], gate)
        assert not queued.query()
        done.synchronize()
        assert queued.query() and torch.equal(out.view(torch.int16), want[2][3].view(torch.int16))
        buf.destroy_handle(r[3])
        buf.destroy_handle(h)
    finally:
        torch.cuda.synchronize()
        buf.close()


@pytest.mark.parametrize("C", [0, 100])
def test_large_backward_through_strided_windows_and_special_values(hx, C):
    """12 000 rows of 8 KiB in windows with a pitch: 128 bytes more per row (two launches) and 16 more (rows that start
    anywhere in a line, one launch).  Same bits, infinities and NaN among gradients, weights and expert outputs
    included; the row gradients are the float32 product rounded once, the weight gradients the float64 sums within
    the bound of a float32 sum of 4096 terms added 16 to a thread, 64 threads, 4 waves."""
    from paper_2603_13606_amd import binding as ep
    from test_gpu_parity import _kernel_launches
    E, T, H, K = 128, 1500, 4096, 8
    gen = torch.Generator(hx.DEV).manual_seed(C + 1)
    topk = torch.randint(0, E, (T, K), generator=gen, device=hx.DEV, dtype=torch.int32)
    topk[::7, 3] = -1
    w = torch.rand((T, K), generator=gen, device=hx.DEV)
    w[5, 1], w[6, 2], w[7, 0] = float("inf"), float("nan"), 0.0
    gs = torch.randn((T, H + 64), generator=gen, device=hx.DEV).bfloat16()
    g = gs[:, :H]
    g[9, 100], g[10, 200], g[11, 4095] = float("inf"), float("nan"), float("-inf")
    rows = E * C if C else T * K
    y = torch.randn((rows, H), generator=gen, device=hx.DEV).bfloat16()
    y[40, 7], y[41, 8] = float("inf"), float("nan")
    group = ep.ep_group_create(ep.make_config(8, E, H, K, T, mode=ep.EP_MODE_LL if C else ep.EP_MODE_HT, slots_per_subregion=C))
    try:
        h = ep.ep_layout(group, topk)
        dst = ep.read_device_i32(ep.ep_handle_query(h).dst_row, T * K).view(T, K).to(hx.DEV).long()
        got = []
        for gap, launches in ((64, 2), (8, 1)):
            def win(fill):
                s = torch.full((rows, H + gap), 7.0, dtype=torch.bfloat16, device=hx.DEV)
                s[:, :H] = fill
                return s, (s.view(E, C, H + gap) if C else s)[..., :H]
            ys, gys = win(y), win(7.0)
            gw = torch.full((T, K), 7.0, device=hx.DEV)
            call = lambda s=None: ep.ep_combine_backward(h, g, gys[1], topk_weights=w, y=ys[1], grad_w=gw, stream=s)
            call()
            torch.cuda.synchronize()
            assert torch.all(gys[0][:, H:] == 7.0)
            got.append((gys[0][:, :H].clone(), gw))
            assert _kernel_launches(ep, call) == launches
        assert torch.equal(got[0][0].view(torch.int16), got[1][0].view(torch.int16))
        assert torch.equal(got[0][1].view(torch.int32), got[1][1].view(torch.int32))
        gy, gw = got[0]
        has = dst >= 0
        want = torch.full((rows, H), 7.0, dtype=torch.bfloat16, device=hx.DEV)
        for k in range(K):
            m = has[:, k]
            want[dst[m, k]] = (w[m, k, None] * g[m].float()).bfloat16()
        assert torch.equal(torch.isnan(gy), torch.isnan(want)) and torch.equal(gy.nan_to_num(nan=3.0), want.nan_to_num(nan=3.0))
        assert torch.all(gw[~has] == 0.0)
        for k in range(K):
            m = has[:, k]
            terms = y[dst[m, k]].double() * g[m].double()
            ref, mag, out = terms.sum(1), terms.abs().sum(1), gw[m, k].double()
            fin = torch.isfinite(ref)
            assert torch.equal(torch.isnan(out), torch.isnan(ref)) and torch.equal(out[torch.isinf(ref)], ref[torch.isinf(ref)])
            assert torch.all((out - ref).abs()[fin] <= (16 + 6 + 3 + 1) * 2.0 ** -24 * mag[fin])
        ep.ep_handle_destroy(h)
    finally:
        torch.cuda.synchronize()
        ep.ep_group_destroy(group)


@pytest.mark.parametrize("mode", ["ht", "ll"])
def test_buffer_autograd_reuses_handle(hx, oracle_mod, mode):
    """One handle through forward and backward of the autograd wrappers: the gradients that come
    out are the composition of the backward calls checked above with the stand-in experts'
    own backward (torch), compared bit for bit with that composition run by hand on the GPU
    tensors, and with a dense float64 reference at the precision bf16 intermediates allow."""
    from paper_2603_13606_amd.buffer import EPBuffer, EPCombineFn, EPDispatchFn
    w = wl.make_workload("tiny")
    spec = w.spec
    buf = EPBuffer(spec.R, spec.E, spec.H, spec.K, max_tokens_per_rank=spec.T, mode=mode)
    try:
        topk = torch.from_numpy(w.topk_idx).to(hx.DEV)
        x = hx.bits_to_dev(w.x_bits).requires_grad_(True)
        gate = torch.from_numpy(w.topk_w).to(hx.DEV).requires_grad_(True)
        scale = (1.0 + torch.arange(spec.E, device=hx.DEV, dtype=torch.float32) / 8.0)
        # forward: handle created by a first dispatch, then reused by the autograd functions
        _, _, _, h, _ = buf.dispatch(x.detach(), topk)
        recv = EPDispatchFn.apply(x, buf, h)
        if mode == "ll":
            row_scale = scale[:, None, None].expand(spec.E, spec.T, 1)
        else:
            counts = torch.bincount(topk.reshape(-1).long(), minlength=spec.E)
            row_scale = torch.repeat_interleave(scale, counts)[:, None]
        y = (recv.float() * row_scale).to(torch.bfloat16)   # stand-in experts
        y.retain_grad()
        out = EPCombineFn.apply(y, gate, buf, h)
        G = torch.randn(spec.T, spec.H, device=hx.DEV, generator=torch.Generator(hx.DEV).manual_seed(3)).bfloat16()
        (out.float() * G.float()).sum().backward()
        torch.cuda.synchronize()
        # the same backward by hand: combine_backward, the experts' backward, unweighted combine
        gy, gw, _ = buf.combine_backward(G, h, gate.detach(), y.detach())
        g_recv = (gy.float() * row_scale).to(torch.bfloat16)
        gx, _ = buf.combine(g_recv, h)
        torch.cuda.synchronize()
        assert torch.equal(y.grad, gy) and torch.equal(gate.grad, gw) and torch.equal(x.grad, gx)
        # dense float64 reference
        xd = x.detach().double()
        wd = gate.detach().double()
        s = scale.double()[topk.long()]                      # [T, K]
        coef = (wd * s).sum(1)                               # [T]
        out_ref = xd * coef[:, None]
        assert torch.allclose(out.detach().double(), out_ref, rtol=2 ** -6, atol=1e-6)
        gx_ref = G.double() * coef[:, None]
        gw_ref = s * (xd * G.double()).sum(1)[:, None]
        assert torch.allclose(x.grad.double(), gx_ref, rtol=2 ** -5, atol=2e-2)
        # y is x * s rounded to bf16 (relative error 2^-9 per element): the dot products inherit it
        mag = s * (xd.abs() * G.double().abs()).sum(1)[:, None]
        assert torch.all((gate.grad.double() - gw_ref).abs() <= 2 ** -8 * mag + 1e-6)
        buf.destroy_handle(h)
    finally:
        buf.close()


def test_buffer_destination_order_gives_the_same_tensors(hx):
    """A buffer configured for the destination order (its dispatch announces the tokens to the
    layout call) returns bit for bit what the default buffer returns."""
    from paper_2603_13606_amd import binding as ep
    from paper_2603_13606_amd.buffer import EPBuffer
    w = wl.make_workload("ll_decode", T=1100, H=512)
    spec = w.spec
    topk = torch.from_numpy(w.topk_idx).to(hx.DEV)
    x = hx.bits_to_dev(w.x_bits)
    gate = torch.from_numpy(w.topk_w).to(hx.DEV)
    got = []
    for order in (ep.EP_ORDER_TOKEN, ep.EP_ORDER_DESTINATION):
        buf = EPBuffer(spec.R, spec.E, spec.H, spec.K, max_tokens_per_rank=spec.T, mode="ht", dispatch_order=order)
        try:
            recv_x, recv_src, recv_w, h, _ = buf.dispatch(x, topk, gate)
            n = sum(buf.get_tokens_per_expert_list())
            out, _ = buf.combine(recv_x, h, gate)
            torch.cuda.synchronize()
            got.append((hx.dev_to_bits(recv_x[:n]), recv_src[:n].cpu().numpy(), recv_w[:n].cpu().numpy(),
                        hx.dev_to_bits(out), n))
            buf.destroy_handle(h)
        finally:
            buf.close()
    assert got[0][4] == got[1][4] == spec.T * spec.K
    for a, b in zip(got[0][:4], got[1][:4]):
        assert np.array_equal(a, b)
