"""hmoe_route_ffn_combine against the calls it stands for, at the sizes where its dispatch changes."""
import numpy as np
import pytest
import torch

import workloads as wl
from hmoe_testlib import build_layer, desc_of, to_device

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def hm():
    import paper_2504_05897_amd as module
    return module


@pytest.mark.parametrize("E,K,hidden,ffn,shared_ffn,tokens", [
    (8, 2, 128, 192, (64,), (1, 3, 8, 9)),          # 9 tokens: routing in a launch of its own
    (64, 6, 256, 64, (192,), (1, 8)),
    (64, 8, 64, 320, (), (1, 8)),                   # 64 assignments, the most
    (65, 9, 64, 64, (64,), (1, 7, 8)),              # two experts per lane; 63 and 72 assignments
    (256, 32, 64, 64, (), (1, 2, 3)),               # 64 and 96 assignments
    (200, 3, 128, 64, (448,), (2, 8)),              # more shared groups than routed ones: several grid rows
    (1, 1, 64, 128, (), (1, 8)),
    (16, 4, 64, 8192, (64,), (1, 4)),               # 200 blocks and more: eight waves
    (96, 8, 128, 512, (64,), (3, 8)),               # the same with two experts per lane
    (200, 8, 128, 512, (), (8,)),                   # and with four
])
def test_route_ffn_combine_equals_the_separate_calls(hm, E, K, hidden, ffn, shared_ffn, tokens):
    """Every output the same bits as hmoe_route_permute, the FFN call and hmoe_combine; ties and masked logits among them."""
    shape = wl.small_shape(dtype=wl.BF16, hidden=hidden, ffn=ffn, n_experts=E, top_k=K, shared_ffn=shared_ffn, x_mode="rmsnorm")
    lay = wl.make_layer(shape, 21 + E, max(tokens))
    layer = build_layer(hm, lay, max_tokens=max(tokens))
    d, sd, c = layer.desc, layer.shared_desc, layer.cache
    rng = np.random.default_rng(E + K)
    for T in tokens:
        print("route_ffn_combine", E, K, hidden, ffn, shared_ffn, T, flush=True)
        lg = rng.standard_normal((T, E)).astype(np.float32)
        lg[0] = np.round(lg[0])                                       # ties
        if E > K:
            lg[T - 1, : (E - K) // 2] = -np.inf                       # masked experts
        lg = to_device(lg)
        x = to_device(lay.x[:T])
        if sd is not None:
            layer.shared_offsets.copy_(torch.tensor([0, T], dtype=torch.int32))
        shared = (sd, layer.shared_cache, layer.shared_offsets) if sd is not None else (None, None, None)
        outs = []
        for fused in (True, False):
            layer.ffn_ws.fill_(0xFF)
            idx, w = torch.full((T, K), -7, dtype=torch.int32, device=DEV), torch.full((T, K), 7.0, device=DEV)
            offs = torch.full((E + 1,), -7, dtype=torch.int32, device=DEV)
            perm, inv = (torch.full((T * K,), -7, dtype=torch.int32, device=DEV) for _ in range(2))
            o = torch.full((T * K, hidden), 7.0, dtype=torch.bfloat16, device=DEV)
            osh = torch.full((T, hidden), 7.0, dtype=torch.bfloat16, device=DEV) if sd is not None else None
            sws = (layer.shared_ws, layer.shared_ws_bytes) if sd is not None else (None, 0)
            y = torch.full((T, hidden), 7.0, dtype=torch.bfloat16, device=DEV)
            if fused:
                hm.hmoe_route_ffn_combine(d, c, x, lg, T, idx, w, offs, perm, inv, layer.perm_ws, layer.perm_ws_bytes, o, layer.ffn_ws,
                                          layer.ffn_ws_bytes, *shared, osh, *sws, y)
            else:
                hm.hmoe_route_permute(d, lg, T, idx, w, offs, perm, inv, None, layer.perm_ws, layer.perm_ws_bytes)
                hm.hmoe_expert_ffn_grouped_gather(d, c, x, perm, offs, T * K, None, o, layer.ffn_ws, layer.ffn_ws_bytes)
                if sd is not None:
                    hm.hmoe_expert_ffn_grouped(*shared[:2], x, layer.shared_offsets, T, None, osh, *sws)
                hm.hmoe_combine(d, o, inv, w, osh, T, y)
            torch.cuda.synchronize()
            outs.append([t.cpu() for t in (idx, w, offs, perm, inv, o, y) + (() if osh is None else (osh,))])
        for a, b in zip(*outs):
            assert torch.equal(a, b), T
    with pytest.raises(hm.HmoeError) as ei:                           # refused before anything is enqueued
        hm.hmoe_route_ffn_combine(d, c, x, lg, 1, idx, w, offs, perm, inv, layer.perm_ws, 0, o, layer.ffn_ws, layer.ffn_ws_bytes,
                                  *shared, osh, *sws, y)
    assert ei.value.status == hm.HMOE_ERR_WORKSPACE
    with pytest.raises(hm.HmoeError) as ei:
        hm.hmoe_route_ffn_combine(d, c, x, lg, 1, idx, w, offs, perm, inv, layer.perm_ws.data_ptr() + 2, layer.perm_ws_bytes, o, layer.ffn_ws,
                                  layer.ffn_ws_bytes, *shared, osh, *sws, y)
    assert ei.value.status == hm.HMOE_ERR_INVALID_ARG
    layer.close()


# A logit of bits 0xFFFFFFFF (the lowest NaN) sorts like a retired expert: a token with fewer others than K names one expert
# several times, and an expert then has more rows than the batch has tokens (15 to 31: up to four passes of the decode kernel).
@pytest.mark.parametrize("E,K,T,rows_nan", [(16, 8, 8, (3,)), (16, 8, 8, (0, 5, 7)), (72, 9, 7, (0, 1, 6)), (200, 4, 8, tuple(range(7)))])
def test_route_ffn_combine_of_an_expert_with_more_rows_than_tokens(hm, E, K, T, rows_nan):
    """The same bits as the separate calls, of the ordinary tokens beside them above all."""
    print("route_ffn_combine lowest NaN", E, K, T, rows_nan, flush=True)
    shape = wl.small_shape(dtype=wl.BF16, hidden=128, ffn=192, n_experts=E, top_k=K, x_mode="rmsnorm")
    lay = wl.make_layer(shape, 5 + E, T)
    layer = build_layer(hm, lay, max_tokens=T)
    d, c = layer.desc, layer.cache
    lg = np.random.default_rng(E).standard_normal((T, E)).astype(np.float32)
    lg[:, 0] += 9.0                                                   # expert 0: every ordinary token's first choice
    lg.view(np.uint32)[list(rows_nan)] = 0xFFFFFFFF
    lg, x = to_device(lg), to_device(lay.x)
    outs = []
    for fused in (True, False):
        layer.ffn_ws.fill_(0xFF)
        o, y = layer.o_perm.fill_(7.0), layer.y.fill_(7.0)
        bufs = (layer.topk_idx, layer.topk_w, layer.offsets, layer.perm, layer.inv_perm)
        if fused:
            hm.hmoe_route_ffn_combine(d, c, x, lg, T, *bufs, layer.perm_ws, layer.perm_ws_bytes, o, layer.ffn_ws, layer.ffn_ws_bytes,
                                      None, None, None, None, None, 0, y)
        else:
            hm.hmoe_route_permute(d, lg, T, *bufs, None, layer.perm_ws, layer.perm_ws_bytes)
            hm.hmoe_expert_ffn_grouped_gather(d, c, x, layer.perm, layer.offsets, T * K, None, o, layer.ffn_ws, layer.ffn_ws_bytes)
            hm.hmoe_combine(d, o, layer.inv_perm, layer.topk_w, None, T, y)
        torch.cuda.synchronize()
        outs.append([t.cpu().view(torch.int16) for t in bufs + (o, y)])
    rows = outs[0][2].view(torch.int32)
    assert int(rows[1] - rows[0]) == K * len(rows_nan) + T - len(rows_nan) > 8
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    layer.close()


# The router spread over blocks of 16 experts with the routing inside the decode launch, as a layer with a router runs them: one and
# several blocks, the last one not full, one, two and four experts per lane, both widths of the launch; T = 9 and 17 leave them.
@pytest.mark.parametrize("E,K,hidden,ffn,shared_ffn,tokens", [
    (16, 2, 128, 64, (), (1, 8)), (17, 4, 64, 128, (64,), (1, 8, 9)), (64, 6, 128, 640, (128,), (1, 7, 17)), (90, 8, 128, 64, (64,), (1, 8)),
    (100, 8, 64, 512, (), (2, 8)), (129, 5, 256, 64, (), (1, 8)), (256, 8, 128, 512, (64,), (1, 8, 9)),
])
def test_forward_with_a_router_of_many_experts_equals_the_calls(hm, E, K, hidden, ffn, shared_ffn, tokens):
    """MoELayer.forward against hmoe_router_route_permute, the FFN calls and hmoe_combine: the same bits in every output."""
    shape = wl.small_shape(dtype=wl.BF16, hidden=hidden, ffn=ffn, n_experts=E, top_k=K, shared_ffn=shared_ffn, x_mode="rmsnorm")
    lay = wl.make_layer(shape, 40 + E, max(tokens))
    one, calls = (build_layer(hm, lay, max_tokens=max(tokens)) for _ in range(2))
    d, c = calls.desc, calls.cache
    for T in tokens:
        print("forward with a router", E, K, T, flush=True)
        x = to_device(lay.x[:T])
        y = one.forward(x)
        hm.hmoe_router_route_permute(d, x, calls.w_router, T, calls.logits, calls.topk_idx, calls.topk_w, calls.offsets, calls.perm,
                                     calls.inv_perm, None, calls.perm_ws, calls.perm_ws_bytes)
        hm.hmoe_expert_ffn_grouped_gather(d, c, x, calls.perm, calls.offsets, T * K, None, calls.o_perm, calls.ffn_ws, calls.ffn_ws_bytes)
        if shared_ffn:
            bounds = torch.tensor([0, T], dtype=torch.int32, device=DEV)
            hm.hmoe_expert_ffn_grouped(calls.shared_desc, calls.shared_cache, x, bounds, T, None, calls.o_shared, calls.shared_ws,
                                       calls.shared_ws_bytes)
        hm.hmoe_combine(d, calls.o_perm, calls.inv_perm, calls.topk_w, calls.o_shared if shared_ffn else None, T, calls.y)
        torch.cuda.synchronize()
        assert y.abs().amax() > 1e-3
        for n, rows in (("logits", T), ("topk_idx", T), ("topk_w", T), ("offsets", E + 1), ("perm", T * K), ("inv_perm", T * K),
                        ("o_perm", T * K), ("y", T)):
            assert torch.equal(getattr(one, n)[:rows].cpu(), getattr(calls, n)[:rows].cpu()), (T, n)
    one.close()
    calls.close()


@pytest.mark.parametrize("dtype,shared_ffn,n_slots,logits_mode,tokens", [
    ("bf16", (64,), 8, "zipf", (1, 8, 9, 32, 33, 70)),      # shared experts in the routed launches, then beside them
    ("bf16", (64,), 8, "router", (1, 16, 17, 33, 5)),
    ("bf16", (), 8, "router", (2, 40)),
    ("bf16", (128,), 3, "zipf", (4, 40, 1)),                # staged, several waves
    ("w4", (128,), 8, "zipf", (1, 16, 17)),
    ("f32", (64,), 8, "router", (1, 33)),
    ("f32", (), 4, "zipf", (3, 20)),
])
def test_forward_in_one_call_equals_the_calls(hm, dtype, shared_ffn, n_slots, logits_mode, tokens):
    """MoELayer.forward (one library call) against the same layer with its switches set to make the calls itself: the same
    bits, plans and slot maps, for batches of changing size, eagerly on a stream of the caller's."""
    hidden, ffn = (128, 256) if dtype == "w4" else (128, 192)
    shape = wl.small_shape(dtype=wl.F32 if dtype == "f32" else wl.BF16, hidden=hidden, ffn=ffn, n_experts=8, top_k=2,
                           shared_ffn=shared_ffn, x_mode="rmsnorm", logits_mode=logits_mode)
    base = wl.make_layer(shape, 61, 1)
    d = hm.make_desc(hidden, ffn, 8, 2, n_slots, {"bf16": hm.HMOE_BF16, "f32": hm.HMOE_F32, "w4": hm.HMOE_BF16_W4}[dtype])
    one, calls = (hm.MoELayer(d, base.experts, base.shared, base.w_router, max_tokens=max(tokens)) for _ in range(2))
    calls.overlap_shared = calls.merge_shared = False
    stream = torch.cuda.Stream()
    for rep, T in enumerate(tokens):
        print("forward in one call", dtype, shared_ffn, n_slots, T, flush=True)
        lay = wl.make_layer(shape, 100 + rep, T, with_weights=False)
        x = to_device(lay.x)
        lg = None if logits_mode == "router" else to_device(lay.logits)
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            a, b = one.forward(x, lg), calls.forward(x, lg)
            stream.synchronize()
        for p, q in ((a, b), (one.topk_w[:T], calls.topk_w[:T]), (one.perm[:2 * T], calls.perm[:2 * T]), (one.offsets, calls.offsets)):
            assert torch.equal(p.cpu(), q.cpu()), T
        assert one.slot_map() == calls.slot_map() and one.staged_bytes == calls.staged_bytes
        if n_slots < 8:
            assert all(np.array_equal(p, q) for p, q in zip(one.last_plan, calls.last_plan))
    one.close()
    with pytest.raises(hm.HmoeError):
        one.forward(x, lg)
    calls.close()


@pytest.mark.parametrize("dtype,sizes", [("w4", (4, 1)), ("w4", (1, 70)), ("bf16", (40, 33)), ("bf16", (8, 64)), ("f32", (3, 20))])
def test_graphs_of_several_batch_sizes_on_one_layer(hm, dtype, sizes):
    """Shared experts beside the routed ones: a replayed graph computes the rows of its own batch, in whatever order graphs and
    eager calls of other sizes come."""
    print("graphs of several batch sizes", dtype, sizes, flush=True)
    shape = wl.small_shape(dtype=wl.F32 if dtype == "f32" else wl.BF16, hidden=128, ffn=256, n_experts=8, top_k=2, shared_ffn=(128,),
                           x_mode="rmsnorm")
    base = wl.make_layer(shape, 77, 1)
    d = hm.make_desc(128, 256, 8, 2, 8, {"bf16": hm.HMOE_BF16, "f32": hm.HMOE_F32, "w4": hm.HMOE_BF16_W4}[dtype])
    layer, alone = (hm.MoELayer(d, base.experts, base.shared, base.w_router, max_tokens=max(sizes)) for _ in range(2))
    xs = [to_device(wl.make_layer(shape, 80 + T, T, with_weights=False).x) for T in sizes]
    want = [alone.forward(x).cpu().clone() for x in xs]
    graphs = []
    for x in xs:                                          # (the first call with each size is the one that is captured)
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            layer.forward(x)
    for i in (0, 1, 1, 0, 0, 1):
        layer.y.fill_(7.0)
        layer.o_shared.fill_(7.0)
        graphs[i].replay()
        torch.cuda.synchronize()
        assert torch.equal(layer.y[:sizes[i]].cpu(), want[i]), i
        eager = layer.forward(xs[1 - i]).cpu()            # an eager call of the other size before the next replay
        assert torch.equal(eager, want[1 - i]), i
    layer.close()
    alone.close()


@pytest.mark.parametrize("dtype,shared_ffn,n_slots,logits_mode", [("bf16", (), 8, "zipf"), ("bf16", (64,), 8, "router"), ("f32", (), 8, "router"),
                                                                  ("bf16", (64,), 3, "zipf")])
def test_an_empty_batch_leaves_zero_offsets(hm, dtype, shared_ffn, n_slots, logits_mode):
    """forward(x[:0]) says that no expert has rows, as the routing call does, whatever the batch before it was."""
    print("empty batch", dtype, shared_ffn, n_slots, flush=True)
    shape = wl.small_shape(dtype=wl.F32 if dtype == "f32" else wl.BF16, hidden=128, ffn=192, n_experts=8, top_k=2, shared_ffn=shared_ffn,
                           x_mode="rmsnorm", logits_mode=logits_mode)
    lay = wl.make_layer(shape, 9, 5)
    layer = build_layer(hm, lay, max_tokens=5, n_slots=n_slots)
    x, lg = to_device(lay.x), None if logits_mode == "router" else to_device(lay.logits)
    for T in (5, 0, 3, 0):
        y = layer.forward(x[:T], None if lg is None else lg[:T])
        torch.cuda.synchronize()
        assert y.shape == (T, 128) and int(layer.offsets[-1]) == 2 * T
        if T == 0:
            assert not layer.offsets.any()
    if dtype == "bf16":
        layer.offsets.fill_(-7)
        hm.hmoe_route_ffn_combine(layer.desc, layer.cache, x, lg, 0, None, None, layer.offsets, None, None, layer.perm_ws,
                                  layer.perm_ws_bytes, None, None, 0, None, None, None, None, None, 0, None)
        torch.cuda.synchronize()
        assert not layer.offsets.any()
    layer.close()


@pytest.mark.parametrize("dtype,shared_ffn,T", [("bf16", (64,), 3), ("bf16", (64,), 40), ("f32", (), 5)])
def test_replaced_buffers_and_streams_are_used(hm, dtype, shared_ffn, T):
    """A layer's attributes may be replaced between two passes, a tensor also through its `data`: the next pass reads the new
    router and writes the new buffers, and the old ones stay as they were."""
    print("replaced buffers", dtype, shared_ffn, T, flush=True)
    shape = wl.small_shape(dtype=wl.F32 if dtype == "f32" else wl.BF16, hidden=128, ffn=192, n_experts=8, top_k=2, shared_ffn=shared_ffn,
                           x_mode="rmsnorm")
    lay, other = wl.make_layer(shape, 31, T), wl.make_layer(shape, 32, T)
    x = to_device(lay.x)
    want = {}
    for name, router in (("first", lay.w_router), ("second", other.w_router)):
        fresh = hm.MoELayer(desc_of(hm, shape), lay.experts, lay.shared, router, max_tokens=T)
        want[name] = fresh.forward(x).cpu().clone()
        fresh.close()
    layer = build_layer(hm, lay, max_tokens=T)
    assert torch.equal(layer.forward(x).cpu(), want["first"])
    kept = {}
    for n in ("logits", "topk_idx", "topk_w", "offsets", "perm", "inv_perm", "o_perm", "y", "perm_ws", "ffn_ws") + \
            (("o_shared", "shared_ws") if shared_ffn else ()):
        kept[n] = getattr(layer, n)
        setattr(layer, n, torch.empty_like(kept[n]))
    before = {n: t.cpu().clone() for n, t in kept.items()}
    layer.w_router = to_device(other.w_router)
    layer.side_stream = torch.cuda.Stream()
    y = layer.forward(x)
    torch.cuda.synchronize()
    assert y.data_ptr() == layer.y.data_ptr() and torch.equal(y.cpu(), want["second"])
    for n, t in kept.items():
        assert torch.equal(t.cpu().view(torch.uint8), before[n].view(torch.uint8)), n
    second = layer.w_router.data
    layer.w_router.data = to_device(lay.w_router)
    assert torch.equal(layer.forward(x).cpu(), want["first"]) and second.data_ptr() != layer.w_router.data_ptr()
    layer.close()
