"""Front end at the sizes where its dispatch changes: block shapes of the router, ways of the permutation."""
import numpy as np
import pytest
import torch

import workloads as wl
from hmoe_testlib import to_device
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def hm():
    import paper_2504_05897_amd as module
    return module


@pytest.mark.parametrize("T,E,K", [(16384, 5, 1), (16385, 5, 1), (8192, 256, 2), (5462, 64, 3), (262144, 3, 1), (262145, 3, 1),
                                   (87383, 130, 3), (1025, 1, 1), (1536, 2, 2), (513, 64, 2), (4096, 1, 1), (4096, 5, 1),
                                   (2048, 2, 2), (586, 256, 7), (4097, 1, 1), (4097, 200, 1)])
def test_permute_at_the_edges_of_its_ways(hm, T, E, K):
    """4 and 256 chunks of 1024 assignments are the last of the one- and two-launch ways; few experts, or most rows at one
    of them, are keys that lanes of a wave share."""
    print("permute edges", T, E, K, flush=True)
    rng = np.random.default_rng(T + E)
    idx = np.minimum(rng.geometric(0.2, (T, K)) - 1, E - 1).astype(np.int32)
    d = hm.make_desc(64, 64, E, K, E, hm.HMOE_BF16)
    A = T * K
    offs = torch.full((E + 1,), -7, dtype=torch.int32, device=DEV)
    perm, inv = (torch.full((A,), -7, dtype=torch.int32, device=DEV) for _ in range(2))
    counts = torch.zeros(E, dtype=torch.int32, pin_memory=True)
    ws_bytes = hm.hmoe_permute_workspace_bytes(d, T)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device=DEV)
    hm.hmoe_permute(d, to_device(idx), T, None, None, offs, perm, inv, counts, ws, ws_bytes)
    torch.cuda.synchronize()
    ro, rp, ri = orc.permute(idx, E)
    assert np.array_equal(offs.cpu().numpy(), ro) and np.array_equal(counts.numpy(), np.diff(ro))
    assert np.array_equal(perm.cpu().numpy(), rp) and np.array_equal(inv.cpu().numpy(), ri)


@pytest.mark.parametrize("T,E,K,H", [(16, 8, 2, 48), (17, 8, 2, 48), (16, 64, 6, 2048), (16, 256, 32, 80), (64, 100, 8, 48), (4096, 16, 2, 64),
                                     (4097, 8, 2, 48), (4097, 33, 4, 80), (8192, 64, 6, 48), (8193, 64, 6, 48), (8193, 100, 6, 64),
                                     (8193, 200, 2, 16),
                                     # pieces of K with a remainder in every shape of the block, and pieces that are empty
                                     (20, 12, 2, 7184), (33, 30, 4, 2080), (5, 64, 8, 1104), (9, 96, 8, 1536), (20, 256, 8, 2064),
                                     (2049, 64, 6, 1104), (2100, 128, 4, 592), (3000, 33, 4, 80), (2200, 256, 8, 80), (4095, 12, 2, 48),
                                     (4097, 64, 6, 1104), (4097, 128, 4, 1104), (4100, 256, 8, 592)])
def test_router_block_shapes(hm, T, E, K, H):
    """Logits within fp32 summation error (|error| <= 2 H 2^-24 sum |x w|), the same bits for a token whatever its batch,
    and the fused call's integers equal to the oracle's for the logits it wrote."""
    print("router block shapes", T, E, K, H, flush=True)
    rng = np.random.default_rng(T + E + H)
    x = wl.store(rng.standard_normal((T, H)).astype(np.float32), wl.BF16)
    wg = wl.store(rng.standard_normal((E, H)).astype(np.float32) * 0.05, wl.BF16)
    d = hm.make_desc(H, 64, E, K, E, hm.HMOE_BF16)
    xd, wd = to_device(x), to_device(wg)
    lg = torch.full((T, E), 9.0, dtype=torch.float32, device=DEV)
    idx = torch.full((T, K), -5, dtype=torch.int32, device=DEV)
    w = torch.zeros(T, K, dtype=torch.float32, device=DEV)
    offs = torch.full((E + 1,), -7, dtype=torch.int32, device=DEV)
    perm, inv = (torch.full((T * K,), -7, dtype=torch.int32, device=DEV) for _ in range(2))
    ws_bytes = hm.hmoe_permute_workspace_bytes(d, T)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device=DEV)
    hm.hmoe_router_route_permute(d, xd, wd, T, lg, idx, w, offs, perm, inv, None, ws, ws_bytes)
    alone, single = torch.empty_like(lg), torch.empty(1, E, dtype=torch.float32, device=DEV)
    hm.hmoe_router_logits(d, xd, wd, T, alone)
    hm.hmoe_router_logits(d, xd[T - 1:].contiguous(), wd, 1, single)
    torch.cuda.synchronize()
    got = lg.cpu().numpy()
    assert np.array_equal(got, alone.cpu().numpy()) and np.array_equal(got[T - 1:], single.cpu().numpy())
    xf, wf = wl.as_f64(x), wl.as_f64(wg)
    assert (np.abs(got - xf @ wf.T) <= 2 * H * 2.0 ** -24 * (np.abs(xf) @ np.abs(wf).T)).all()
    ridx, rw = orc.route(got, K)
    ro, rp, ri = orc.permute(ridx, E)
    assert np.array_equal(idx.cpu().numpy(), ridx) and np.abs(w.cpu().numpy() - rw).max() < 1e-6
    assert np.array_equal(offs.cpu().numpy(), ro) and np.array_equal(perm.cpu().numpy(), rp) and np.array_equal(inv.cpu().numpy(), ri)


@pytest.mark.parametrize("T,E,K", [(1, 8, 8), (21, 64, 8), (64, 16, 3), (5, 30, 30), (40, 100, 9), (33, 256, 31)])
def test_equal_logits_go_to_the_smaller_id(hm, T, E, K):
    """Few distinct values (both zeros, both signs among them), so that most choices are ties within and across lanes."""
    print("ties", T, E, K, flush=True)
    rng = np.random.default_rng(T * E + K)
    lg = rng.choice(np.array([0.0, -0.0, 1.5, -2.0, 1e-38], np.float32), (T, E)).astype(np.float32)
    d = hm.make_desc(64, 64, E, K, E, hm.HMOE_BF16)
    ridx, rw = orc.route(lg, K)
    ro, rp, ri = orc.permute(ridx, E)
    for fused in (False, True):
        idx = torch.full((T, K), -5, dtype=torch.int32, device=DEV)
        w = torch.zeros(T, K, dtype=torch.float32, device=DEV)
        offs = torch.full((E + 1,), -7, dtype=torch.int32, device=DEV)
        perm, inv = (torch.full((T * K,), -7, dtype=torch.int32, device=DEV) for _ in range(2))
        ws_bytes = hm.hmoe_permute_workspace_bytes(d, T)
        ws = torch.empty(ws_bytes, dtype=torch.uint8, device=DEV)
        if fused:
            hm.hmoe_route_permute(d, to_device(lg), T, idx, w, offs, perm, inv, None, ws, ws_bytes)
        else:
            hm.hmoe_route(d, to_device(lg), T, idx, w)
            hm.hmoe_permute(d, idx, T, None, None, offs, perm, inv, None, ws, ws_bytes)
        torch.cuda.synchronize()
        assert np.array_equal(idx.cpu().numpy(), ridx) and np.abs(w.cpu().numpy() - rw).max() < 1e-6
        assert np.array_equal(offs.cpu().numpy(), ro) and np.array_equal(perm.cpu().numpy(), rp) and np.array_equal(inv.cpu().numpy(), ri)


@pytest.mark.parametrize("T,E,K", [(3, 8, 2), (40, 16, 3), (64, 30, 8), (200, 64, 6), (70, 100, 9), (33, 256, 31)])
def test_masked_and_undefined_logits(hm, T, E, K):
    """Experts masked with -inf or with the type's lowest value: the choice among the others is the oracle's, a token with fewer
    unmasked experts than K chooses those first and its masked ones with weight 0, no expert twice.  Logits that are NaN or +inf
    leave the result open, but ids stay ids and the permutation a permutation."""
    print("masked logits", T, E, K, flush=True)
    rng = np.random.default_rng(T + E + K)
    lg = rng.standard_normal((T, E)).astype(np.float32)
    masked = rng.random((T, E)) < 0.5
    masked[:, :1] = False
    lg[masked] = np.where(rng.random((T, E)) < 0.5, -np.inf, np.finfo(np.float32).min)[masked]
    odd = lg.copy()
    odd[rng.random((T, E)) < 0.2] = np.nan
    odd[::3, -1] = np.inf
    odd[1::3, 0] = np.array([0xFFC00000], np.uint32).view(np.float32)[0]  # NaN with its sign bit set
    d = hm.make_desc(64, 64, E, K, E, hm.HMOE_BF16)
    ws_bytes = hm.hmoe_permute_workspace_bytes(d, T)
    for values in (lg, odd):
        for fused in (False, True):
            idx = torch.full((T, K), -5, dtype=torch.int32, device=DEV)
            w = torch.zeros(T, K, dtype=torch.float32, device=DEV)
            offs = torch.full((E + 1,), -7, dtype=torch.int32, device=DEV)
            perm, inv = (torch.full((T * K,), -7, dtype=torch.int32, device=DEV) for _ in range(2))
            ws = torch.empty(ws_bytes, dtype=torch.uint8, device=DEV)
            if fused:
                hm.hmoe_route_permute(d, to_device(values), T, idx, w, offs, perm, inv, None, ws, ws_bytes)
            else:
                hm.hmoe_route(d, to_device(values), T, idx, w)
                hm.hmoe_permute(d, idx, T, None, None, offs, perm, inv, None, ws, ws_bytes)
            torch.cuda.synchronize()
            got = idx.cpu().numpy()
            assert got.min() >= 0 and got.max() < E
            ro, rp, ri = orc.permute(got, E)
            assert np.array_equal(offs.cpu().numpy(), ro) and np.array_equal(perm.cpu().numpy(), rp) and np.array_equal(inv.cpu().numpy(), ri)
            if values is lg:
                assert all(len(set(row)) == K for row in got.tolist())
                order = np.argsort(-values.astype(np.float64), axis=1, kind="stable")[:, :K]   # equal logits: smaller id first
                assert np.array_equal(got, order)
                chosen = np.take_along_axis(values, got, 1).astype(np.float64)
                ref = np.exp(chosen - chosen[:, :1])
                assert np.abs(w.cpu().numpy() - ref / ref.sum(1, keepdims=True)).max() < 1e-6


@pytest.mark.parametrize("memory", ["pinned", "inside pinned", "pageable"])
@pytest.mark.parametrize("T,E,K", [(3, 8, 2), (70, 64, 6), (300, 70, 6), (2000, 200, 8), (40000, 64, 7)])
def test_counts_and_scores_to_host_memory(hm, memory, T, E, K):
    """Pinned memory is written by the kernels, any other by a copy behind them: every way of the permutation and of the
    routing scores (one block, several), at an offset into an allocation too."""
    print("host memory", memory, T, E, K, flush=True)
    pinned = memory != "pageable"
    shift = 5 if memory == "inside pinned" else 0
    rng = np.random.default_rng(T + E)
    lg = rng.standard_normal((T, E)).astype(np.float32)
    d = hm.make_desc(64, 64, E, K, E, hm.HMOE_BF16)
    counts = torch.full((E + 2 * shift,), -7, dtype=torch.int32, pin_memory=pinned)
    scores_h = torch.full((E + 2 * shift,), -7.0, pin_memory=pinned)
    idx, w = torch.empty(T, K, dtype=torch.int32, device=DEV), torch.empty(T, K, device=DEV)
    offs = torch.empty(E + 1, dtype=torch.int32, device=DEV)
    perm, inv = (torch.empty(T * K, dtype=torch.int32, device=DEV) for _ in range(2))
    ws_bytes = max(hm.hmoe_permute_workspace_bytes(d, T), hm.hmoe_route_scores_workspace_bytes(d, T))
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device=DEV)
    scores = torch.empty(E, device=DEV)
    lg_dev = to_device(lg)
    hm.hmoe_route_permute(d, lg_dev, T, idx, w, offs, perm, inv, counts[shift:shift + E], ws, ws_bytes)
    torch.cuda.synchronize()
    hm.hmoe_route_scores(d, lg_dev, T, scores, scores_h[shift:shift + E], ws, ws_bytes)
    torch.cuda.synchronize()
    ridx, _ = orc.route(lg, K)
    ro, _, _ = orc.permute(ridx, E)
    assert np.array_equal(counts[shift:shift + E].numpy(), np.diff(ro))
    assert np.array_equal(scores_h[shift:shift + E].numpy(), scores.cpu().numpy())
    p = np.exp(lg.astype(np.float64) - lg.max(1, keepdims=True))
    ref = (p / p.sum(1, keepdims=True)).mean(0)
    # expf and the division to a few ulp, then fp32 sums of up to 64 tokens per wave and T / 64 partial sums
    assert np.abs(scores.cpu().numpy() - ref).max() <= (16 + 64 + T / 64) * 2.0 ** -24 * ref.max()
    if shift:
        assert set(counts[:shift].tolist() + counts[-shift:].tolist()) == {-7} and set(scores_h[:shift].tolist()) == {-7.0}
