"""Tile heights and ragged edges of the fp32 matrix kernels and the 4-bit prefill kernel, against the oracle in 64 bits."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import moe_oracle as orc
from oracle import w4_oracle as w4
from hmoe_testlib import TOL, desc_of, max_rel_err, to_device, to_host_f32

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def grouped_ffn(hm, d, experts, x_bits, offsets, path):
    A = int(offsets[-1])
    layer = hm.MoELayer(d, experts, (), None, max_tokens=A)
    o = torch.full((A, d.hidden), float("nan"), dtype=layer.dt, device=DEV)
    ws_bytes = hm.hmoe_ffn_workspace_bytes(d, A)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device=DEV)
    hm.hmoe_expert_ffn_grouped(d, layer.cache, to_device(x_bits), to_device(offsets), A, None, o, ws, ws_bytes, path)
    torch.cuda.synchronize()
    got = to_host_f32(o)
    layer.close()
    return got


def case(dtype, hidden, ffn, counts):
    shape = wl.small_shape(dtype=dtype, hidden=hidden, ffn=ffn, n_experts=len(counts), top_k=min(2, len(counts)))
    lay = wl.make_layer(shape, hidden + ffn, n_tokens=1)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    x = wl.store(np.random.default_rng(7).standard_normal((int(offsets[-1]), hidden)).astype(np.float32), dtype)
    return shape, lay, offsets, x


def reference(x, offsets, experts, hidden, to_f64):
    ref = np.zeros((int(offsets[-1]), hidden))
    for e, (lo, hi) in enumerate(zip(offsets[:-1], offsets[1:])):
        if hi > lo:
            ref[lo:hi] = orc.expert_ffn(wl.as_f64(x[lo:hi]), *(to_f64(m) for m in experts[e]))
    return ref


# one 16-row fragment per tile and two; K of one and several rounds of 128 (four waves, two pieces of 16 each) with remainders; widths
# that are no multiple of 16
@pytest.mark.parametrize("hidden,ffn,counts", [
    (256, 512, [1, 0, 16, 5]), (4, 8, [3, 1]), (260, 36, [17, 2, 0, 1]), (516, 772, [2, 9]),
    (256, 512, [31, 0, 33, 64, 1]), (100, 44, [40, 15]), (1028, 20, [65, 32]),
    # large enough for the tiles: one fragment per tile (fewer than 16 rows per expert on average), and two
    (516, 772, [1, 17, 0, 16, 5, 2, 0, 9]), (260, 1540, [2, 0, 15, 16, 3, 17, 1, 1, 0, 40, 5, 9]), (4, 33028, [65, 40]),
    (2052, 36, [33, 70, 64]), (1028, 300, [31, 0, 33, 64, 1]),
])
def test_ffn_f32_tiles(hm, hidden, ffn, counts):
    shape, lay, offsets, x = case(wl.F32, hidden, ffn, counts)
    d = desc_of(hm, shape, n_slots=len(counts))
    got = grouped_ffn(hm, d, lay.experts, x, offsets, hm.HMOE_FFN_AUTO)
    # the general kernels' 64 sums of K / 64 products each in fp32: at most 24 roundings of 2^-24 per GEMM at these sizes, and a
    # handful in silu: 2e-6 of the largest value, and as much again for cancellation (the tiles' 64-bit sums are closer)
    assert max_rel_err(got, reference(x, offsets, lay.experts, hidden, wl.as_f64)) < 4e-6
    general = grouped_ffn(hm, d, lay.experts, x, offsets, hm.HMOE_FFN_REFERENCE)
    # the calls that are too small for the tiles take the general kernels
    assert np.array_equal(got, general) == (12 * hidden * ffn * (int(offsets[-1]) - len(counts)) < 30e6)


# An explicit HMOE_FFN_REFERENCE takes the general kernels whatever the sizes.  Rows and columns of zeros behind the
# others leave every sum of theirs as it is, bit for bit, and make the sizes such that nothing else takes them.
@pytest.mark.parametrize("hidden,ffn,counts", [(72, 100, [3, 0, 7]), (256, 512, [31, 0, 33, 64, 1])])
def test_ffn_f32_reference_is_the_general_kernels(hm, hidden, ffn, counts):
    print("ffn f32 reference", hidden, ffn, counts, flush=True)
    shape, lay, offsets, x = case(wl.F32, hidden, ffn, counts)
    d = desc_of(hm, shape, n_slots=len(counts))
    got = grouped_ffn(hm, d, lay.experts, x, offsets, hm.HMOE_FFN_REFERENCE)
    assert max_rel_err(got, reference(x, offsets, lay.experts, hidden, wl.as_f64)) < 4e-6
    pad = lambda m, rows, cols: np.pad(m, ((0, rows - m.shape[0]), (0, cols - m.shape[1])))
    H, F = hidden + 1, ffn + 2
    wide = [(pad(g, F, H), pad(u, F, H), pad(w, H, F)) for g, u, w in lay.experts]
    dw = hm.make_desc(H, F, len(counts), 2, len(counts), hm.HMOE_F32)
    for path in (hm.HMOE_FFN_REFERENCE, hm.HMOE_FFN_AUTO):
        other = grouped_ffn(hm, dw, wide, pad(x, len(x), H), offsets, path)
        assert np.array_equal(other[:, :hidden], got) and not other[:, hidden:].any()


# every height of one tile (1 to 6 fragments), experts of several tiles with uneven heights, ragged last fragments, a
# column tile that is not full, and one, two, three and more scale groups (the ring holds three).  The last six have more
# than 256 tiles in one projection (the first four of them gate/up, with 3, 4, 5 and 7 scale groups and every height), which
# then takes the blocks of one set of waves; fewer take those of two sets.
@pytest.mark.parametrize("hidden,ffn,counts", [
    (256, 128, [1, 16, 17, 33, 49, 80, 81, 96]), (128, 256, [97, 0, 112, 113]), (384, 640, [193, 96, 290]),
    (512, 384, [64, 65]), (1152, 128, [95, 3]),
    # (the cases above take tiles of at most 2 fragments; gate/up of these of at most 2, 2, 4, then one set of waves with 4,
    # then two with 6)
    (256, 256, [33, 64, 65]), (640, 384, [129]), (1024, 1920, [64, 0, 129, 33, 16]), (1024, 4224, [128, 65]), (512, 8192, [256]),
    (128, 4096, [96, 33, 81, 49]), (2048, 4096, [96, 33, 81, 17]), (2176, 4096, [97, 17, 64, 80]), (2304, 4096, [49, 81, 90, 65]),
    # idle experts between busy ones, more than 64 and 128 of them, columns that eight does not divide
    (256, 1152, [i % 7 * 20 if i % 3 else 0 for i in range(130)]), (384, 640, [0, 130, 0, 0, 33, 300, 0, 1, 96, 97, 0, 5, 20, 64, 0, 2]),
    (384, 16768, [100]), (512, 4224, [1, 17, 33, 49, 80, 81, 96, 97]), (640, 4224, [97, 96, 2, 16, 47, 65, 81, 33]),
    (896, 4224, [193, 1, 17, 33, 49, 80, 81, 96]), (4096, 128, [97, 33, 16, 50, 81, 1, 2, 64, 96]), (4096, 640, [96, 34, 17, 51, 80, 2, 3, 64, 65]),
])
def test_ffn_w4_tile_heights(hm, hidden, ffn, counts):
    shape, lay, offsets, x = case(wl.BF16, hidden, ffn, counts)
    E = len(counts)
    d = hm.make_desc(hidden, ffn, E, 2 if E > 1 else 1, E, hm.HMOE_BF16_W4)
    got = grouped_ffn(hm, d, lay.experts, x, offsets, hm.HMOE_FFN_TILED)
    ref = reference(x, offsets, lay.experts, hidden, lambda m: w4.dequantize_w4(*w4.quantize_w4(wl.as_f32(m))))
    assert max_rel_err(got, ref) < TOL[wl.BF16]


# Inputs of 4 GiB and more: the intermediate of a wide expert, and tokens that the gate/up projection gathers from.
@pytest.mark.parametrize("hidden,ffn,rows,gather", [(128, 16384, 131200, False), (128, 16384, 131200, True), (4096, 128, 524400, True)])
def test_ffn_w4_large_inputs(hm, hidden, ffn, rows, gather):
    """Same bits as for the first and the last rows by themselves (a row's sums do not depend on the tile it is in), some rows
    against the oracle."""
    print("w4 large inputs", hidden, ffn, rows, gather, flush=True)
    shape, lay, _, _ = case(wl.BF16, hidden, ffn, [16])
    d = hm.make_desc(hidden, ffn, 1, 1, 1, hm.HMOE_BF16_W4)
    layer = hm.MoELayer(d, lay.experts, (), None, max_tokens=16)
    x = torch.randn(rows, hidden, device=DEV, generator=torch.Generator(DEV).manual_seed(3)).bfloat16()

    def ffn_of(xs):
        n = len(xs)
        o = torch.empty(n, hidden, dtype=torch.bfloat16, device=DEV)
        ws_bytes = hm.hmoe_ffn_workspace_bytes(d, n)
        ws = torch.empty(ws_bytes, dtype=torch.uint8, device=DEV)
        offsets = torch.tensor([0, n], dtype=torch.int32, device=DEV)
        if gather:  # the rows in descending order
            perm = torch.arange(n - 1, -1, -1, dtype=torch.int32, device=DEV)
            hm.hmoe_expert_ffn_grouped_gather(d, layer.cache, xs, perm, offsets, n, None, o, ws, ws_bytes, hm.HMOE_FFN_TILED)
            o = o.flip(0)
        else:
            hm.hmoe_expert_ffn_grouped(d, layer.cache, xs, offsets, n, None, o, ws, ws_bytes, hm.HMOE_FFN_TILED)
        torch.cuda.synchronize()
        return o

    got, part = ffn_of(x), 26000  # enough for more than one tile per CU, as the whole has
    assert torch.equal(got[:part], ffn_of(x[:part].contiguous()))
    assert torch.equal(got[-part:], ffn_of(x[-part:].contiguous()))
    some = [0, 1, rows // 2, rows - 2, rows - 1]
    ref = orc.expert_ffn(x[some].double().cpu().numpy(), *(w4.dequantize_w4(*w4.quantize_w4(wl.as_f32(m))) for m in lay.experts[0]))
    assert max_rel_err(to_host_f32(got[some]), ref) < TOL[wl.BF16]
    layer.close()


# the edges of the rule that gives a dense expert's down projection 256x128 tiles (more than 256 rows, K of 12288 or more,
# at most 192 tiles), widths that are no multiple of 128
@pytest.mark.parametrize("rows,hidden,ffn", [(256, 192, 12288), (257, 192, 12288), (300, 320, 12352), (513, 64, 12288),
                                             (300, 192, 12224), (12300, 448, 12288)])
def test_dense_down_tiles(hm, monkeypatch, rows, hidden, ffn):
    """Same bits as with the 128x256 tiles (a tile sums all of K in order), sampled rows against the oracle."""
    print("dense down", rows, hidden, ffn, flush=True)
    shape, lay, offsets, x = case(wl.BF16, hidden, ffn, [rows])
    d = hm.make_desc(hidden, ffn, 1, 1, 1, hm.HMOE_BF16)
    got = grouped_ffn(hm, d, lay.experts, x, offsets, hm.HMOE_FFN_TILED)
    monkeypatch.setenv("HMOE_TILED_VARIANT", "3")
    assert np.array_equal(got, grouped_ffn(hm, d, lay.experts, x, offsets, hm.HMOE_FFN_TILED))
    some = np.unique(np.r_[0:min(rows, 260):37, rows - 3:rows])
    ref = orc.expert_ffn(wl.as_f64(x[some]), *(wl.as_f64(m) for m in lay.experts[0]))
    assert max_rel_err(got[some], ref) < TOL[wl.BF16]


# experts of 320 rows and more on average: tiles of 64 x 256 where they make fewer rounds than the others.  Ragged heights, column
# tiles that are half full (gate/up and down), one to seven scale groups (four are in flight).
@pytest.mark.parametrize("hidden,ffn,counts", [(128, 8192, [1000, 40, 0, 300]), (384, 16768, [700]), (640, 8320, [512, 129]),
                                               (896, 4224, [650, 1, 700, 0]), (4224, 128, [1900, 77, 64])])
def test_ffn_w4_wide_tiles(hm, hidden, ffn, counts):
    print("w4 wide tiles", hidden, ffn, counts, flush=True)
    shape, lay, offsets, x = case(wl.BF16, hidden, ffn, counts)
    E = len(counts)
    d = hm.make_desc(hidden, ffn, E, min(2, E), E, hm.HMOE_BF16_W4)
    got = grouped_ffn(hm, d, lay.experts, x, offsets, hm.HMOE_FFN_TILED)
    some = np.unique(np.concatenate([np.r_[lo:hi:61, max(lo, hi - 2):hi] for lo, hi in zip(offsets[:-1], offsets[1:])])).astype(int)
    for e, (lo, hi) in enumerate(zip(offsets[:-1], offsets[1:])):
        rows = some[(some >= lo) & (some < hi)]
        if len(rows):
            ref = orc.expert_ffn(wl.as_f64(x[rows]), *(w4.dequantize_w4(*w4.quantize_w4(wl.as_f32(m))) for m in lay.experts[e]))
            assert max_rel_err(got[rows], ref) < TOL[wl.BF16], e


@pytest.fixture(scope="module")
def hm():
    import paper_2504_05897_amd as hm
    return hm
