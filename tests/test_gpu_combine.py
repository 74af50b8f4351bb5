"""hmoe_combine at the sizes where its dispatch changes: experts per token, block sizes, ways of loading."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def hm():
    import paper_2504_05897_amd as module
    return module


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,K,H,shared", [(3, 1, 72, True), (3, 2, 520, False), (64, 3, 72, True), (65, 4, 72, False), (2, 5, 2056, True),
                                          (5, 7, 72, False), (5, 8, 72, True), (5, 9, 72, True), (66, 16, 72, False), (3, 17, 520, True),
                                          (2, 32, 72, False),
                                          (4096, 3, 2048, True), (4095, 3, 2048, True), (1500, 9, 2240, False)])   # at, below and above 64 MiB (bf16)
def test_combine_dispatch(hm, dtype, T, K, H, shared):
    """Every element within the rounding of its type: fp32 sums of K (+ 1) terms, each term and each addition rounded
    once, then one rounding to bfloat16.  Rows that no token names hold NaN and must not be read into a sum."""
    print("combine", dtype, T, K, H, shared, flush=True)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device=DEV).manual_seed(T + K)
    A = T * K
    o = torch.randn(A + 1, H, device=DEV, generator=gen).to(td)
    o[A] = float("nan")
    osh = torch.randn(T, H, device=DEV, generator=gen).to(td) if shared else None
    w = torch.rand(T, K, device=DEV, generator=gen)
    inv = torch.randperm(A, device=DEV, generator=gen).int()
    d = hm.make_desc(H, 64, 64, K, 64, hm.HMOE_BF16 if dtype == "bf16" else hm.HMOE_F32)
    y = torch.empty(T, H, dtype=td, device=DEV)
    hm.hmoe_combine(d, o, inv, w, osh, T, y)
    terms = o[inv.long()].view(T, K, H).double() * w.double()[:, :, None]
    ref, size = terms.sum(1), terms.abs().sum(1)
    if shared:
        ref, size = ref + osh.double(), size + osh.double().abs()
    bound = (2 * K + 2) * 2.0 ** -24 * size + (2.0 ** -8 * ref.abs() if dtype == "bf16" else 0.0)
    assert bool(((y.double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("H", [66, 70])
def test_combine_of_fp32_rows_that_are_no_vectors(hm, H):
    T, K = 5, 3
    o, w = torch.randn(T * K, H, device=DEV), torch.rand(T, K, device=DEV)
    inv = torch.randperm(T * K, device=DEV).int()
    y = torch.empty(T, H, device=DEV)
    hm.hmoe_combine(hm.make_desc(H, 64, 64, K, 64, hm.HMOE_F32), o, inv, w, None, T, y)
    terms = o[inv.long()].view(T, K, H).double() * w.double()[:, :, None]
    assert bool(((y.double() - terms.sum(1)).abs() <= 8 * 2.0 ** -24 * terms.abs().sum(1)).all())
