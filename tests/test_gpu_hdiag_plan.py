"""hdiag at the edges of its plans: one launch for few tokens (16 rows at once
up to 256 tokens, 128 rows up to 1024 of few columns), short slices, slices moved off a
2 MB spacing, and the coarse slices of a smaller workspace."""
from __future__ import annotations

import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def hs():
    import paper_2608_28113_amd as hs
    assert torch.cuda.is_available()
    return hs


@pytest.mark.parametrize("T,n", [(1, 16), (15, 112), (128, 512), (256, 144), (257, 64), (1024, 1040), (1025, 1040),
                                 (1056, 4096), (2040, 4096), (4095, 528), (2048, 14336), (8192, 4096), (8193, 8192),
                                 (65537, 48), (1024, 16384), (1024, 16400), (896, 32768), (897, 32768),
                                 (257, 32784), (3, 262144), (3, 262160), (64, 262160)])
def test_hdiag_plans(hs, T, n):
    g = torch.Generator(device=DEV).manual_seed(T * 31 + n)
    X = (torch.randn((T, n), generator=g, device=DEV) * torch.exp(torch.randn(n, generator=g, device=DEV))).bfloat16()
    ref = X.double().square_().sum(0)
    h = hs.hdiag(X)
    # Slices of at least 256 tokens: what a workspace of that size is given.
    slices = max(1, min(1792 // -(-n // 512), -(-T // 256)))
    coarse = -(-T // -(-T // slices)) * n * 8
    assert coarse <= hs.hdiag_workspace_bytes(T, n)
    h_coarse = hs.hdiag(X, workspace=torch.empty(coarse, dtype=torch.uint8, device=DEV))
    h64 = torch.zeros(n, dtype=torch.float64, device=DEV)
    hs.hdiag_accumulate(X, h64)
    h_acc = hs.hdiag_finalize(h64)
    torch.cuda.synchronize()
    for name, v in (("hdiag", h), ("coarse", h_coarse), ("accumulated", h_acc)):
        rel = ((v.double() - ref).abs() / ref.clamp_min(1e-30)).max().item()
        print(f"[{T}x{n}] {name} max rel {rel:.2e}", flush=True)
        assert rel <= 2e-6  # chains of at most 32 fp32 additions: 31.5 x 2^-24
    assert torch.equal(h, h_acc)
    assert torch.equal(h, hs.hdiag(X))


@pytest.mark.parametrize("full,last,n", [(16384, 16129, 4096), (8192, 8065, 8192), (4096, 3841, 16384)])
def test_a_workspace_for_a_full_batch_serves_the_last_one(hs, full, last, n):
    """Slices of the full batch are moved off a 2 MB spacing and fewer than
    the shorter batch's."""
    ws = torch.empty(hs.hdiag_workspace_bytes(full, n), dtype=torch.uint8, device=DEV)
    X = torch.randn((full, n), generator=torch.Generator(device=DEV).manual_seed(n), device=DEV).bfloat16()
    for T in (full, last):
        h = hs.hdiag(X[:T], workspace=ws)
        ref = X[:T].double().square_().sum(0)
        torch.cuda.synchronize()
        print(f"[{T}x{n}] workspace {ws.numel()}, asked for {hs.hdiag_workspace_bytes(T, n)}", flush=True)
        assert ((h.double() - ref).abs() <= 2e-6 * ref).all()
        assert torch.equal(h, hs.hdiag(X[:T]))


def test_hdiag_of_very_many_columns(hs):
    """Blocks of 64 columns and 1024 threads would make a grid of 2^32
    threads, which no launch takes."""
    T, n = 257, 1 << 28
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GB of free GPU memory")
    X = torch.zeros((T, n), dtype=torch.bfloat16, device=DEV)
    cols = torch.tensor([0, 12345, n // 2 + 7, n - 1], device=DEV)
    X[:, cols] = 0.5
    print(f"[{T}x{n}]", flush=True)
    h = hs.hdiag(X)
    torch.cuda.synchronize()
    assert torch.equal(h[cols], torch.full((4,), T * 0.25, device=DEV))
    assert int(torch.count_nonzero(h)) == 4
    del X, h
    torch.cuda.empty_cache()
