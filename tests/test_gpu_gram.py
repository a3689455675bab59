"""The Gram route of hscale_output_error (many output rows on one X) against
the direct route on the same inputs and against float64.

The route is chosen from the sizes and from the workspace: a workspace of the
direct route's size keeps the direct product, which gives both on one input.
"""
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


def _direct_bytes(T, n, m):
    """Workspace of the direct route: two padded bf16 planes of dW and fp64
    partials of at most 1024 token tiles of 384."""
    ldd, rows = -(-n // 32) * 32, -(-m // 256) * 256
    plane = -(-rows * ldd * 2 // 256) * 256
    return 2 * plane + min(-(-T // 384), 1024) * m * 8


def _case(T, n, m, seed):
    """Activations with shared directions and outlier channels, weights with
    any stored codes near their max-abs ones, and dW in float64."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    sigma = torch.exp(0.6 * torch.randn(n, generator=g, device=DEV))
    sigma[:: max(1, n // 3)] *= 50.0
    mix = 0.3 * torch.randn((4, n), generator=g, device=DEV)
    X = torch.empty((T, n), dtype=torch.bfloat16, device=DEV)
    for t in range(0, T, 16384):
        k = min(16384, T - t)
        z = torch.randn((k, n), generator=g, device=DEV)
        X[t:t + k] = (z + torch.randn((k, 4), generator=g, device=DEV) @ mix) * sigma
    W = (0.02 * torch.randn((m, n), generator=g, device=DEV)).to(torch.bfloat16)
    return X, W


def _stored(hs, W):
    h = torch.ones(W.shape[1], device=DEV)
    s_g = float((W.abs().max().float() / 2688.0).item())
    codes, packed = hs.search(W, h, s_g, window=2)
    return s_g, codes, packed


def _reference(X, W, s_g, codes, packed):
    """Eq. 3 per row in float64 torch."""
    m, n = W.shape
    grid = torch.tensor([s * v for s in (1.0, -1.0) for v in (0, 0.5, 1, 1.5, 2, 3, 4, 6)], dtype=torch.float64,
                        device=DEV)
    S = (codes.view(torch.float8_e4m3fn).float() * torch.tensor(s_g, device=DEV)).double()
    q = torch.stack([packed & 15, packed >> 4], -1).view(m, n)
    dW = W.double() - (grid[q.long()].view(m, n // 16, 16) * S[..., None]).view(m, n)
    dW = dW.t().contiguous()
    out = torch.zeros(m, dtype=torch.float64, device=DEV)
    for t in range(0, X.shape[0], 16384):
        out += (X[t:t + 16384].double() @ dW).square_().sum(0)
    return out


def _both(hs, X, W, s_g, codes, packed):
    T, n = X.shape
    m = W.shape[0]
    need, direct = hs.output_error_workspace_bytes(T, n, m), _direct_bytes(T, n, m)
    assert need > direct, "the sizes no longer take the Gram route"
    print(f"[gram {T}x{n}x{m}] workspace {need} direct {direct}", flush=True)
    gram = hs.output_error(X, W, s_g, codes, packed)
    ws = torch.empty(direct, dtype=torch.uint8, device=DEV)
    plain = hs.output_error(X, W, s_g, codes, packed, workspace=ws)
    torch.cuda.synchronize()
    return gram, plain


def _rel(a, ref):
    return ((a - ref).abs() / ref).max().item()


# The direct route's bar (tests/test_gpu_diag.py): dW in two bf16 parts, each
# element to within 2^-16, rows of few dominant channels included.
REL_TOL = 1e-4
# The Gram route's, for rows whose terms do not cancel (L about D or more): D in
# fp64 but for the chains of G, at most 128 steps of 16 tokens that round to
# 2^-24 of their sum each; in random order about sqrt(128) / 2 of that, 3.4e-7,
# and what many entries add to a row averages out.  The planes hold 22 bits,
# 2.4e-7.  Four times the sum of the two; measured 2e-7 to 6e-7, and 1.4e-6 over
# 24577 rows of 16384 columns, whose product with G adds up in 3072 fp32 steps.
GRAM_TOL = 2.4e-6


def _chunks_held(hs, T, n, m):
    """Chunks whose partials the workspace holds (256 KB to a tile and chunk),
    and two more where fp64 sums of the tiles are carried between passes.
    Chunks have at most 2048 tokens, the chain length that repeated tokens
    need (tested below): so T beyond as many takes several passes."""
    nt = -(-n // 256)
    ldg, tri = nt * 256, nt * (nt + 1) // 2
    rest = 2 * ldg * ldg * 2 + 12 * ldg + 16 * m + 8 * nt * m + 256 + 4 * m
    least = hs._lib.hscale_output_error_least_workspace_bytes(T, n, m)
    return (hs.output_error_workspace_bytes(T, n, m) - rest - least) // (tri << 18)


# One column tile and a ragged one; a last tile of 16 columns; ragged tokens
# and rows; more partial tiles than one pass holds (136 and 528 tiles to a
# chunk), the last pass shorter and its last chunk ragged; and more passes than
# add up in fp32 (2080 tiles, 17 passes of 2 chunks).
@pytest.mark.parametrize("T,n,m", [(400001, 240, 4097), (120000, 528, 3000), (70007, 1040, 4100),
                                   (65536, 2048, 2048), (8192 * 34 + 77, 4096, 4096), (2048 * 34 + 77, 8192, 8192),
                                   (2048 * 33 + 77, 16384, 24577)])
def test_gram_route_matches_float64_and_the_direct_route(hs, T, n, m):
    X, W = _case(T, n, m, seed=T + n + m)
    held = _chunks_held(hs, T, n, m)
    assert (held * 2048 < T) == (n >= 4096) and (n < 16384 or held == 4)
    s_g, codes, packed = _stored(hs, W)
    codes[m // 2].zero_()  # a zero scale: dW = W
    gram, plain = _both(hs, X, W, s_g, codes, packed)
    ref = _reference(X, W, s_g, codes, packed)
    norm = [((v - ref).norm() / ref.norm()).item() for v in (gram, plain)]
    print(f"  max rel gram {_rel(gram, ref):.2e} direct {_rel(plain, ref):.2e}; norm {norm[0]:.2e} {norm[1]:.2e}",
          flush=True)
    assert torch.isfinite(gram).all() and _rel(gram, ref) <= GRAM_TOL and _rel(plain, ref) <= REL_TOL
    assert norm[0] <= norm[1] + 1e-6  # no precision lost against the direct product
    again = hs.output_error(X, W, s_g, codes, packed, row_err=gram.clone())
    torch.cuda.synchronize()
    assert torch.equal(again, gram + gram)  # accumulates, and is repeatable bit for bit


def _opposed(T, n, m, noise):
    """Neighbouring channels nearly opposite; equal weights in even rows (y
    cancels to about noise^2 / 2 of its diagonal part) and opposite ones in
    odd rows (y adds up)."""
    X, W = _case(T, n, m, seed=5)
    g = torch.Generator(device=DEV).manual_seed(1)
    X[:, 1::2] = -X[:, 0::2] * (1.0 + noise * torch.randn((T, n // 2), device=DEV, generator=g))
    W[0::2, 1::2] = W[0::2, 0::2]
    W[1::2, 1::2] = -W[1::2, 0::2]
    return X, W


@pytest.mark.parametrize("noise", [0.02, 0.1, 0.2, 0.4])
def test_cancelling_rows_lose_no_precision(hs, noise):
    """Rows on both sides of the line below which the direct product takes
    over (up to 0.2 the even rows lie below it)."""
    X, W = _opposed(65536, 1024, 4100, noise)
    s_g, codes, packed = _stored(hs, W)
    gram, plain = _both(hs, X, W, s_g, codes, packed)
    ref = _reference(X, W, s_g, codes, packed)
    for rows in (slice(0, None, 2), slice(1, None, 2)):
        print(f"  noise {noise} max rel gram {_rel(gram[rows], ref[rows]):.2e} direct "
              f"{_rel(plain[rows], ref[rows]):.2e}", flush=True)
        assert _rel(gram[rows], ref[rows]) <= max(REL_TOL, 1.5 * _rel(plain[rows], ref[rows]))
    if noise <= 0.2:
        even = slice(0, None, 2)
        assert ((gram[even] - plain[even]).abs() <= 1e-12 * plain[even]).all()  # the direct sums, in another order


@pytest.mark.parametrize("kind", ["padding", "two tokens", "constant channels"])
def test_repeated_tokens_lose_no_precision(hs, kind):
    """Equal tokens add with equal rounding, so a long fp32 chain over them
    drifts, where the direct product sums over tokens in float64.  Of the rows
    that the Gram route answers itself, the error as a whole and on average is
    no larger than the direct product's.  So is the largest but for chance:
    one row that cancels to just above the line decides it on either side."""
    X, W = _case(147456, 4096, 4096, seed=3)
    T = X.shape[0]
    if kind == "padding":
        X[T // 2:] = X[5].clone()
    elif kind == "two tokens":
        X[:] = X[:2].repeat(T // 2, 1)
    else:
        X[:, ::2] = X[3, ::2].clone()
    s_g, codes, packed = _stored(hs, W)
    gram, plain = _both(hs, X, W, s_g, codes, packed)
    ref = _reference(X, W, s_g, codes, packed)
    own = (gram - plain).abs() > 1e-12 * plain
    g, d = (((v - ref).abs() / ref)[own] for v in (gram, plain))
    print(f"  {kind}: own rows {own.float().mean().item():.3f} max {g.max().item():.2e} direct {d.max().item():.2e}; "
          f"mean {g.mean().item():.2e} {d.mean().item():.2e}; norm {((gram - ref).norm() / ref.norm()).item():.2e} "
          f"{((plain - ref).norm() / ref.norm()).item():.2e}", flush=True)
    assert (gram - ref).norm() <= (plain - ref).norm()
    assert g.mean() <= d.mean() and g.max() <= 1.5 * d.max()


# Channels that are zero, or whose squares underflow fp32, beside live ones: the
# scales of the 16-bit planes must not depend on them.  Rows of this input do
# not cancel, and without such channels the largest relative error is 2e-7 at
# every scale (the direct product's 1.3e-5).
@pytest.mark.parametrize("log2_scale", [-10, -24, -30, -40])
@pytest.mark.parametrize("tiny", [0.0, 2.0 ** -40])
def test_channels_without_activations(hs, log2_scale, tiny):
    X, W = _case(65536, 1024, 4096, seed=3)
    X[:, 7::100] *= tiny
    X = X.mul_(2.0 ** log2_scale)
    s_g, codes, packed = _stored(hs, W)
    gram, plain = _both(hs, X, W, s_g, codes, packed)
    ref = _reference(X, W, s_g, codes, packed)
    print(f"  2^{log2_scale} max rel gram {_rel(gram, ref):.2e} direct {_rel(plain, ref):.2e}", flush=True)
    assert _rel(gram, ref) <= GRAM_TOL


@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** 70])
def test_squares_outside_fp32_go_direct(hs, scale):
    X, W = _case(65536, 1024, 4096, seed=6)
    X = X.mul_(scale)
    s_g, codes, packed = _stored(hs, W)
    gram, plain = _both(hs, X, W, s_g, codes, packed)
    assert torch.isfinite(gram).all()
    assert ((gram - plain).abs() <= 1e-12 * plain).all()


# The direct route's tiles, tokens x rows: 64 x 128 (the first five cases, of
# 1, 1, 2, 3 and 33 stages), 128 x 128 (two), 128 x 256 (three), 256 x 256
# (three) and 384 x 256 (the last); edges, ragged rows and columns, more than a
# round.
@pytest.mark.parametrize("T,n,m", [(1, 16, 1), (127, 32, 255), (129, 48, 257), (65, 80, 129), (385, 1040, 513),
                                   (2945, 48, 1025), (3000, 96, 700), (1801, 16, 3001), (1300, 80, 3900),
                                   (6500, 208, 700), (2050, 16, 3900), (2049, 528, 4100), (4096, 256, 4096),
                                   (5000, 80, 4096)])
def test_direct_tiles_and_smaller_workspaces(hs, T, n, m):
    X, W = _case(T, n, m, seed=T + m)
    s_g, codes, packed = _stored(hs, W)
    ref = _reference(X, W, s_g, codes, packed)
    full = hs.output_error(X, W, s_g, codes, packed)
    least = torch.empty(_direct_bytes(T, n, m), dtype=torch.uint8, device=DEV)
    passes = hs.output_error(X, W, s_g, codes, packed, workspace=least)  # 384 x 256 tiles
    torch.cuda.synchronize()
    print(f"[direct {T}x{n}x{m}] max rel {_rel(full, ref):.2e}", flush=True)
    assert _rel(full, ref) <= REL_TOL
    assert ((full - passes).abs() <= 1e-12 * full).all()


@pytest.mark.parametrize("T,n,m", [(385, 1040, 513), (3000, 96, 700), (2049, 528, 4100), (5000, 80, 4096)])
def test_a_smaller_workspace_takes_one_pass(hs, T, n, m):
    """The least workspace holds the partials of all tokens in 384-token
    tiles: one pass leaves them there, and they add up to the result.  Small
    tiles in it would take several passes over the same partials."""
    X, W = _case(T, n, m, seed=T + m)
    s_g, codes, packed = _stored(hs, W)
    tiles = -(-T // 384)
    ws = torch.zeros(_direct_bytes(T, n, m), dtype=torch.uint8, device=DEV)
    L = hs.output_error(X, W, s_g, codes, packed, workspace=ws)
    parts = ws[ws.numel() - tiles * m * 8:].view(torch.float64).view(tiles, m)
    torch.cuda.synchronize()
    print(f"[least {T}x{n}x{m}]", flush=True)
    assert ((parts.sum(0) - L).abs() <= 1e-13 * L).all()


def test_short_of_memory_takes_the_least_workspace(hs):
    """Where the faster route's workspace does not fit in the memory left, the
    call still runs in the direct product's, with its result."""
    T, n, m = 120000, 1040, 4100
    X, W = _case(T, n, m, seed=2)
    s_g, codes, packed = _stored(hs, W)
    need, least = hs.output_error_workspace_bytes(T, n, m), _direct_bytes(T, n, m)
    plain = hs.output_error(X, W, s_g, codes, packed, workspace=torch.empty(least, dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    room = least + (32 << 20)
    assert need > room
    total = torch.cuda.get_device_properties(DEV).total_memory
    print(f"[short of memory {T}x{n}x{m}] asked for {need}, room for {room}", flush=True)
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + room) / total)
    try:
        L = hs.output_error(X, W, s_g, codes, packed)
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(L, plain)


def test_very_many_rows(hs):
    """2^26 rows, more than one launch of the other route's row kernel holds."""
    T, n, m = 8000, 16, 1 << 26
    if torch.cuda.mem_get_info()[0] < 64 << 30:
        pytest.skip("needs 64 GB of free GPU memory")
    X, _ = _case(T, n, 16, seed=8)
    W = torch.zeros((m, n), dtype=torch.bfloat16, device=DEV)
    rows = torch.tensor([0, 4099, m // 2 + 1, m - 1], device=DEV)
    W[rows] = (0.02 * torch.randn((4, n), generator=torch.Generator(device=DEV).manual_seed(9), device=DEV)).bfloat16()
    codes = torch.zeros((m, 1), dtype=torch.uint8, device=DEV)  # scale 0: dW = W
    packed = torch.zeros((m, n // 2), dtype=torch.uint8, device=DEV)
    print(f"[direct {T}x{n}x{m}]", flush=True)
    L = hs.output_error(X, W, 1.0, codes, packed)
    torch.cuda.synchronize()
    ref = (X.double() @ W[rows].double().t().contiguous()).square_().sum(0)
    assert _rel(L[rows], ref) <= REL_TOL
    assert int(torch.count_nonzero(L)) == 4
    del W, codes, packed, L
    torch.cuda.empty_cache()
