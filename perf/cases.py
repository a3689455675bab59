"""The work that users of this framework have it do, as timed cases.

A calibration program reduces activations X [tokens, in] to h = diag(X^T X),
searches the NVFP4 scales of each linear layer's W [out, in] under that h (or
takes the plain max-abs scales), and scores the stored result: per-group
statistics, and the layer-output error of the codes on X.  Each case is one
such call, or the short sequence of calls that a program makes together, at
the shapes of 8B- and 70B-class decoder layers, of single sequences, and of
small layers where latency counts.
"""
import math

import torch

import paper_2608_28113_amd as hs

GROUP = 16
E2M1 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)
MAX_BYTES = 2 * 262144 * 14336           # X of the largest listed hdiag
MAX_FLOPS = 2 * 262144 * 4096 * 14336    # X dW^T of the largest listed output error
# (name, out, in) of a decoder block's seven linear layers, in units of the
# hidden size, the feed-forward size and the key/value width.
BLOCK = (("q", "hidden", "hidden"), ("k", "kv", "hidden"), ("v", "kv", "hidden"), ("o", "hidden", "hidden"),
         ("gate", "ffn", "hidden"), ("up", "ffn", "hidden"), ("down", "hidden", "ffn"))


def listed():
    return [
        # One small layer from activations to codes: every launch and every
        # host step shows (the sizes of the repository's smallest workload).
        dict(name="tiny_layer", kind="layer", tokens=128, n=512, m=256, down=4, up=4),
        # Streamed calibration: h of an attention input over sequences of a
        # little under 2048 tokens, one call for each as it arrives.
        dict(name="calib_stream", kind="stream", tokens=2040, n=4096, batches=8),
        # h of a stored down_proj input, 128 sequences of 2048 tokens.
        dict(name="hdiag_down", kind="hdiag", tokens=262144, n=14336),
        # The headline search: an 8B-class down_proj at +-4.
        dict(name="search_down", kind="search", m=4096, n=14336, down=4, up=4, init="maxabs", heavy=True),
        # The paper's window from 4over6 anchors on an attention projection.
        dict(name="search_attn_4over6", kind="search", m=4096, n=4096, down=9, up=6, init="4over6", heavy=False),
        # All seven layers of a decoder block at +-8 in one call.
        dict(name="search_block_layers", kind="layers", hidden=4096, kv=1024, ffn=14336, down=8, up=8, init="maxabs"),
        # The max-abs baseline of a 70B-class down_proj, and the final
        # re-quantization of moved weights at the chosen codes.
        dict(name="rtn_requantize_70b", kind="rtn", m=8192, n=28672),
        # GPTQ-style use: blocks of 128 columns of one layer, one after another.
        dict(name="gptq_column_blocks", kind="gptq", m=4096, n=4096, cols=128, down=9, up=6),
        # Selected-shift statistics of an up projection.
        dict(name="shift_statistics", kind="stats", m=14336, n=4096, down=4, up=4),
        # Output error on one sequence (a quick score while tuning a window).
        dict(name="output_error_sequence", kind="error", tokens=2048, m=4096, n=4096),
        # Output error of a gate projection on the whole calibration set.
        dict(name="output_error_gate", kind="error", tokens=262144, m=14336, n=4096),
        # Output error of a down_proj on a quarter of it.
        dict(name="output_error_down", kind="error", tokens=65536, m=4096, n=14336),
    ]


def _log(rng, lo, hi, mult=1):
    """A multiple of `mult` in lo..hi, spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / mult)) * mult))


def _window(rng):
    down, up = rng.choice([(1, 1), (2, 2), (4, 4), (8, 8), (9, 6), (6, 0), (0, 6), (12, 11), (16, 16)])
    return dict(down=down, up=up)


def draw(rng):
    kind = rng.choice(["layer", "stream", "hdiag", "search", "layers", "rtn", "gptq", "stats", "error", "error"])
    n, m = _log(rng, 64, 28672, GROUP), _log(rng, 17, 14336)
    if kind == "layer":
        return dict(kind=kind, tokens=_log(rng, 64, 2048), n=_log(rng, 64, 2048, GROUP), m=_log(rng, 17, 2048),
                    **_window(rng))
    if kind == "stream":
        return dict(kind=kind, tokens=_log(rng, 64, 8192), n=n, batches=rng.randint(1, 16))
    if kind == "hdiag":
        return dict(kind=kind, tokens=_log(rng, 256, min(262144, MAX_BYTES // (2 * n))), n=n)
    if kind == "search":
        return dict(kind=kind, m=m, n=min(n, 14336), init=rng.choice(["maxabs", "4over6", "given"]),
                    heavy=rng.random() < 0.5, **_window(rng))
    if kind == "layers":
        hidden = _log(rng, 256, 4096, 64)
        return dict(kind=kind, hidden=hidden, kv=max(64, hidden // rng.choice([1, 4, 8]) // GROUP * GROUP),
                    ffn=_log(rng, 256, 14336, GROUP), init=rng.choice(["maxabs", "4over6"]), down=4, up=4)
    if kind == "rtn":
        return dict(kind=kind, m=min(m, 8192), n=n)
    if kind == "gptq":
        cols = rng.choice([64, 128, 256])
        return dict(kind=kind, m=m, n=cols * rng.randint(2, 24), cols=cols, **_window(rng))
    if kind == "stats":
        return dict(kind=kind, m=m, n=min(n, 4096), **_window(rng))
    n = min(n, 14336)
    return dict(kind=kind, tokens=_log(rng, 64, max(64, min(262144, MAX_FLOPS // (2 * m * n)))), m=m, n=n)


# ---------------------------------------------------------------------------
# Inputs: bf16 weights and activations as calibration meets them
# ---------------------------------------------------------------------------


def _device():
    return torch.device("cuda:0")


def _gen(seed, salt):
    return torch.Generator(device=_device()).manual_seed(int(seed) * 1000003 + salt)


def _sigma(n, g):
    """Channel standard deviations: log-normal, and a few outlier channels."""
    s = torch.exp(0.6 * torch.randn(n, generator=g, device=_device()))
    s[torch.randperm(n, generator=g, device=_device())[:max(1, n // 896)]] *= 50.0
    return s


def _activations(T, n, seed, salt=0):
    """X [T, n]: per-channel spread, and a part that the channels share (eight
    common directions), so that X^T X is not diagonal."""
    g = _gen(seed, 10 + salt)
    sigma = _sigma(n, g)
    mix = 0.25 * torch.randn((8, n), generator=g, device=_device())
    X = torch.empty((T, n), dtype=torch.bfloat16, device=_device())
    rows = max(1, (1 << 27) // n)
    for t in range(0, T, rows):
        k = min(rows, T - t)
        z = torch.randn((k, n), generator=g, device=_device())
        z.addmm_(torch.randn((k, 8), generator=g, device=_device()), mix)
        X[t:t + k].copy_(z.mul_(sigma))
    return X


def _weight(m, n, seed, salt=0, heavy=False):
    """W [m, n]: Student-t(4) entries (down projections), or normal entries
    with 0.1% outliers."""
    g = _gen(seed, 100 + salt)
    W = torch.empty((m, n), dtype=torch.bfloat16, device=_device())
    rows = max(1, (1 << 26) // n)
    for r in range(0, m, rows):
        shape = (min(rows, m - r), n)
        w = torch.randn(shape, generator=g, device=_device()).mul_(0.02)
        if heavy:
            e = torch.rand(shape, generator=g, device=_device()).mul_(torch.rand(shape, generator=g, device=_device()))
            w.div_(e.clamp_(min=1e-9).log_().neg_().mul_(0.5).sqrt_())  # -2 log(u v) is chi-squared with 4 degrees
        else:
            w[torch.rand(shape, generator=g, device=_device()) < 1e-3] *= 8.0
        W[r:r + shape[0]].copy_(w)
    return W


def _h(n, seed, salt=0):
    """The diagonal that calibration on 262144 tokens gives (fp32 [n])."""
    g = _gen(seed, 1000 + salt)
    s = _sigma(n, g)
    return (s * s * 262144.0 * (1.0 + 0.003 * torch.randn(n, generator=g, device=_device()))).contiguous()


def _scale(W):
    """s_g = fp32(max|W| / 2688), which maps the largest weight to 6 * 448."""
    return float((W.abs().max().float() / 2688.0).item())


def _rtn_codes(W, s_g):
    """The max-abs E4M3 code byte of every group, by torch's own cast."""
    m, n = W.shape
    amax = W.view(m, n // GROUP, GROUP).abs().amax(-1).float()
    t = (amax / 6.0) / torch.tensor(s_g, dtype=torch.float32, device=W.device)
    return t.clamp_(max=448.0).to(torch.float8_e4m3fn).view(torch.uint8).clamp_(1, 126)


def _effective(codes, s_g):
    """fp32(s_g * l_c) of code bytes."""
    return codes.view(torch.float8_e4m3fn).float() * torch.tensor(s_g, dtype=torch.float32, device=codes.device)


def _quantized(W, S):
    """E2M1 codes (uint8 0..15) of W at the groups' effective scales."""
    m, n = W.shape
    x = W.view(m, n // GROUP, GROUP).float() * (1.0 / S)[..., None]
    q = torch.zeros_like(x, dtype=torch.uint8)
    a = x.abs()
    for mid, below in ((0.25, False), (0.75, True), (1.25, False), (1.75, True), (2.5, False), (3.5, True), (5.0, False)):
        q += (a >= mid) if below else (a > mid)  # ties to the even code
    return (q | (torch.signbit(x).to(torch.uint8) << 3)).view(m, n)


def _packed(q):
    return (q[:, 0::2] | (q[:, 1::2] << 4)).contiguous()


def _stored(W, s_g):
    """(codes, packed) of the max-abs NVFP4 tensor of W."""
    codes = _rtn_codes(W, s_g)
    return codes, torch.cat([_packed(_quantized(W[r:r + 1024], _effective(codes[r:r + 1024], s_g)))
                             for r in range(0, W.shape[0], 1024)])


def _layers_of(case):
    return [(case[o], case[i], name == "down") for name, o, i in BLOCK]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "layer":
        W = _weight(case["m"], case["n"], seed)
        return dict(case=case, X=_activations(case["tokens"], case["n"], seed), W=W, s_g=_scale(W))
    if kind == "stream":
        X = [_activations(case["tokens"], case["n"], seed, salt=k) for k in range(case["batches"])]
        return dict(case=case, X=X, h64=torch.zeros(case["n"], dtype=torch.float64, device=_device()))
    if kind == "hdiag":
        return dict(case=case, X=_activations(case["tokens"], case["n"], seed))
    if kind == "layers":
        layers = []
        for k, (m, n, heavy) in enumerate(_layers_of(case)):
            W = _weight(m, n, seed, salt=k, heavy=heavy)
            layers.append((W, _h(n, seed, salt=m if n != case["hidden"] else 0), _scale(W)))
        return dict(case=case, layers=layers)
    W = _weight(case["m"], case["n"], seed, heavy=case.get("heavy", kind in ("rtn", "error") and case["n"] > case["m"]))
    state = dict(case=case, W=W, s_g=_scale(W))
    if kind == "error":
        state["codes"], state["packed"] = _stored(W, state["s_g"])
        state["X"] = _activations(case["tokens"], case["n"], seed)
        return state
    state["h"] = _h(case["n"], seed)
    if kind == "search":
        # A baseline's codes, one step off the max-abs ones here and there.
        init = case["init"]
        if init == "given":
            step = torch.randint(-2, 3, (case["m"], case["n"] // GROUP), generator=_gen(seed, 7), device=_device())
            init = (_rtn_codes(W, state["s_g"]).long() + step).clamp(1, 126).to(torch.uint8)
        state["init"] = init
    elif kind == "rtn":
        noise = torch.randn(W.shape, generator=_gen(seed, 8), device=_device(), dtype=torch.bfloat16)
        state["W2"] = W + 0.002 * noise
    elif kind == "gptq":
        m, n = W.shape
        state["codes"] = torch.empty((m, n // GROUP), dtype=torch.uint8, device=_device())
        state["packed"] = torch.empty((m, n // 2), dtype=torch.uint8, device=_device())
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "layer":
        h = hs.hdiag(state["X"])
        return (h,) + tuple(hs.search(state["W"], h, state["s_g"], down=case["down"], up=case["up"]))
    if kind == "stream":
        h64 = state["h64"].zero_()
        for X in state["X"]:
            hs.hdiag_accumulate(X, h64)
        return hs.hdiag_finalize(h64), h64
    if kind == "hdiag":
        return hs.hdiag(state["X"])
    if kind == "search":
        return hs.search(state["W"], state["h"], state["s_g"], down=case["down"], up=case["up"], init=state["init"])
    if kind == "layers":
        return hs.search_layers(state["layers"], down=case["down"], up=case["up"], init=case["init"])
    if kind == "rtn":
        codes, packed = hs.search(state["W"], state["h"], state["s_g"], window=0)
        return codes, packed, hs.quantize(state["W2"], state["s_g"], codes)
    if kind == "gptq":
        B, W, h, codes, packed = case["cols"], state["W"], state["h"], state["codes"], state["packed"]
        for i in range(0, case["n"], B):
            hs.search_block(W[:, i:i + B], h[i:i + B], state["s_g"], case["down"], case["up"],
                            codes[:, i // GROUP:(i + B) // GROUP], packed[:, i // 2:(i + B) // 2])
        return codes, packed
    if kind == "stats":
        out = hs.search_stats(state["W"], state["h"], state["s_g"], case["down"], case["up"])
        out["summary"] = hs.shift_summary(out["shift"], out["err_best"], out["err_init"], case["down"], case["up"])
        return out
    return hs.output_error(state["X"], state["W"], state["s_g"], state["codes"], state["packed"])


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how far correct results may differ
# ---------------------------------------------------------------------------


def _search_work(m, n, K, given=False):
    """W and h in, codes and nibbles out.  Per weight and candidate: product,
    rounding, residual (2), square (1), weight (1) and sum (1); one candidate
    alone needs no score."""
    return dict(bytes=m * n * 2 + n * 4 + m * n // 2 + m * n // GROUP * (2 if given else 1),
                flops=m * n * (3 + (7 * K if K > 1 else 2)))


def work(case):
    kind = case["kind"]
    K = case.get("down", 0) + case.get("up", 0) + 1
    m, n, T = case.get("m", 0), case.get("n", 0), case.get("tokens", 0)
    if kind == "layer":
        w = _search_work(m, n, K)
        return dict(bytes=w["bytes"] + 2 * T * n, flops=w["flops"] + 2 * T * n)
    if kind == "stream":
        T *= case["batches"]
        return dict(bytes=2 * T * n + 12 * n, flops=2 * T * n)
    if kind == "hdiag":
        return dict(bytes=2 * T * n + 4 * n, flops=2 * T * n)
    if kind == "layers":
        each = [_search_work(o, i, K) for o, i, _ in _layers_of(case)]
        return dict(bytes=sum(w["bytes"] for w in each), flops=sum(w["flops"] for w in each))
    if kind == "rtn":
        w = _search_work(m, n, 1)
        return dict(bytes=2 * w["bytes"] - 8 * n, flops=2 * w["flops"])
    if kind == "stats":
        w = _search_work(m, n, K)
        return dict(bytes=w["bytes"] + 9 * (m * n // GROUP) + 32 * K, flops=w["flops"])
    if kind in ("search", "gptq"):
        return _search_work(m, n, K, given=case.get("init") == "given")
    # X dW^T once, or the symmetric X^T X and dW against it, whichever is less.
    return dict(bytes=2 * T * n + m * n * 2 + m * n // 2 + m * n // GROUP + 8 * m,
                flops=min(2 * T * n * m, T * n * (n + 1) + m * n * (n + 1)))


def tolerance(case):
    kind = case["kind"]
    if kind == "layer":
        # h as below; a last-bit change of h may move a group whose two best
        # candidates are within fp32 rounding of each other.
        return dict(rel=1e-6, max=4e-6, differ=1e-3)
    if kind in ("hdiag", "stream"):
        return dict(rel=1e-6, max=4e-6)  # fp32 chains folded into fp64
    if kind == "stats":
        return dict(rel=2e-6, max=8e-6, differ=0.0)  # fp32 scores of 16 terms; codes and counts exact
    if kind == "error":
        return dict(rel=2e-5, max=1e-4)  # dW in 17 bits: 3e-6 to 5e-6 from 64 bits, rows of few outlier channels more
    return "exact"  # code bytes under the documented arithmetic


# ---------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------


def _hdiag64(X):
    n = X.shape[1]
    rows = max(1, (1 << 26) // n)
    return sum(X[t:t + rows].double().square_().sum(0) for t in range(0, X.shape[0], rows))


def _stats64(case, state):
    """Scores of every candidate in 64 bits, the first minimum of each group
    and the per-shift sums."""
    W, h, s_g, down, up = state["W"], state["h"].double(), state["s_g"], case["down"], case["up"]
    m, n = W.shape
    grid = torch.tensor(E2M1, dtype=torch.float64, device=W.device)
    best, init, shift = [], [], []
    rows = max(1, (1 << 24) // n)
    for r in range(0, m, rows):
        w = W[r:r + rows]
        c0 = _rtn_codes(w, s_g).int()
        w64 = w.view(-1, n // GROUP, GROUP).double()
        scores = []
        for d in range(-down, up + 1):
            S = _effective((c0 + d).clamp(1, 126).to(torch.uint8), s_g)
            q = _quantized(w, S).view(-1, n // GROUP, GROUP)
            v = grid[(q & 7).long()] * torch.where(q > 7, -1.0, 1.0)
            scores.append(((w64 - v * S.double()[..., None]).square_() * h.view(n // GROUP, GROUP)).sum(-1))
        e = torch.stack(scores)
        b, k = e.min(0)
        best.append(b)
        init.append(e[down])
        shift.append(k)
    eb, ei, k = torch.cat(best), torch.cat(init), torch.cat(shift).flatten()
    rel = torch.where(ei > 0, (ei - eb) / ei, 0.0)

    def per_shift(v):
        return torch.zeros(down + up + 1, dtype=torch.float64, device=W.device).index_add_(0, k, v.flatten())
    return dict(scale_codes=None, packed_e2m1=None, shift=None, err_best=eb, err_init=ei,
                summary=dict(count=None, sum_init=per_shift(ei), sum_best=per_shift(eb), sum_rel=per_shift(rel)))


def _error64(state):
    W, X, s_g = state["W"], state["X"], state["s_g"]
    m, n = W.shape
    S = _effective(state["codes"], s_g).double()
    lo, hi = state["packed"] & 15, state["packed"] >> 4
    q = torch.stack([lo, hi], -1).view(m, n)
    grid = torch.tensor([s * v for s in (1.0, -1.0) for v in E2M1], dtype=torch.float64, device=W.device)
    dW = W.double() - (grid[q.long()].view(m, n // GROUP, GROUP) * S[..., None]).view(m, n)
    del q, lo, hi
    dW = dW.t().contiguous()
    out = torch.zeros(m, dtype=torch.float64, device=W.device)
    for t in range(0, X.shape[0], 8192):
        out += (X[t:t + 8192].double() @ dW).square_().sum(0)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("layer", "stream", "hdiag", "stats", "error"):
        return None
    state = prepare(case, seed)
    if kind == "layer":
        return _hdiag64(state["X"]), None, None
    if kind == "stream":
        h = sum(_hdiag64(X) for X in state["X"])
        return h, h
    if kind == "hdiag":
        return _hdiag64(state["X"])
    return _stats64(case, state) if kind == "stats" else _error64(state)
