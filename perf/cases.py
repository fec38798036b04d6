"""The work a user of this library has it do, as cases that can be timed and compared.

Two kinds of use:

* inference: one quantised linear layer applied to 1..64 activation vectors (`PackedLayer.gemv`,
  `PackedLayer.gemm_skinny`), and the weight set of one decoder block in sequence;
* quantising a layer: accumulate the Hessian over calibration batches, search scales and tyings, factor
  the inverse Hessian, run the GPTQ pass, fuse the integers into sign planes and pack them.

`listed()` holds the cases, `draw(rng)` gives more of the same ranges, `prepare` makes the inputs on the
GPU from a seed, `run` is one pass through the public entry points, `work` what a pass cannot do without,
`tolerance` how far two correct implementations may be apart, and `exact` the same result in 64 bits from
plain torch.
"""
import math

import torch

import paper_2407_02891_amd as bcq

# ------------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------------


def listed():
    return [
        # Decode of one token.  The key projection of a block with grouped queries: the smallest call of a
        # decoder, where start-up and the launch count.
        _linear("decode_kv_1024x8192", 1024, 8192, 3),
        # The widest layer of an OPT-30B-shaped block: the ordinary memory-bound decode call.
        _linear("decode_ffn_7168x28672", 7168, 28672, 3),
        # All weights of one Llama-2-70B-shaped block in sequence (q/k/v and gate/up stacked), two planes with
        # the parameters the paper's quantiser leaves: one scale record and one offset per row.
        {"name": "decode_block_rowwise", "kind": "block", "q": 2},
        # A handful of sequences decoded together, on the largest layer (OPT-66B-shaped), activations with
        # outlier channels.
        _linear("batch4_9216x36864", 9216, 36864, 3, batch=4, outliers=True),
        # Sixteen sequences.
        _linear("batch16_7168x28672", 7168, 28672, 3, batch=16),
        # Ragged sizes, two planes with offset, fine scaling groups, an odd number of sequences.
        _linear("batch27_g64_5000x7232", 5000, 7232, 2, group=64, offset=True, batch=27),
        # The largest batch of a call: a gate or up projection.
        _linear("batch64_28672x8192", 28672, 8192, 3, batch=64),
        # Quantising one 7168 x 7168 layer, step by step.  Calibration: four batches of 2048 samples.
        {"name": "hessian_7168", "kind": "hessian", "N": 7168, "T": 2048, "batches": 4},
        # Inverse-Hessian factor, once per layer input.
        {"name": "factor_7168", "kind": "factor", "N": 7168},
        # Search over scales and tyings (the defaults of the command-line quantiser).
        {"name": "search_7168_n3q2", "kind": "search", "M": 7168, "N": 7168, "n": 3, "q": 2, "grid": 8},
        # Column-by-column pass with error compensation.
        {"name": "gptq_7168_n4q3", "kind": "gptq", "M": 7168, "N": 7168, "n": 4, "q": 3},
        # Integers to sign planes, then the packed blob: the tall feed-forward layer.
        {"name": "fuse_pack_28672x7168", "kind": "fuse", "M": 28672, "N": 7168, "n": 3, "q": 2, "rows": True},
    ]


def _linear(name, M, N, q, group=128, offset=False, batch=1, outliers=False):
    c = {"kind": "linear", "M": M, "N": N, "q": q, "group": group, "offset": offset, "batch": batch, "outliers": outliers}
    if name:
        c["name"] = name
    return c


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_BITS = [(3, 2), (3, 2), (4, 3), (4, 2), (3, 3), (5, 3)]           # (bits of the linear step, planes)
_TYINGS = {(3, 2): 3, (4, 3): 6, (4, 2): 7, (3, 3): 1, (5, 3): 25}  # ways of tying the planes


def draw(rng):
    kind = rng.choice(["linear"] * 7 + ["hessian", "factor", "search", "gptq", "fuse"])
    if kind == "linear":
        group = rng.choice([128, 128, 128, 64, 32, 256, 0])  # 0: one group per row
        step = group or 32
        while True:
            M, N = _log_uniform(rng, 512, 36864), max(1, _log_uniform(rng, 512, 36864) // step) * step
            if M * N <= 9216 * 36864:
                break
        batch = rng.choice([1, 1, 1, 2, 3, 4, 6, 8, 13, 16, 21, 32, 45, 64])
        return _linear(None, M, N, rng.choice([1, 2, 2, 3, 3, 3, 4]), group=group or N, offset=rng.random() < 0.4,
                       batch=batch, outliers=rng.random() < 0.3)
    M, N = rng.randrange(256, 7169), 4 * rng.randrange(128, 1793)
    n, q = rng.choice(_BITS)
    if kind == "hessian":
        return {"kind": "hessian", "N": N, "T": rng.randrange(256, 2049), "batches": rng.randrange(1, 5)}
    if kind == "factor":
        return {"kind": "factor", "N": N}
    if kind == "search":
        most = max(1, int(24 * 7168 ** 3 / (_TYINGS[n, q] * M * N * N)))  # no dearer than the listed one
        return {"kind": "search", "M": M, "N": N, "n": n, "q": q, "grid": min(most, rng.randrange(1, 17))}
    if kind == "gptq":
        return {"kind": "gptq", "M": M, "N": N, "n": n, "q": q}
    if rng.random() < 0.5:
        return {"kind": "fuse", "M": 4 * M + 1, "N": 32 * max(1, N // 32), "n": n, "q": q, "rows": True}
    return {"kind": "fuse", "M": 4 * M + 1, "N": 128 * max(1, N // 128), "n": n, "q": q, "rows": False}


# ------------------------------------------------------------------------------------------------
# inputs, from the seed alone
# ------------------------------------------------------------------------------------------------


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _layer_inputs(M, N, q, group, offset, batch, outliers, seed):
    """Codes (bit i = sign of plane i), scales N(0, 0.02) in magnitude and descending over the planes, offsets
    N(0, 0.01), activations N(0, 1) with, where asked for, one channel in a hundred twenty times as large."""
    g = _gen(seed)
    G = N // group
    codes = torch.randint(0, 1 << q, (M, N), device="cuda", generator=g, dtype=torch.uint8)
    alpha = (torch.randn((M, G, q), device="cuda", generator=g) * 0.02).abs().sort(dim=2, descending=True).values.half()
    off = (torch.randn((M, G), device="cuda", generator=g) * 0.01).half() if offset else None
    X = torch.randn((batch, N), device="cuda", generator=g)
    if outliers:
        X[:, torch.randperm(N, device="cuda", generator=g)[: max(1, N // 100)]] *= 20.0
    return codes, alpha, off, X.half()


# One decoder block: layers that share their input are stacked (rows, columns).
_BLOCK = [("qkv", 8192 + 1024 + 1024, 8192), ("o", 8192, 8192), ("gate_up", 2 * 28672, 8192), ("down", 8192, 28672)]


def _block_layer_inputs(case, k, seed):
    _, M, N = _BLOCK[k]
    return _layer_inputs(M, N, case["q"], N, True, 1, False, 4 * seed + k)


def _packed(M, N, q, group, offset, batch, codes, alpha, off):
    layer = bcq.PackedLayer(M, N, q, group, offset, max_batch=batch)
    return layer.pack_from(codes, alpha, off)


def _weights(M, N, g):
    """A Gaussian bulk with one weight in a hundred four times as large."""
    W = torch.randn((M, N), device="cuda", generator=g) * 0.02
    return W * (1.0 + 3.0 * (torch.rand((M, N), device="cuda", generator=g) < 0.01))


def _calibration(T, N, g, mix=None, loud=None):
    """T samples of correlated channels, one in 32 of them six times as loud."""
    if mix is None:
        mix = torch.randn((8, N), device="cuda", generator=g)
        loud = torch.ones(N, device="cuda")
        loud[torch.randperm(N, device="cuda", generator=g)[: max(1, N // 32)]] = 6.0
    X = torch.randn((T, N), device="cuda", generator=g) + 0.5 * (torch.randn((T, 8), device="cuda", generator=g) @ mix)
    return (X * loud).contiguous(), mix, loud


def _hessian_of(N, g):
    """H = 2 X^T X of 2 N samples, in 32 bits, symmetric."""
    X, _, _ = _calibration(2 * N, N, g)
    H = 2.0 * (X.t().contiguous() @ X)
    return ((H + H.t()) * 0.5).contiguous()


def _upper_factor(H, damp=0.01):
    """U, upper triangular, with (H + damp mean(diag H) I)^-1 = U^T U, in 64 bits: with the rows and columns in
    reverse order H = L L^T, U is the inverse of L, reversed again."""
    N = H.shape[0]
    Hd = H.double()
    Hd.diagonal().add_(damp * Hd.diagonal().mean())
    L = torch.linalg.cholesky(Hd.flip(0, 1).contiguous())
    inv = torch.linalg.solve_triangular(L, torch.eye(N, dtype=torch.float64, device=H.device), upper=False)
    return inv.flip(0, 1).contiguous()


def _partitions(n, q):
    """All ways of tying n planes into q classes, as class labels per plane; the classes ordered by their smallest
    plane, the partitions lexicographically by their classes."""
    found = []

    def go(i, lab, used):
        if i == n:
            if used == q:
                found.append(lab)
            return
        for c in range(min(used + 1, q)):
            go(i + 1, lab + [c], max(used, c + 1))

    go(0, [], 0)
    return sorted(found, key=lambda lab: [[i + 1 for i in range(n) if lab[i] == c] for c in range(q)])


def _choices(lab, n, q):
    """Integers a tying can represent, ascending."""
    return sorted(sum(1 << i for i in range(n) if (m >> lab[i]) & 1) for m in range(1 << q))


def _labels(M, n, q, g):
    """A tying per row."""
    parts = torch.tensor(_partitions(n, q), device="cuda", dtype=torch.int8)
    return parts[torch.randint(0, len(parts), (M,), device="cuda", generator=g)].contiguous()


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    kind = case["kind"]
    if kind == "linear":
        M, N, q, group, off, batch = (case[k] for k in ("M", "N", "q", "group", "offset", "batch"))
        codes, alpha, z, X = _layer_inputs(M, N, q, group, off, batch, case["outliers"], seed)
        s.layer = _packed(M, N, q, group, off, batch, codes, alpha, z)
        s.X = X if batch > 1 else X[0]
        s.Y = torch.empty((batch, M) if batch > 1 else M, dtype=torch.float16, device="cuda")
        return s
    if kind == "block":
        s.layers = []
        for k, (_, M, N) in enumerate(_BLOCK):
            codes, alpha, z, X = _block_layer_inputs(case, k, seed)
            y = torch.empty(M, dtype=torch.float16, device="cuda")
            s.layers.append((_packed(M, N, case["q"], N, True, 1, codes, alpha, z), X[0], y))
        return s
    g = _gen(seed)
    N = case["N"]
    if kind == "hessian":
        X, mix, loud = _calibration(case["T"], N, g)
        s.batches = [X] + [_calibration(case["T"], N, g, mix, loud)[0] for _ in range(case["batches"] - 1)]
        s.H = torch.empty((N, N), device="cuda")
        return s
    if kind == "factor":
        s.H = _hessian_of(N, g)
        s.U = torch.empty_like(s.H)
        s.ws = torch.empty(bcq.quant_factor_workspace_bytes(N), dtype=torch.uint8, device="cuda")
        return s
    M, n, q = case["M"], case["n"], case["q"]
    if kind == "search":
        s.W, s.H = _weights(M, N, g), _hessian_of(N, g)
        s.S, s.qbias, s.err = (torch.empty(M, device="cuda") for _ in range(3))
        s.labels = torch.empty((M, n), dtype=torch.int8, device="cuda")
        s.ws = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
        return s
    if kind == "gptq":
        s.W = _weights(M, N, g)
        s.U = _upper_factor(_hessian_of(N, g)).float()
        lo, hi = s.W.min(1).values, s.W.max(1).values
        # a scale inside the interval that the search walks
        s.S = ((hi - lo) / ((1 << n) - 1) * (0.6 + 0.8 * torch.rand(M, device="cuda", generator=g))).contiguous()
        s.qbias = lo.contiguous()
        s.labels = _labels(M, n, q, g)
        s.w_int = torch.empty((M, N), dtype=torch.uint8, device="cuda")
        s.ws = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
        return s
    assert kind == "fuse", kind
    s.w_int, s.S, s.qbias, s.labels = _fuse_inputs(case, g)
    group = N if case["rows"] else 128
    s.codes = torch.empty((M, N), dtype=torch.uint8, device="cuda")
    s.alpha = torch.empty((M, N // group, q), dtype=torch.float16, device="cuda")
    s.offset = torch.empty((M, N // group), dtype=torch.float16, device="cuda")
    s.layer = bcq.PackedLayer(M, N, q, group, True)
    return s


def _fuse_inputs(case, g):
    M, N, n, q = (case[k] for k in ("M", "N", "n", "q"))
    shape = (M,) if case["rows"] else (M, N // 128)
    w_int = torch.randint(0, 1 << n, (M, N), device="cuda", generator=g, dtype=torch.uint8)
    S = 0.002 + 0.02 * torch.rand(shape, device="cuda", generator=g)
    qbias = 0.05 * torch.randn(shape, device="cuda", generator=g)
    labels = _labels(M, n, q, g) if case["rows"] else _labels(1, n, q, g)[0].tolist()
    return w_int, S, qbias, labels


# ------------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------------


def run(s):
    case = s.case
    kind = case["kind"]
    if kind == "linear":
        return s.layer.gemv(s.X, s.Y) if case["batch"] == 1 else s.layer.gemm_skinny(s.X, s.Y)
    if kind == "block":
        return [layer.gemv(x, y) for layer, x, y in s.layers]
    N = case["N"]
    if kind == "hessian":
        s.H.zero_()
        for X in s.batches:
            bcq.quant_hessian(N, X.shape[0], X, s.H)
        return s.H
    if kind == "factor":
        bcq.quant_factor(N, 0.01, s.H, s.U, s.ws)
        return s.U
    M, n, q = case["M"], case["n"], case["q"]
    if kind == "search":
        bcq.quant_search(M, N, n, q, case["grid"], s.W, s.H, s.S, s.qbias, s.labels, s.err, s.ws)
        # the scale is one of the grid's values: its bits are a choice, like the tying
        return {"S": s.S.view(torch.int32), "qbias": s.qbias, "labels": s.labels, "err": s.err}
    if kind == "gptq":
        bcq.quant_gptq(M, N, n, q, s.W, s.U, s.S, s.qbias, s.labels, s.w_int, s.ws)
        return s.w_int
    if case["rows"]:
        bcq.from_linear_rows(M, N, n, q, s.labels, s.w_int, s.S, s.qbias, s.codes, s.alpha, s.offset)
    else:
        bcq.from_linear(M, N, 128, n, q, s.labels, s.w_int, s.S, s.qbias, s.codes, s.alpha, s.offset)
    s.layer.pack_from(s.codes, s.alpha, s.offset)
    return {"codes": s.codes, "alpha": s.alpha, "offset": s.offset, "packed": s.layer.packed}


# ------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------------


def _linear_work(M, N, q, group, offset, batch):
    """Sign planes and scales once, activations in, outputs out; one product per weight and vector."""
    weights = q * M * N / 8 + 2 * (q + bool(offset)) * M * (N // group)
    return {"bytes": weights + 2 * batch * (M + N), "flops": 2 * M * N * batch}


def work(case):
    kind = case["kind"]
    if kind == "linear":
        return _linear_work(*(case[k] for k in ("M", "N", "q", "group", "offset", "batch")))
    if kind == "block":
        each = [_linear_work(M, N, case["q"], N, True, 1) for _, M, N in _BLOCK]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    N = case["N"]
    if kind == "hessian":  # symmetric: half the products
        T = case["T"] * case["batches"]
        return {"bytes": 4 * (T * N + N * N), "flops": T * N * N}
    if kind == "factor":   # a Cholesky factorisation and the inverse of its factor
        return {"bytes": 8 * N * N, "flops": 2 * N ** 3 / 3}
    M, n, q = case["M"], case["n"], case["q"]
    if kind == "search":   # one quadratic form with a symmetric matrix per row and candidate
        return {"bytes": 4 * (M * N + N * N) + 16 * M, "flops": case["grid"] * _TYINGS[n, q] * M * N * N}
    if kind == "gptq":     # every column's error reaches the later columns
        return {"bytes": 4 * (M * N + N * N / 2) + M * N, "flops": M * N * N}
    scales = 2 * (q + 1) * M * (1 if case["rows"] else N // 128)
    return {"bytes": 2 * M * N + q * M * N / 8 + 2 * scales, "flops": 0}


# ------------------------------------------------------------------------------------------------
# how far two correct implementations may be apart, and the result in 64 bits
# ------------------------------------------------------------------------------------------------


def tolerance(case):
    kind = case["kind"]
    if kind in ("linear", "block"):
        # the output is rounded to 16 bits: measured 2.1e-4 against 64 bits, at most half a unit of the last
        # place (4.9e-4) for one value
        return {"rel": 8e-4, "max": 2e-3}
    if kind == "hessian":
        return {"rel": 2e-6}   # sums of 8192 products in 32 bits: measured 3.4e-7 against 64 bits
    if kind == "factor":
        return {"rel": 2.5e-5}  # 32 bits at this dampening: measured 5.7e-6
    if kind == "search":
        # the errors: measured 4.6e-7.  A row's two best candidates may be as close as that, and then either
        # is right; one row of the smallest layer is 4e-3 of its rows
        return {"rel": 2e-6, "differ": 5e-3}
    if kind == "gptq":
        # a weight within the rounding of its sum of a decision boundary may go either way, and its error then
        # travels along the row: measured against 64 bits, 9 of 7168 rows differ, in 3.6e-5 of all integers;
        # one such row of the smallest layer is 1.2e-4
        return {"rel": 0.0, "differ": 5e-4}
    return "exact"


def _dequantised(codes, alpha, off, lo, hi):
    """Rows [lo, hi) of the weight, in 64 bits."""
    _, N = codes.shape
    G, q = alpha.shape[1:]
    W = torch.zeros((hi - lo, G, N // G), dtype=torch.float64, device="cuda")
    for i in range(q):
        sign = ((codes[lo:hi] >> i) & 1).view(hi - lo, G, N // G).double().mul_(2.0).sub_(1.0)
        W += sign * alpha[lo:hi, :, i, None].double()
    if off is not None:
        W += off[lo:hi, :, None].double()
    return W.view(hi - lo, N)


def _exact_linear(codes, alpha, off, X):
    M = codes.shape[0]
    Y = torch.empty((X.shape[0], M), dtype=torch.float64, device="cuda")
    Xt = X.double().t().contiguous()
    for lo in range(0, M, 2048):
        hi = min(M, lo + 2048)
        Y[:, lo:hi] = (_dequantised(codes, alpha, off, lo, hi) @ Xt).t()
    return Y


def _nearest(w, choices):
    """The member of `choices` nearest to each integer, the smaller one on a tie."""
    top = max(choices)
    table = [min(choices, key=lambda c: (abs(c - k), c)) for k in range(top + 1)]
    return torch.tensor(table, device=w.device, dtype=torch.float64)[w.clamp(0, top).long()]


def _exact_search_errors(case, seed):
    g = _gen(seed)
    M, N, n, q, grid = (case[k] for k in ("M", "N", "n", "q", "grid"))
    W, H = _weights(M, N, g).double(), _hessian_of(N, g).double()
    qbias = W.min(1).values
    span = W.max(1).values - qbias
    lo, hi = span / ((1 << (n + 1)) - 1), span / ((1 << (n - 1)) - 1)
    best = torch.full((M,), math.inf, dtype=torch.float64, device="cuda")
    for k in range(grid):
        S = lo + (hi - lo) * ((k + 1) / (grid + 1))
        for lab in _partitions(n, q):
            for a in range(0, M, 2048):
                b = min(M, a + 2048)
                w = W[a:b]
                t = ((w - qbias[a:b, None]) / S[a:b, None]).round().clamp_(0, (1 << n) - 1)
                d = S[a:b, None] * _nearest(t, _choices(lab, n, q)) + qbias[a:b, None] - w
                best[a:b] = torch.minimum(best[a:b], ((d @ H) * d).sum(1) * 0.5)
    return qbias, best


def exact(case, seed):
    kind = case["kind"]
    if kind == "linear":
        M, N, q, group, off, batch = (case[k] for k in ("M", "N", "q", "group", "offset", "batch"))
        Y = _exact_linear(*_layer_inputs(M, N, q, group, off, batch, case["outliers"], seed))
        return Y if batch > 1 else Y[0]
    if kind == "block":
        return [_exact_linear(*_block_layer_inputs(case, k, seed))[0] for k in range(len(_BLOCK))]
    g = _gen(seed)
    N = case["N"]
    if kind == "hessian":
        X, mix, loud = _calibration(case["T"], N, g)
        H = torch.zeros((N, N), dtype=torch.float64, device="cuda")
        for b in range(case["batches"]):
            if b:
                X = _calibration(case["T"], N, g, mix, loud)[0]
            Xd = X.double()
            H += 2.0 * (Xd.t().contiguous() @ Xd)
        return H
    if kind == "factor":
        return _upper_factor(_hessian_of(N, g))
    if kind == "search":
        qbias, best = _exact_search_errors(case, seed)
        return {"S": None, "qbias": qbias, "labels": None, "err": best}
    if kind == "gptq":
        return None  # whole numbers only
    n, q = case["n"], case["q"]
    _, S, qbias, labels = _fuse_inputs(case, g)
    weights = torch.tensor([(1 << i) / 2.0 for i in range(n)], dtype=torch.float64, device="cuda")
    rows = labels if case["rows"] else torch.tensor([labels], device="cuda", dtype=torch.int8)
    hat = torch.stack([((rows == c) * weights).sum(1) for c in range(q)], dim=1).sort(dim=1, descending=True).values
    S, qbias = S.double().view(case["M"], -1), qbias.double().view(case["M"], -1)
    return {"codes": None, "alpha": S[:, :, None] * hat[:, None, :], "offset": ((1 << n) - 1) / 2.0 * S + qbias, "packed": None}
