"""GPU parity of the quantiser (Sec. II-A Eq. 1-2, Sec. II-B Eq. 5-6, Sec. II-C Eq. 7) against
oracle/quantizer.py on small synthetic layers.

The device takes every integer decision in binary64 like the oracle but sums the quadratic form and
the error compensation in binary32, so:
  * search: a row's winner may differ from the oracle's only between candidates whose oracle errors
    agree to 1e-4 (relative); the reported error agrees to 1e-4;
  * GPTQ pass: all integers are members of the row's representable set, and every integer is
    EXPLAINED by the oracle: the oracle replays the pass in binary64 with the same factor U, column by
    column; wherever the device's integer differs from the oracle's own decision, the oracle's working
    weight t (in quantisation steps) must lie within EPS of a rounding boundary k + 1/2 of Eq. 5 step 1
    and the device's integer must be what the other side of that boundary gives (Eq. 6); the replay then
    continues from the device's integer, so later columns are checked against the same history.  Rows
    without such an event equal the oracle's bit for bit.  EPS = N * 2^(n+2) * 2^-24 steps: a working
    weight is at most 2^(n+1) steps (Eq. 7's smallest scale) and receives up to N binary32 updates of
    relative error 2^-24 each (twice that for the rounding of the products);
  * fusion with a tying per row: bit-exact against oracle/fuse.py.
"""
import functools
import os
import re

import numpy as np
import pytest
import torch

import bcq_synth
import paper_2407_02891_amd as bcq
from oracle import fuse, quantizer, ref
from paper_2407_02891_amd import build as hip_build
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def _layer(M, N, seed):
    """Weights with a Gaussian bulk and a few larger entries; calibration inputs with correlated
    channels and a handful of high-energy ones, 2 N samples."""
    rng = np.random.default_rng(seed)
    W = rng.standard_normal((M, N)) * 0.02
    W[rng.random((M, N)) < 0.01] *= 4.0
    T = 2 * N
    base = rng.standard_normal((N, T))
    mix = rng.standard_normal((N, 8)) @ rng.standard_normal((8, T))
    X = base + 0.5 * mix
    X[rng.choice(N, size=max(1, N // 32), replace=False)] *= 6.0
    W32 = W.astype(np.float32)
    H32 = quantizer.hessian(X).astype(np.float32)
    H32 = ((H32 + H32.T) / 2).astype(np.float32)
    return W32, H32


def _labels_of(partition, n):
    lab = np.empty(n, dtype=np.int8)
    for c, cls in enumerate(partition):
        for i in cls:
            lab[i - 1] = c
    return lab


def _partition_of(labels):
    q = int(labels.max()) + 1
    return tuple(sorted(tuple(i + 1 for i in range(len(labels)) if labels[i] == c) for c in range(q)))


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _eps_steps(N, n):
    """Largest distance (in quantisation steps) between the oracle's binary64 working weight and a rounding
    boundary at which the device, whose working copy is binary32, may round the other way."""
    return N * 2.0 ** (n + 2 - 24)


def _assert_gptq_explained(W32, U, S, b, choices, n, Wq_g, what=""):
    """Every device integer is the oracle's, or the other side of a near-tie (see the module docstring).
    Returns the number of near-tie events."""
    M, N = W32.shape
    for m in range(M):
        assert np.isin(Wq_g[m], choices[m]).all(), (what, m)
    events = quantizer.gptq_follow(W32, U, S, b, choices, n, Wq_g)
    eps = _eps_steps(N, n)
    worst = 0.0
    for (m, j, t, own, taken) in events:
        k = np.rint(t)
        side = 1.0 if t > k else -1.0
        assert t != k, (what, m, j, t, own, taken)
        dist = abs(t - (k + 0.5 * side))
        other = int(fuse.nearest_bcchoice(np.clip(np.array([k + side]), 0, 2 ** n - 1).astype(np.int64), choices[m])[0])
        assert dist <= eps and taken == other, (what, m, j, t, own, taken, other, dist, eps)
        worst = max(worst, dist)
    print(f"{what}: {len(events)} near-tie columns of {M * N}, largest distance {worst:.2e} steps (allowed {eps:.2e})")
    return len(events)


def _gpu_search(W32, H32, n, q, grid):
    M, N = W32.shape
    S = torch.empty(M, dtype=torch.float32, device="cuda")
    b = torch.empty(M, dtype=torch.float32, device="cuda")
    lab = torch.empty((M, n), dtype=torch.int8, device="cuda")
    err = torch.empty(M, dtype=torch.float32, device="cuda")
    ws = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
    bcq.quant_search(M, N, n, q, grid, _dev(W32), _dev(H32), S, b, lab, err, ws)
    torch.cuda.synchronize()
    return S.cpu().numpy(), b.cpu().numpy(), lab.cpu().numpy(), err.cpu().numpy()


@pytest.mark.parametrize("M,N,n,q,grid", [(70, 160, 3, 2, 6), (33, 192, 4, 3, 5), (16, 96, 5, 3, 3), (20, 64, 4, 2, 4)])
def test_search(M, N, n, q, grid):
    W32, H32 = _layer(M, N, seed=100 + N + n)
    S_o, b_o, p_o, e_o = quantizer.search(W32, H32, n, q, grid)
    S_g, b_g, lab_g, e_g = _gpu_search(W32, H32, n, q, grid)
    parts = fuse.all_partitions(n, q)
    assert np.array_equal(b_g, b_o.astype(np.float32))
    same = 0
    for m in range(M):
        part_g = _partition_of(lab_g[m])
        assert part_g in parts
        if part_g == parts[p_o[m]] and S_g[m] == np.float32(S_o[m]):
            same += 1
            continue
        # a different winner: the scale must be a grid point, and its oracle error must tie the best
        grid_pts = quantizer.scale_grid(float(W32[m].min()), float(W32[m].max()), n, grid)
        k = int(np.argmin(np.abs(grid_pts - S_g[m])))
        assert np.float32(grid_pts[k]) == S_g[m]
        wq = quantizer.quant_row(W32[m].astype(np.float64), grid_pts[k], b_o[m], fuse.bcchoice(part_g, n), n)
        e_alt = quantizer.output_error(W32[m:m + 1], wq[None, :], grid_pts[k:k + 1], b_o[m:m + 1], H32)[0]
        assert e_alt <= e_o[m] * (1 + 1e-4), (m, e_alt, e_o[m])
    assert same >= 0.9 * M, f"only {same} of {M} rows agree on the winner"
    assert np.allclose(e_g, e_o, rtol=1e-4, atol=0), np.abs(e_g / e_o - 1).max()


@pytest.mark.parametrize("M,N,n,q,grid,shift", [(5, 132, 3, 2, 3, 0), (130, 136, 3, 2, 2, 0), (33, 136, 4, 3, 2, 1),
                                                (3, 1288, 3, 3, 2, 0), (129, 40, 6, 2, 2, 0), (4, 8, 2, 1, 4, 0)])
def test_search_paths(M, N, n, q, grid, shift):
    """Both ways of feeding the quadratic form: split into halves beforehand (columns a multiple of 8, weights on 16 bytes) and
    split by the product, at the edges of tiles, chunks (1024 columns) and octets, against the oracle; a constant row (no
    range to scale by) and a row of the smallest weights; the lower triangle of H is not read."""
    W32, H32 = _layer(M, N, seed=700 + N + n)
    W32[0] = np.float32(0.02)
    if M > 1:
        W32[1] *= np.float32(2.0 ** -60)
    S_o, b_o, p_o, e_o = quantizer.search(W32, H32, n, q, grid)
    flat = torch.zeros(M * N + 4, dtype=torch.float32, device="cuda")
    flat[shift: shift + M * N] = _dev(W32).reshape(-1)
    H_up = _dev(H32)
    H_up[_dev(np.tril(np.ones((N, N), dtype=bool), -1))] = float("nan")
    S = torch.empty(M, dtype=torch.float32, device="cuda")
    b = torch.empty(M, dtype=torch.float32, device="cuda")
    lab = torch.empty((M, n), dtype=torch.int8, device="cuda")
    err = torch.empty(M, dtype=torch.float32, device="cuda")
    ws = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
    ws.fill_(0xff)
    bcq.quant_search(M, N, n, q, grid, flat[shift:], H_up, S, b, lab, err, ws)
    torch.cuda.synchronize()
    assert np.array_equal(b.cpu().numpy(), b_o.astype(np.float32))
    e_g = err.cpu().numpy()
    assert e_g[0] == 0.0 and np.allclose(e_g, e_o, rtol=1e-4, atol=0), np.abs(e_g / e_o - 1).max()
    parts = fuse.all_partitions(n, q)
    S_g, lab_g = S.cpu().numpy(), lab.cpu().numpy()
    same = sum(_partition_of(lab_g[m]) == parts[p_o[m]] and S_g[m] == np.float32(S_o[m]) for m in range(M))
    assert same >= 0.9 * M


def _search(W, H, n, q, grid):
    M, N = W.shape
    out = [torch.full((M,), 7.0, device="cuda") for _ in range(3)]
    labels = torch.full((M, n), 9, dtype=torch.int8, device="cuda")
    ws = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
    bcq.quant_search(M, N, n, q, grid, W, H, out[0], out[1], labels, out[2], ws)
    torch.cuda.synchronize()
    return [t.view(torch.int32).cpu() for t in out] + [labels.cpu()]


@pytest.mark.parametrize("M,N,n,q,grid,kind", [
    (256, 256, 3, 2, 3, "samples"), (257, 264, 4, 3, 2, "samples"), (700, 520, 3, 2, 2, "loud"), (513, 776, 2, 2, 4, "samples"), (513, 776, 2, 2, 12, "samples"),
    (300, 512, 5, 3, 3, "samples"), (400, 1032, 3, 2, 2, "one direction"), (260, 640, 8, 2, 1, "one direction"), (300, 264, 4, 2, 2, "zero"),
    (2048, 320, 3, 2, 2, "few samples"), (256, 736, 3, 2, 4, "indefinite"), (300, 296, 3, 2, 2, "infinite"), (1020, 776, 3, 2, 8, "tiny"), (510, 776, 3, 2, 3, "huge"),
    (765, 736, 3, 2, 4, "very indefinite"), (765, 1032, 3, 2, 8, "mirrored"), (510, 520, 4, 2, 3, "low rank"), (1020, 1032, 3, 2, 8, "16 bits"), (640, 2048, 3, 2, 8, "16 bits"),
    (600, 264, 3, 2, 2, "no diagonal"), (512, 1024, 5, 3, 3, "16 bits"), (264, 760, 3, 2, 4, "very indefinite"), (256, 768, 3, 2, 5, "samples"),
    (256, 776, 3, 2, 2, "samples"), (1400, 4096, 3, 2, 3, "one direction"),
    (5003, 1288, 3, 2, 3, "samples"), (2500, 3592, 4, 2, 2, "few samples")])
def test_search_screened(M, N, n, q, grid, kind):
    """Layers of 256 rows or more are screened: a bound excludes candidates before they are evaluated.  The results are the bits of the
    search of at most 255 rows at a time, which evaluates all: at the edges of tiles, chunks of candidates (48) and planes, with
    rows that are constant, zero, tiny, huge or hold infinities and no numbers, and with Hessians that let the bound exclude nearly everything or
    nothing, or that are not positive semidefinite (so that errors are negative, too)."""
    if M > 2048:  # these are for the large tiles
        tile = _constant("kScreenTile")
        assert -(-N // tile) * -(-M // tile) * {1288: 3, 3592: 2}[N] >= _constant("kScreenLargeFrom")
    g = torch.Generator(device="cuda").manual_seed(7 * M + N + n)
    W = torch.randn((M, N), device="cuda", generator=g) * 0.02
    W *= 1.0 + 3.0 * (torch.rand((M, N), device="cuda", generator=g) < 0.01)
    W[3], W[4], W[5] = 0.01, 0.0, W[5] * 1e-20
    W[6] *= 1e15
    W[7, 11], W[8, 5], W[9, N - 1] = float("inf"), float("nan"), -float("inf")
    W[10, 1:] = W[10, :1]
    W[M - 1, N // 2] = 3.0
    T = N // 4 if kind == "few samples" else 2 * N
    X = torch.randn((T, N), device="cuda", generator=g)
    X += 0.5 * torch.randn((T, 8), device="cuda", generator=g) @ torch.randn((8, N), device="cuda", generator=g)
    if kind == "loud":
        X[:, ::37] *= 2.0 ** 10
    H = 2.0 * (X.t().contiguous() @ X)
    if kind == "one direction":  # all candidates close to each other compared with |H|
        H = 100.0 * H.diagonal().mean() * torch.ones_like(H) + H
    if kind == "zero":
        H.zero_()
    if kind in ("tiny", "huge"):  # squares of its values are no binary32 numbers; channels with means, next to which the errors are small
        mean = 50.0 * torch.randn(N, device="cuda", generator=g)
        H += 2.0 * T * mean[:, None] * mean[None]
        H *= 2.0 ** (-110 if kind == "tiny" else 80)
    if kind == "infinite":
        H[17, 200] = H[200, 17] = float("inf")
    H = ((H + H.t()) * 0.5).contiguous()
    if kind in ("indefinite", "very indefinite"):  # errors positive for nearly all rows, and of both signs
        H.diagonal().sub_((0.3 if kind == "indefinite" else 1.0) * H.diagonal().mean())
    if kind == "mirrored":  # as large as a positive semidefinite H of its diagonal, with channel means; errors of either sign
        mean = 5.0 * torch.randn(N, device="cuda", generator=g)
        H += 2.0 * T * mean[:, None] * mean[None]
        H = 2.0 * torch.diag(H.diagonal()) - H
    if kind == "no diagonal":
        H.fill_diagonal_(0.0)
    if kind == "low rank":  # equal channels and weights that fall into line with them: errors of rounding, of either sign
        X = torch.randn((8, N // 4), device="cuda", generator=g).repeat_interleave(4, 1)
        X[:, 1::2] *= -1.0
        H = 2.0 * (X.t().contiguous() @ X)
        W[20:] = W[20:, ::2].repeat_interleave(2, 1)
    if kind == "16 bits":  # a Hessian that was kept in bfloat16, with channel means: small eigenvalues of either sign
        mean = 20.0 * torch.randn(N, device="cuda", generator=g)
        H = (H + 2.0 * T * mean[:, None] * mean[None]).bfloat16().float()
    whole = _search(W, H, n, q, grid)
    for lo in range(0, M, 255):
        part = _search(W[lo:lo + 255].clone(), H, n, q, grid)
        for a, b, what in zip(whole, part, ("S", "qbias", "err", "labels")):
            same = (a[lo:lo + 255] == b).reshape(len(b), -1).all(1)
            assert same.all(), (kind, what, lo + torch.nonzero(~same).flatten()[:8])


@pytest.mark.parametrize("M,N,n,q", [(70, 320, 3, 2), (40, 256, 4, 3), (9, 96, 3, 3)])
def test_gptq_pass(M, N, n, q):
    W32, H32 = _layer(M, N, seed=200 + N + n)
    S, b, p, _ = quantizer.search(W32, H32, n, q, grid=3)
    S32, b32 = S.astype(np.float32), b.astype(np.float32)
    parts = fuse.all_partitions(n, q)
    choices = [fuse.bcchoice(parts[i], n) for i in p]
    labels = np.stack([_labels_of(parts[i], n) for i in p])
    Wq_o = quantizer.gptq(W32, H32, S32.astype(np.float64), b32.astype(np.float64), choices, n)
    U32 = quantizer.cholesky_factor(H32).astype(np.float32)
    w_int = torch.full((M, N), 255, dtype=torch.uint8, device="cuda")
    ws = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
    W_dev = _dev(W32)
    bcq.quant_gptq(M, N, n, q, W_dev, _dev(U32), _dev(S32), _dev(b32), _dev(labels), w_int, ws)
    torch.cuda.synchronize()
    assert np.array_equal(W_dev.cpu().numpy(), W32)                      # the input is left alone
    Wq_g = w_int.cpu().numpy().astype(np.int64)
    S64, b64 = S32.astype(np.float64), b32.astype(np.float64)
    events = _assert_gptq_explained(W32, U32, S64, b64, choices, n, Wq_g, f"gptq {M}x{N} n={n} q={q}")
    if events == 0:
        assert np.array_equal(Wq_g, Wq_o)
    e_g = quantizer.output_error(W32, Wq_g, S64, b64, H32).sum()
    # and the compensation does its job: better than rounding every weight on its own
    Wq_rtn = np.stack([quantizer.quant_row(W32[m].astype(np.float64), S32[m], b32[m], choices[m], n) for m in range(M)])
    e_rtn = quantizer.output_error(W32, Wq_rtn, S32.astype(np.float64), b32.astype(np.float64), H32).sum()
    assert e_g < e_rtn


@pytest.mark.parametrize("M,N,n,q", [(33, 1156, 4, 3), (31, 516, 5, 3), (9, 644, 8, 4), (1, 1024, 2, 2), (65, 132, 6, 1)])
def test_gptq_blocks_and_panels(M, N, n, q):
    """The GPTQ pass at the edges of its blocks (128 columns, 32 rows, groups of 8 columns) and panels (512 columns), with
    tables of nibbles (up to four bits) and of bytes, every tying among the rows, and weights placed exactly on a rounding
    boundary of the first column (which the reciprocal of the scale must not decide differently from the division)."""
    rng = np.random.default_rng(500 + N + n)
    W32, H32 = _layer(M, N, seed=500 + N + n)
    parts = fuse.all_partitions(n, q)
    pick = rng.integers(0, len(parts), size=M)
    choices = [fuse.bcchoice(parts[i], n) for i in pick]
    labels = np.stack([_labels_of(parts[i], n) for i in pick])
    b32 = W32.min(axis=1)
    S32 = ((W32.max(axis=1) - b32) / (2 ** n - 1)).astype(np.float32)
    # halves of a grid of exactly representable steps
    S32[::2] = np.float32(2.0 ** -6) * (1 + (np.arange(S32[::2].size) % 3)).astype(np.float32)
    b32[::2] = -np.float32(0.25)
    W32[::2, 0] = b32[::2] + S32[::2] * (rng.integers(0, 2 ** n - 1, size=S32[::2].size) + 0.5).astype(np.float32)
    U32 = quantizer.cholesky_factor(H32).astype(np.float32)
    w_int = torch.full((M, N), 255, dtype=torch.uint8, device="cuda")
    ws = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
    ws.fill_(0xff)
    bcq.quant_gptq(M, N, n, q, _dev(W32), _dev(U32), _dev(S32), _dev(b32), _dev(labels), w_int, ws)
    torch.cuda.synchronize()
    Wq = w_int.cpu().numpy().astype(np.int64)
    S64, b64 = S32.astype(np.float64), b32.astype(np.float64)
    first = np.array([quantizer.quant_row(W32[m, :1].astype(np.float64), S64[m], b64[m], choices[m], n)[0] for m in range(M)])
    assert np.array_equal(Wq[:, 0], first)
    _assert_gptq_explained(W32, U32, S64, b64, choices, n, Wq, f"gptq {M}x{N} n={n} q={q}")


def _constant(name):
    """A constant of the quantiser's source, so that a test of what it decides notices when it moves."""
    text = open(os.path.join(hip_build.CSRC, "bcq_quant.hip")).read() + open(os.path.join(hip_build.CSRC, "bcq_screen.h")).read()
    return int(re.search(r"\b%s = (\d+)[,;]" % name, text)[1])


@functools.lru_cache(maxsize=1)
def _large_factor(N):
    return quantizer.cholesky_factor(_layer(1, N, seed=N)[1]).astype(np.float32)


@pytest.mark.parametrize("n,q", [(3, 2), (4, 3), (5, 3)])
def test_gptq_far_columns_beside_a_panel(n, q):
    """Layers with enough tiles beyond a panel have them updated by its errors in the launch of the next panel: two panels with such
    an update (so that both buffers of errors take both parts), two without, a ragged last one and ragged rows."""
    M, N = 7001, 2948

    def tiles(p1):  # beyond the panel that ends at p1
        return ((N - p1 + 127) // 128 * ((M + 127) // 128) + 7) // 8 * 8

    assert [tiles(p1) >= _constant("kBesideTiles") for p1 in (1024, 1536, 2048, 2560)] == [True, True, False, False]
    g = torch.Generator(device="cuda").manual_seed(n)
    W = torch.randn((M, N), device="cuda", generator=g) * 0.02
    W *= 1.0 + 3.0 * (torch.rand((M, N), device="cuda", generator=g) < 0.01)
    lo, hi = W.min(1).values, W.max(1).values
    S, b = ((hi - lo) / (2 ** n - 1) * (0.6 + 0.8 * torch.rand(M, device="cuda", generator=g))).contiguous(), lo.contiguous()
    parts = fuse.all_partitions(n, q)
    pick = np.arange(M) % len(parts)
    labels = np.stack([_labels_of(p, n) for p in parts])[pick]
    w_int = torch.full((M, N), 255, dtype=torch.uint8, device="cuda")
    ws = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
    ws.fill_(0xff)
    U32 = _large_factor(N)
    bcq.quant_gptq(M, N, n, q, W, _dev(U32), S, b, _dev(labels), w_int, ws)
    torch.cuda.synchronize()
    rows = [0, 31, 32, 127, 128, 3583, 3584, 6911, 6912, 6999, 7000]
    Wq = w_int[rows].cpu().numpy().astype(np.int64)
    _assert_gptq_explained(W[rows].cpu().numpy(), U32, S[rows].double().cpu().numpy(), b[rows].double().cpu().numpy(),
                           [fuse.bcchoice(parts[pick[m]], n) for m in rows], n, Wq, f"gptq {M}x{N} n={n} q={q}")


@pytest.mark.parametrize("M,N", [(2 ** 23 + 2 ** 20 + 165, 132), (2 ** 20 + 37, 8)])
def test_many_rows(M, N):
    """More rows than the byte offsets of a tile reach (2^23, from 128 columns on) or than are taken at a time: the search and the GPTQ
    pass give sampled rows what they give them alone."""
    n, q, grid = 2, 1, 1
    free, _ = torch.cuda.mem_get_info()
    if free < 10 * 4 * M * max(N, 64):
        pytest.skip("not enough device memory")
    g = torch.Generator(device="cuda").manual_seed(5)
    W = torch.randn((M, N), device="cuda", generator=g) * 0.02
    _, H32 = _layer(4, N, seed=N)
    H, Uf = _dev(H32), _dev(quantizer.cholesky_factor(H32).astype(np.float32))

    def both(W):
        rows = W.shape[0]
        S, b, err = (torch.empty(rows, device="cuda") for _ in range(3))
        lab = torch.full((rows, n), 7, dtype=torch.int8, device="cuda")
        w_int = torch.full((rows, N), 255, dtype=torch.uint8, device="cuda")
        ws = torch.empty(bcq.quant_workspace_bytes(rows, N), dtype=torch.uint8, device="cuda")
        bcq.quant_search(rows, N, n, q, grid, W, H, S, b, lab, err, ws)
        bcq.quant_gptq(rows, N, n, q, W, Uf, S, b, lab, w_int, ws)
        torch.cuda.synchronize()
        return S, b, lab, err, w_int

    whole = both(W)
    for lo in (0, 2 ** 20 - 128, M // 2 // 128 * 128, (M - 200) // 128 * 128):
        hi = min(M, lo + 300)
        for a, part in zip(whole, both(W[lo:hi].contiguous())):
            a = a[lo:hi]
            if a.dtype == torch.float32:
                assert torch.allclose(a, part, rtol=1e-5, atol=0)
            else:
                assert (a != part).float().mean() <= 1e-4   # (other rows of a tile may move the rounding of a sum)


def test_gptq_unusual_diagonals():
    """Diagonal entries of U at which a reciprocal does not stand for the division: infinite, zero, subnormal and with a subnormal or
    infinite reciprocal, and errors that are zero or leave the normal range.  Integers of a column-by-column replay in
    binary32 with divisions, bit for bit (one block; a weight that is not a number gives 0)."""
    M, N, n, q = 37, 96, 4, 3
    rng = np.random.default_rng(3)
    W32 = (rng.standard_normal((M, N)) * 0.02).astype(np.float32)
    W32[1] = np.float32(0.01)                                              # errors of zero
    W32[2] *= np.float32(2.0 ** -110)
    W32[3] *= np.float32(2.0 ** 100)
    U32 = (np.triu(rng.standard_normal((N, N)) * 0.3, 1) + np.diag(0.5 + rng.random(N))).astype(np.float32)
    for j, d in ((5, np.inf), (11, 2.0 ** 127), (17, 2.0 ** 125), (23, 2.0 ** -20), (31, -np.inf), (40, 2.0 ** 60), (70, 1e-41),
                 (80, 0.0)):
        U32[j, j] = d
        if abs(d) < 1e-3:
            U32[j, j + 1:] *= np.float32(2.0 ** -20)
    b32 = W32.min(axis=1)
    span = W32.max(axis=1) - b32
    S32 = np.where(span > 0, span / 15, 1.0).astype(np.float32)
    parts = fuse.all_partitions(n, q)
    pick = rng.integers(0, len(parts), size=M)
    labels = np.stack([_labels_of(parts[i], n) for i in pick])
    nearest = np.stack([fuse.nearest_bcchoice(np.arange(16), fuse.bcchoice(parts[i], n)) for i in pick])
    s, b, w = S32.astype(np.float64), b32.astype(np.float64), W32.copy()
    want = np.empty((M, N), dtype=np.uint8)
    with np.errstate(all="ignore"):
        for j in range(N):
            t = np.rint((w[:, j].astype(np.float64) - b) / s)
            wq = nearest[np.arange(M), np.nan_to_num(np.clip(t, 0, 15), nan=0.0).astype(np.int64)]
            want[:, j] = wq
            err = (w[:, j] - (s * wq + b).astype(np.float32)) / U32[j, j]
            w[:, j + 1:] = (w[:, j + 1:].astype(np.float64) - err[:, None].astype(np.float64) * U32[j, j + 1:]).astype(np.float32)
    w_int = torch.full((M, N), 255, dtype=torch.uint8, device="cuda")
    ws = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
    bcq.quant_gptq(M, N, n, q, _dev(W32), _dev(U32), _dev(S32), _dev(b32), _dev(labels), w_int, ws)
    torch.cuda.synchronize()
    got = w_int.cpu().numpy()
    assert np.array_equal(got, want), np.argwhere(got != want)[:10]


@pytest.mark.parametrize("n,q", [(2, 2), (3, 2), (4, 3), (5, 3), (8, 4)])
def test_gptq_decisions_where_binary32_does_not_tell(n, q):
    """The GPTQ pass decides from a binary32 quotient unless that is close to a half or the scale is out of the ordinary: weights on
    and next to the halves, offsets 2^20 steps away, scales of 2^-70 and 2^70, weights beyond the grid.  Without compensation
    (U diagonal) the integers are those of the definition in binary64, all of them."""
    M, N = 24, 136
    rng = np.random.default_rng(40 + n)
    S32 = (0.01 + 0.02 * rng.random(M)).astype(np.float32)
    S32[3] *= np.float32(2.0 ** -64)
    S32[4] *= np.float32(2.0 ** 76)
    S32[5] *= np.float32(-1.0)
    b32 = (-S32 * (2 ** (n - 1)) * rng.random(M)).astype(np.float32)
    b32[1] = S32[1] * np.float32(2.0 ** 20)
    b32[2] = -S32[2] * np.float32(2.0 ** 10)
    steps = rng.integers(-2, 2 ** n + 2, size=(M, N)) + rng.choice([0.0, 0.25, 0.5, 0.5 - 2.0 ** -20, 0.5 + 2.0 ** -22], size=(M, N))
    W32 = (b32[:, None] + steps * S32[:, None].astype(np.float64)).astype(np.float32)
    parts = fuse.all_partitions(n, q)
    pick = rng.integers(0, len(parts), size=M)
    labels = np.stack([_labels_of(parts[i], n) for i in pick])
    nearest = np.stack([fuse.nearest_bcchoice(np.arange(2 ** n), fuse.bcchoice(parts[i], n)) for i in pick])
    t = np.rint((W32.astype(np.float64) - b32[:, None]) / S32[:, None].astype(np.float64))
    want = np.take_along_axis(nearest, np.clip(t, 0, 2 ** n - 1).astype(np.int64), axis=1)
    w_int = torch.full((M, N), 255, dtype=torch.uint8, device="cuda")
    ws = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
    U = torch.diag(torch.linspace(0.5, 2.0, N)).cuda()
    bcq.quant_gptq(M, N, n, q, _dev(W32), U, _dev(S32), _dev(b32), _dev(labels), w_int, ws)
    torch.cuda.synchronize()
    got = w_int.cpu().numpy()
    assert np.array_equal(got, want), np.argwhere(got != want)[:10]


@pytest.mark.parametrize("n,q", [(3, 2), (4, 3), (5, 3)])
def test_gptq_rows_do_not_depend_on_their_neighbours(n, q):
    """Within a panel a row's integers are its own: the same beside ordinary rows as beside rows whose decisions binary32 does not
    tell (offsets of 2^20 steps, constant rows, scales of 2^-70, infinities), which send their wave through every group twice."""
    M, N = 40960, 512  # (enough that sums rounded otherwise would show in some integer)
    g = torch.Generator(device="cuda").manual_seed(n)
    W = torch.randn((M, N), device="cuda", generator=g) * 0.02
    X = torch.randn((2 * N, N), device="cuda", generator=g)
    H = (2.0 * (X.t().contiguous() @ X)).cpu().numpy()
    U = _dev(quantizer.cholesky_factor(H).astype(np.float32))
    lo, hi = W.min(1).values, W.max(1).values
    S, b = ((hi - lo) / ((1 << n) - 1) * 0.8).contiguous(), lo.contiguous()
    parts = torch.tensor(np.stack([_labels_of(p, n) for p in fuse.all_partitions(n, q)]), device="cuda")
    labels = parts[torch.arange(M, device="cuda") % len(parts)].contiguous()

    def integers(W, S, b):
        out = torch.full((M, N), 255, dtype=torch.uint8, device="cuda")
        ws = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
        bcq.quant_gptq(M, N, n, q, W.contiguous(), U, S, b, labels, out, ws)
        torch.cuda.synchronize()
        return out

    plain = integers(W, S, b)
    W, S, b = W.clone(), S.clone(), b.clone()
    k = torch.arange(0, M, 8, device="cuda")
    for first, what in enumerate(("far", "constant", "tiny", "infinite")):
        at = k[first::4]
        if what == "far":
            W[at] += S[at][:, None] * 2.0 ** 20
            b[at] += S[at] * 2.0 ** 20
        elif what == "constant":
            W[at], S[at], b[at] = 0.25, 0.0, 0.25
        elif what == "tiny":
            W[at], S[at], b[at] = W[at] * 2.0 ** -64, S[at] * 2.0 ** -64, b[at] * 2.0 ** -64
        else:
            W[at, 100] = float("inf")
    beside = integers(W, S, b)
    same = (plain == beside).all(1)
    same[k] = True
    assert same.all(), torch.nonzero(~same).flatten()[:8]
    assert (beside[k[1::4]] == beside[k[1::4]][:, :1]).all()  # (a constant row: one integer)


@pytest.mark.parametrize("M,N,n,q", [(37, 1024, 3, 2), (12, 512, 4, 3), (5, 1536, 5, 3), (8, 512, 4, 4)])
def test_from_linear_rows(M, N, n, q):
    rng = np.random.default_rng(300 + N + n + q)
    parts = fuse.all_partitions(n, q)
    pick = rng.integers(0, len(parts), size=M)
    labels = np.stack([_labels_of(parts[i], n) for i in pick])
    W_int = rng.integers(0, 2 ** n, size=(M, N), dtype=np.int64)
    W_int[:, : 2 ** n] = np.arange(2 ** n)
    S = (0.002 + 0.02 * rng.random(M)).astype(np.float32)
    qb = (rng.standard_normal(M) * 0.05).astype(np.float32)
    codes = torch.empty((M, N), dtype=torch.uint8, device="cuda")
    alpha = torch.empty((M, 1, q), dtype=torch.float16, device="cuda")
    off = torch.empty((M, 1), dtype=torch.float16, device="cuda")
    bcq.from_linear_rows(M, N, n, q, _dev(labels), _dev(W_int.astype(np.uint8)), _dev(S), _dev(qb), codes, alpha, off)
    torch.cuda.synchronize()
    planes = np.zeros((q, M, N // 32), dtype=np.uint32)
    a16 = np.empty((M, 1, q), dtype=np.float16)
    z16 = np.empty((M, 1), dtype=np.float16)
    for m in range(M):
        part = parts[pick[m]]
        wq = fuse.nearest_bcchoice(W_int[m:m + 1], fuse.bcchoice(part, n))
        pl, a64, z64 = fuse.fuse(wq, S[m:m + 1].astype(np.float64), qb[m:m + 1].astype(np.float64), part, n, N)
        planes[:, m] = pl[:, 0]
        a16[m], z16[m] = a64[0].astype(np.float16), z64[0].astype(np.float16)
    assert np.array_equal(codes.cpu().numpy(), bcq_synth.planes_to_codes(planes))
    assert np.array_equal(alpha.cpu().numpy().view(np.uint16), a16.view(np.uint16))
    assert np.array_equal(off.cpu().numpy().view(np.uint16), z16.view(np.uint16))
    x = rng.standard_normal((1, N)).astype(np.float16)
    layer = bcq.PackedLayer(M, N, q, N, True)
    layer.pack_from(codes, alpha, off)
    y = U.gpu_gemv(layer, U.to_dev(x.view(np.uint16).astype(np.int16)).view(torch.float16))
    U.gate(y[None, :], ref.gemm(planes, a16, z16, x), f"from_linear_rows n={n} q={q}")


@pytest.mark.parametrize("M,N,n,q", [(5, 1028, 3, 2), (33, 64, 8, 4), (4100, 96, 4, 3)])
@pytest.mark.parametrize("shift", [0, 1, 4, 8])
def test_fuse_and_pack_alignment(M, N, n, q, shift):
    """The widths of the fusion kernels (16, 4 or 1 weights per access, by the alignment of the pointers and of the rows) and
    of the packing (8-byte or single codes): all give the codes of the oracle, and the same blob."""
    rng = np.random.default_rng(N + n + shift)
    parts = fuse.all_partitions(n, q)
    pick = rng.integers(0, len(parts), size=M)
    labels = np.stack([_labels_of(parts[i], n) for i in pick])
    w = rng.integers(0, 256, size=(M, N), dtype=np.uint8)      # (bits beyond n are ignored)
    S = (0.002 + 0.02 * rng.random(M)).astype(np.float32)
    qb = (rng.standard_normal(M) * 0.05).astype(np.float32)
    w_dev = torch.zeros(M * N + 16, dtype=torch.uint8, device="cuda")
    w_dev[shift: shift + M * N] = _dev(w).reshape(-1)
    c_dev = torch.full((M * N + 16,), 0xee, dtype=torch.uint8, device="cuda")
    alpha = torch.empty((M, 1, q), dtype=torch.float16, device="cuda")
    off = torch.empty((M, 1), dtype=torch.float16, device="cuda")
    bcq.from_linear_rows(M, N, n, q, _dev(labels), w_dev[shift:], _dev(S), _dev(qb), c_dev[shift:], alpha, off)
    torch.cuda.synchronize()
    tables = {}
    for i in set(pick.tolist()):
        wq = fuse.nearest_bcchoice(np.arange(2 ** n)[None], fuse.bcchoice(parts[i], n))
        wq = np.pad(wq, ((0, 0), (0, (-wq.shape[1]) % 32)))
        pl, _, _ = fuse.fuse(wq, np.ones(1), np.zeros(1), parts[i], n, wq.shape[1])
        tables[i] = bcq_synth.planes_to_codes(pl)[0][: 2 ** n]
    want = np.stack([tables[i][w[m] & (2 ** n - 1)] for m, i in enumerate(pick.tolist())])
    got = c_dev.cpu().numpy()
    assert np.array_equal(got[shift: shift + M * N].reshape(M, N), want)
    assert (got[:shift] == 0xee).all() and (got[shift + M * N:] == 0xee).all()
    # one tying for the whole layer
    c2 = torch.full((M * N + 16,), 0xee, dtype=torch.uint8, device="cuda")
    a2 = torch.empty((M, 1, q), dtype=torch.float16, device="cuda")
    bcq.from_linear(M, N, N, n, q, labels[0].tolist(), w_dev[shift:], _dev(S), _dev(qb), c2[shift:], a2, off)
    torch.cuda.synchronize()
    assert np.array_equal(c2.cpu().numpy()[shift: shift + M * N].reshape(M, N), tables[int(pick[0])][w & (2 ** n - 1)])
    assert (c2.cpu().numpy()[shift + M * N:] == 0xee).all()
    if N % 32 == 0:
        blobs = []
        for codes in (_dev(want).reshape(-1), c_dev[shift: shift + M * N]):
            layer = bcq.PackedLayer(M, N, q, N, True)
            layer.packed.fill_(0x5a)
            blobs.append(layer.pack_from(codes, alpha, off).packed)
        assert torch.equal(blobs[0], blobs[1])
        back = torch.empty((M, N), dtype=torch.uint8, device="cuda")
        bcq.unpack(layer.desc, layer.packed, back, None, None)
        assert np.array_equal(back.cpu().numpy(), want)


@pytest.mark.parametrize("N,T", [(160, 300), (256, 64), (72, 1000)])
def test_hessian(N, T):
    """H = 2 X X^T (Sec. II-A) accumulated over two batches of inputs, against the oracle in binary64."""
    rng = np.random.default_rng(N + T)
    X = (rng.standard_normal((N, T)) * (1 + 5 * (rng.random((N, 1)) < 0.05))).astype(np.float32)   # [N][T], paper's orientation
    H_o = quantizer.hessian(X)
    Xt = _dev(X.T)                                                                                 # [T][N] for the device
    H = torch.zeros((N, N), dtype=torch.float32, device="cuda")
    T1 = T // 3
    bcq.quant_hessian(N, T1, Xt[:T1], H)
    bcq.quant_hessian(N, T - T1, Xt[T1:], H)
    torch.cuda.synchronize()
    H_g = H.cpu().numpy().astype(np.float64)
    scale = np.sqrt(np.outer(np.diag(H_o), np.diag(H_o)))
    assert np.abs(H_g - H_o).max() <= 1e-5 * scale.max() and (np.abs(H_g - H_o) / scale).max() <= 1e-5
    assert np.array_equal(H_g, H_g.T)


@pytest.mark.parametrize("N,T", [(4, 1), (132, 31), (124, 32), (516, 33), (260, 65), (1028, 16)])
def test_hessian_tiles_and_scales(N, T):
    """The split product at the edges of its tiles (128 columns, 32 samples, blocks of 4 x 4 tiles), with channels of very
    different size, channels that are zero in the first samples and a channel that grows by 2^20 after them (both make a
    tile choose its scales again), added to an H that is not symmetric.  Bound per element, in units of 2^-24 of sum |x_r x_c|:
    three binary32 roundings per 16 samples; the halves of an operand leave at most 2^-23 of it (2 units each), the dropped
    product of the two small halves is at most 2^-22 (4); the final addition 1: 9, of which 8 are allowed (the worst cases of
    the halves exclude each other).  A value far below its channel's largest is only held to 2^-27 of that one: the smallest
    step of a half is 2^-24 (rounded to nearest: 2^-25) and the scaled largest is at least 2^2."""
    rng = np.random.default_rng(N * 7 + T)
    X = rng.standard_normal((T, N)).astype(np.float32)
    X *= np.exp2(rng.integers(-40, 41, size=N)).astype(np.float32)
    X[: (T + 1) // 2, rng.random(N) < 0.2] = 0.0
    X[:, 1] = 0.0
    X[:1, 2] *= np.float32(2.0 ** -20)
    X[-1, 2] = np.float32(2.0 ** 20)
    H0 = np.zeros((N, N), dtype=np.float32)
    H0[0, 3] = 5.0
    H = _dev(H0)
    bcq.quant_hessian(N, T, _dev(X), H)
    torch.cuda.synchronize()
    X64 = X.astype(np.float64)
    want = H0 + 2.0 * (X64.T @ X64)
    big = np.abs(X64).max(axis=0)
    size = 2.0 * (np.abs(X64).T @ np.abs(X64))
    bound = (3 * ((T + 15) // 16) + 8) * 2.0 ** -24 * (size + np.abs(H0)) + 4.0 * T * 2.0 ** -27 * np.outer(big, big) * (T > 1)
    got = H.cpu().numpy().astype(np.float64)
    assert (np.abs(got - want) <= bound + 1e-44).all(), (np.abs(got - want) / (bound + 1e-44)).max()
    assert np.array_equal(got[4:, 4:], got[4:, 4:].T)
    # a channel that is not finite leaves every sum with it not finite and the others alone
    X[T - 1, N - 1] = np.inf
    H.zero_()
    bcq.quant_hessian(N, T, _dev(X), H)
    torch.cuda.synchronize()
    bad = H.cpu().numpy()
    assert not np.isfinite(bad[N - 1, N - 1]) and np.isfinite(bad[: N - 1, : N - 1]).all()


@pytest.mark.parametrize("T", [1, 2, 7, 16, 20, 21, 24, 32, 33])
def test_hessian_of_few_samples(T):
    """With few samples the roundings of the operands do not average out (up to 20 are summed in binary32): the result is as close to
    the binary64 one as a chain of binary32 multiply-adds is (5 % for a different order)."""
    N = 260
    rng = np.random.default_rng(T)
    X = rng.standard_normal((T, N)).astype(np.float32)
    H = torch.zeros((N, N), dtype=torch.float32, device="cuda")
    bcq.quant_hessian(N, T, _dev(X), H)
    torch.cuda.synchronize()
    X64 = X.astype(np.float64)
    want = 2.0 * (X64.T @ X64)
    chain = np.zeros((N, N), dtype=np.float32)
    for t in range(T):
        chain = (chain + np.outer(X64[t], X64[t])).astype(np.float32)
    err, err32 = np.linalg.norm(H.cpu().numpy() - want), np.linalg.norm(2.0 * chain.astype(np.float64) - want)
    print(f"T={T}: {err / np.linalg.norm(want):.2e}, binary32 chain {err32 / np.linalg.norm(want):.2e}")
    assert err <= 1.05 * err32


@pytest.mark.parametrize("N,T", [(132, 300), (260, 97), (516, 640)])
def test_hessian_channels_that_grow(N, T):
    """Channels that grow by 2^9 or 2^14 at one sample, or again and again, at every position of a step and of the two stages,
    one that starts late and small, and one with an infinity on the way: tiles whose scales from the first samples do not
    do are computed again.  Bound as in test_hessian_tiles_and_scales."""
    rng = np.random.default_rng(N + T)
    X = rng.standard_normal((T, N)).astype(np.float32)
    for c in range(0, 100, 3):
        X[rng.integers(1, T):, c] *= np.float32(2.0 ** rng.choice([9, 14]))
    for t in range(40, min(T, 240), 33):
        X[t:, 101] *= np.float32(2.0 ** 7)
    X[: T // 2, 102] = 0.0
    X[T // 2:, 102] *= np.float32(2.0 ** -9)
    X *= np.float32(2.0) ** rng.integers(-20, 1, size=N).astype(np.float32)
    H = torch.zeros((N, N), dtype=torch.float32, device="cuda")
    bcq.quant_hessian(N, T, _dev(X), H)
    torch.cuda.synchronize()
    X64 = X.astype(np.float64)
    want, size = 2.0 * (X64.T @ X64), 2.0 * (np.abs(X64).T @ np.abs(X64))
    total, big = np.abs(X64).sum(axis=0), np.abs(X64).max(axis=0)
    low = 2.0 * 2.0 ** -27 * (np.outer(big, total) + np.outer(total, big))
    bound = (3 * ((T + 15) // 16) + 8) * 2.0 ** -24 * size + low
    got = H.cpu().numpy().astype(np.float64)
    assert (np.abs(got - want) <= bound).all(), (np.abs(got - want) / bound).max()
    assert np.array_equal(got, got.T)
    X[T // 3, 103] = np.inf
    X[T // 2, 104] = np.nan
    H.zero_()
    bcq.quant_hessian(N, T, _dev(X), H)
    torch.cuda.synchronize()
    bad = H.cpu().numpy()
    assert not np.isfinite(bad[[103, 104]]).any()
    keep = np.setdiff1d(np.arange(N), [103, 104])
    assert (np.abs(bad[np.ix_(keep, keep)] - want[np.ix_(keep, keep)]) <= bound[np.ix_(keep, keep)]).all()


@pytest.mark.parametrize("N,loud,damp", [(384, 2.0 ** 10, 1e-4), (520, 2.0 ** 12, 1e-6)])
def test_factor_with_loud_channels(N, loud, damp):
    """Four channels 2^10 or 2^12 times as loud as the others at the start of every diagonal block: their entries are the largest
    of the columns that the panels multiply by a block's inverse, which scales them down again, so the ordinary entries must
    not be held to a step of the large ones.  Error per column of U against binary64, over that of a binary32 factorisation
    (LAPACK): at most 8, where binary32 matrix instructions give 2.3 and 4 (and this 2.3 and 2.6)."""
    from scipy.linalg import solve_triangular
    rng = np.random.default_rng(1)
    X = rng.standard_normal((2 * N, N)) + 0.5 * rng.standard_normal((2 * N, 8)) @ rng.standard_normal((8, N))
    for b in range(0, N, 128):
        X[:, b + 3: b + 7] *= loud
    H32 = (2 * X.T @ X).astype(np.float32)
    H32 = ((H32 + H32.T) / 2).astype(np.float32)

    def factor(dtype):
        Hd = H32.astype(dtype) + dtype(damp * np.mean(np.diag(H32.astype(np.float64)))) * np.eye(N, dtype=dtype)
        inv = solve_triangular(np.linalg.cholesky(Hd[::-1, ::-1]), np.eye(N, dtype=dtype), lower=True)
        return inv[::-1, ::-1].astype(np.float64)

    U_o, U_32 = factor(np.float64), factor(np.float32)
    U = torch.empty((N, N), dtype=torch.float32, device="cuda")
    ws = torch.empty(bcq.quant_factor_workspace_bytes(N), dtype=torch.uint8, device="cuda")
    bcq.quant_factor(N, damp, _dev(H32), U, ws)
    torch.cuda.synchronize()
    size = np.linalg.norm(U_o, axis=0)
    err, err32 = (np.linalg.norm((u - U_o) / size) for u in (U.cpu().numpy().astype(np.float64), U_32))
    print(f"N={N}: {err / N ** 0.5:.2e}, binary32 {err32 / N ** 0.5:.2e}")
    assert err <= 8 * err32


@pytest.mark.parametrize("N", [2564, 3072, 6660])
def test_factor_updates_beside_the_blocks(N):
    """Layers whose trailing updates run beside the diagonal blocks of the next panel: after a first panel of four channels (four
    terms, with as many tiles as the rule asks for, and with more than fit beside a panel: the rest goes before it) and after
    full panels.  Error per column of U against binary64, over that of a binary32 factorisation (LAPACK), as above."""
    from scipy.linalg import solve_triangular
    g = torch.Generator(device="cuda").manual_seed(N)
    X = torch.randn((2 * N, N), device="cuda", generator=g)
    X[:, :N // 32] *= 6
    H = 2 * (X.t().contiguous() @ X)
    H32 = ((H + H.t()) * 0.5).cpu().numpy()

    def factor(dtype):
        Hd = H32.astype(dtype)
        Hd[np.diag_indices(N)] += dtype(0.01 * np.mean(np.diag(H32).astype(np.float64)))
        inv = solve_triangular(np.linalg.cholesky(Hd[::-1, ::-1]), np.eye(N, dtype=dtype), lower=True)
        return inv[::-1, ::-1].astype(np.float64)

    U_o, U_32 = factor(np.float64), factor(np.float32)
    U = torch.full((N, N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(bcq.quant_factor_workspace_bytes(N), dtype=torch.uint8, device="cuda")
    bcq.quant_factor(N, 0.01, _dev(H32), U, ws)
    torch.cuda.synchronize()
    U_g = U.cpu().numpy().astype(np.float64)
    assert (np.tril(U_g, -1) == 0).all()
    size = np.linalg.norm(U_o, axis=0)
    err, err32 = (np.linalg.norm((u - U_o) / size, axis=0) for u in (U_g, U_32))
    print(f"N={N}: {err.max():.2e}, binary32 {err32.max():.2e}")
    assert err.max() <= 8 * err32.max()


def test_factor_of_many_channels():
    """9220 channels, where more than half of a trailing update does not fit beside the next panel's blocks: the leading block of
    U^T U, which every update reaches, against that of H_d^-1 in binary64, over the error of a binary32 factorisation (LAPACK)."""
    from scipy.linalg import cho_factor, cho_solve
    N, lead = 9220, 256
    g = torch.Generator(device="cuda").manual_seed(N)
    X = torch.randn((2 * N, N), device="cuda", generator=g)
    X[:, :N // 32] *= 6
    H = 2 * (X.t().contiguous() @ X)
    H = ((H + H.t()) * 0.5).contiguous()
    U = torch.full((N, N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(bcq.quant_factor_workspace_bytes(N), dtype=torch.uint8, device="cuda")
    bcq.quant_factor(N, 0.01, H, U, ws)
    torch.cuda.synchronize()
    assert not torch.tril(U, -1).any()
    H32, U_g = H.cpu().numpy(), U[:lead, :lead].cpu().numpy().astype(np.float64)

    def leading(dtype):
        Hd = H32.astype(dtype)
        Hd[np.diag_indices(N)] += dtype(0.01 * np.mean(np.diag(H32).astype(np.float64)))
        return cho_solve(cho_factor(Hd, overwrite_a=True, check_finite=False), np.eye(N, lead, dtype=dtype), check_finite=False)[:lead].astype(np.float64)

    K = leading(np.float64)
    err, err32 = (np.linalg.norm(k - K) / np.linalg.norm(K) for k in (U_g.T @ U_g, leading(np.float32)))
    print(f"{err:.2e}, binary32 {err32:.2e}")
    assert err <= 8 * err32


@pytest.mark.parametrize("N", [64, 132, 160, 384, 404, 408, 1000])   # (a last block of 4, 20 and 24 columns: products of as many terms)
def test_inverse_hessian_factor(N):
    """U with (H + 0.01 mean(diag H) I)^-1 = U^T U, U upper triangular, against the oracle's binary64 factor;
    the device works in binary32, so the comparison is relative to the size of the entries of U and the
    defining identity is checked in binary64 from the device's U."""
    rng = np.random.default_rng(N)
    _, H32 = _layer(8, N, seed=N)
    U_o = quantizer.cholesky_factor(H32)
    U = torch.full((N, N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(bcq.quant_factor_workspace_bytes(N), dtype=torch.uint8, device="cuda")
    H_dev = _dev(H32)
    bcq.quant_factor(N, 0.01, H_dev, U, ws)
    torch.cuda.synchronize()
    assert np.array_equal(H_dev.cpu().numpy(), H32)
    U_g = U.cpu().numpy().astype(np.float64)
    assert np.isfinite(U_g).all() and (np.tril(U_g, -1) == 0).all() and (np.diag(U_g) > 0).all()
    assert np.abs(U_g - U_o).max() <= 2e-4 * np.abs(U_o).max(), np.abs(U_g - U_o).max() / np.abs(U_o).max()
    Hd = H32.astype(np.float64) + 0.01 * np.mean(np.diag(H32.astype(np.float64))) * np.eye(N)
    assert np.abs(U_g.T @ U_g @ Hd - np.eye(N)).max() <= 2e-3
    # and it drives the GPTQ pass to the oracle's integers
    M, n, q = 24, 3, 2
    W32 = (rng.standard_normal((M, N)) * 0.02).astype(np.float32)
    S, b, p, _ = quantizer.search(W32, H32, n, q, grid=3)
    S32, b32 = S.astype(np.float32), b.astype(np.float32)
    parts = fuse.all_partitions(n, q)
    choices = [fuse.bcchoice(parts[i], n) for i in p]
    labels = np.stack([_labels_of(parts[i], n) for i in p])
    w_int = torch.empty((M, N), dtype=torch.uint8, device="cuda")
    ws2 = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
    bcq.quant_gptq(M, N, n, q, _dev(W32), U, _dev(S32), _dev(b32), _dev(labels), w_int, ws2)
    torch.cuda.synchronize()
    _assert_gptq_explained(W32, U_g, S32.astype(np.float64), b32.astype(np.float64), choices, n,
                           w_int.cpu().numpy().astype(np.int64), f"gptq with the device's factor, N={N}")


def test_constant_row_and_single_outlier_row():
    """Degenerate rows: a constant row (Eq. 7's interval is empty: scale 1, integers 0, error 0) and a row
    that is constant except for one large weight."""
    M, N, n, q, grid = 6, 128, 3, 2, 4
    W32, H32 = _layer(M, N, seed=11)
    W32[2] = np.float32(-0.0421)
    W32[4] = np.float32(0.01)
    W32[4, 77] = np.float32(0.9)
    S_o, b_o, p_o, e_o = quantizer.search(W32, H32, n, q, grid)
    S_g, b_g, lab_g, e_g = _gpu_search(W32, H32, n, q, grid)
    parts = fuse.all_partitions(n, q)
    assert S_g[2] == 1.0 and b_g[2] == W32[2, 0] and e_g[2] == 0.0 and _partition_of(lab_g[2]) == parts[0]
    assert np.array_equal(b_g, b_o.astype(np.float32))
    for m in range(M):
        assert _partition_of(lab_g[m]) == parts[p_o[m]] and S_g[m] == np.float32(S_o[m]), m
    assert np.allclose(e_g, e_o, rtol=1e-4, atol=0)
    U32 = quantizer.cholesky_factor(H32).astype(np.float32)
    w_int = torch.full((M, N), 255, dtype=torch.uint8, device="cuda")
    ws = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
    bcq.quant_gptq(M, N, n, q, _dev(W32), _dev(U32), _dev(S_g), _dev(b_g), _dev(lab_g), w_int, ws)
    torch.cuda.synchronize()
    Wq = w_int.cpu().numpy()
    assert (Wq[2] == 0).all()
    choices = [fuse.bcchoice(parts[i], n) for i in p_o]
    Wq_o = quantizer.gptq(W32, H32, S_g.astype(np.float64), b_g.astype(np.float64), choices, n)
    assert np.array_equal(Wq[4], Wq_o[4]) and Wq[4, 77] == Wq[4].max() > 0


def test_many_column_blocks():
    """A layer wide enough for 16 blocks of the GPTQ pass and 32 column tiles of the quadratic form;
    the oracle runs on sampled rows (rows are independent in both steps)."""
    M, N, n, q, grid = 300, 2048, 3, 2, 3
    W32, H32 = _layer(M, N, seed=9)
    rows = np.array([0, 63, 64, 255, 299])
    S_g, b_g, lab_g, e_g = _gpu_search(W32, H32, n, q, grid)
    S_o, b_o, p_o, e_o = quantizer.search(W32[rows], H32, n, q, grid)
    parts = fuse.all_partitions(n, q)
    assert np.array_equal(b_g[rows], b_o.astype(np.float32))
    assert np.allclose(e_g[rows], e_o, rtol=1e-4, atol=0)
    for k, m in enumerate(rows):
        assert _partition_of(lab_g[m]) == parts[p_o[k]] and S_g[m] == np.float32(S_o[k]), m
    U32 = quantizer.cholesky_factor(H32).astype(np.float32)
    w_int = torch.empty((M, N), dtype=torch.uint8, device="cuda")
    ws = torch.empty(bcq.quant_workspace_bytes(M, N), dtype=torch.uint8, device="cuda")
    bcq.quant_gptq(M, N, n, q, _dev(W32), _dev(U32), _dev(S_g), _dev(b_g), _dev(lab_g), w_int, ws)
    torch.cuda.synchronize()
    Wq_g = w_int.cpu().numpy().astype(np.int64)[rows]
    choices = [fuse.bcchoice(parts[i], n) for i in p_o]
    Sr, br = S_g[rows].astype(np.float64), b_g[rows].astype(np.float64)
    _assert_gptq_explained(W32[rows], U32, Sr, br, choices, n, Wq_g, "gptq 300x2048, sampled rows")


def test_quantise_then_multiply():
    """The whole chain on one small layer (quantize_layer: search, GPTQ pass, fusion, packing), then the
    product; it must reproduce the dequantised weights S W_q + qbias up to the binary16 scales."""
    from paper_2407_02891_amd.quantize import quantize_layer
    M, N, n, q = 48, 512, 3, 2
    W32, H32 = _layer(M, N, seed=77)
    layer, info = quantize_layer(_dev(W32), _dev(H32), n, q, grid=4)
    torch.cuda.synchronize()
    S, b = info["S"].cpu().numpy().astype(np.float64), info["qbias"].cpu().numpy().astype(np.float64)
    Wq = info["w_int"].cpu().numpy().astype(np.int64)
    rng = np.random.default_rng(5)
    x = rng.standard_normal((1, N)).astype(np.float16)
    y = U.gpu_gemv(layer, U.to_dev(x.view(np.uint16).astype(np.int16)).view(torch.float16))
    y_lin = (S[:, None] * Wq + b[:, None]) @ x[0].astype(np.float64)
    rms = np.sqrt(np.mean(y_lin ** 2))
    assert np.abs(y.astype(np.float64) - y_lin).max() <= 4e-3 * max(rms, np.abs(y_lin).max())
    # the result is what the oracle's chain gives from the same search result
    parts = fuse.all_partitions(n, q)
    choices = [fuse.bcchoice(_partition_of(l), n) for l in info["class_of_plane"].cpu().numpy()]
    assert all(_partition_of(l) in parts for l in info["class_of_plane"].cpu().numpy())
    _assert_gptq_explained(W32, info["U"].cpu().numpy(), S, b, choices, n, Wq, "quantize_layer 48x512")
    # and the quantised layer is a usable approximation of the original one on the calibration statistics
    e = quantizer.output_error(W32, Wq, S, b, H32).sum()
    ref_energy = np.einsum("mk,kl,ml->", W32.astype(np.float64), H32.astype(np.float64) / 2, W32.astype(np.float64))
    assert e < 0.25 * ref_energy
