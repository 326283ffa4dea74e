"""Per-sample gradients whose fp32 operands run as three bf16 parts on the
matrix units, at the edges of tiles, stages, loads and alignments, against
64-bit sums.

Bound per element: fp32 sums of K products differ from the exact sum by at
most about K * 2^-24 * sum |b a| whatever their order (each of at most K + 8
roundings is relative to a partial sum that sum |b a| bounds; the parts of a
product that the split leaves out are below 2^-24 of it and counted in the 8).
"""
import sys

import numpy as np
import pytest
import torch

from paper_2109_12298_amd import binding as dp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def placed(x, shift):
    """x on the device, its first element `shift` elements into an allocation."""
    buf = torch.zeros(x.numel() + shift, dtype=x.dtype, device=DEV)
    buf[shift:] = x.reshape(-1).to(DEV)
    return buf[shift:]


def linear(A, B, shift, bias=True, scale=1.5):
    """dp_grad_sample_linear on A [N, T, d_in], B [N, T, d_out]; guarded outputs."""
    N, T, di = A.shape
    do = B.shape[2]
    dt = dp.dtype_of(A)
    a, b = placed(A, shift), placed(B, shift)
    gW = torch.full((N * do * di + shift + 64,), 7.0, device=DEV)
    gb = torch.full((N * do + 64,), 7.0, device=DEV)
    sq = torch.full((N,), 7.0, device=DEV)
    ws = torch.empty(max(dp.dp_grad_sample_linear_workspace_bytes(N, T, di, do, dt), 4), dtype=torch.uint8, device=DEV)
    dp.dp_grad_sample_linear(a, b, dt, N, T, di, do, scale, gW[shift:], gb if bias else None, sq, None, ws)
    torch.cuda.synchronize()
    assert (gW[:shift] == 7).all() and (gW[shift + N * do * di:] == 7).all(), "wrote outside gW"
    assert (gb[N * do:] == 7).all(), "wrote outside gb"
    return (gW[shift:shift + N * do * di].reshape(N, do, di).cpu().numpy(), gb[:N * do].reshape(N, do).cpu().numpy(),
            sq.cpu().numpy())


CASES = [  # N, T, d_in, d_out
    (2, 2, 4, 8), (3, 31, 8, 4), (1, 32, 64, 128), (2, 33, 65, 129), (2, 64, 63, 127), (1, 65, 5, 9),
    (3, 17, 130, 66), (2, 96, 100, 400), (1, 130, 67, 260), (2, 7, 257, 33),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_linear_edges(case, shift, dtype):
    N, T, di, do = case
    if dtype == "bf16":
        di, do = max(di, 8), max(do, 8)
    say("linear", case, "shift", shift, dtype)
    g = torch.Generator().manual_seed(N * 1000 + T)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    A = (torch.randn(N, T, di, generator=g) * 3).to(td)
    B = (torch.randn(N, T, do, generator=g) / 7).to(td)
    gW, gb, sq = linear(A, B, shift)
    A64, B64 = A.double().numpy(), B.double().numpy()
    ref = 1.5 * np.einsum("nti,ntj->nij", B64, A64)
    mag = 1.5 * np.einsum("nti,ntj->nij", abs(B64), abs(A64))
    assert (abs(gW - ref) <= (T + 8) * 2.0 ** -24 * mag).all()
    assert (abs(gb - 1.5 * B64.sum(1)) <= (T + 8) * 2.0 ** -24 * 1.5 * abs(B64).sum(1)).all()
    sref = (gW.astype(np.float64) ** 2).sum((1, 2)) + (gb.astype(np.float64) ** 2).sum(1)
    assert (abs(sq - sref) <= 1e-5 * sref).all()      # 64 + log2-deep trees of positive terms


# N, T, d_in, d_out: the tiles that the size of the grid, the positions and the padding choose (64 x 128 and
# 128 x 64, 64 x 64 with one and two stages), at both sides of the lines between them
TILES = [
    (129, 193, 64, 128), (129, 193, 128, 64), (129, 192, 64, 128), (128, 193, 64, 128), (20, 200, 100, 400),
    (257, 2, 64, 64), (256, 2, 64, 64), (300, 16, 17, 33), (300, 17, 33, 17), (300, 47, 63, 65), (300, 49, 4, 5),
    (90, 33, 130, 66), (260, 260, 20, 12), (257, 15, 8, 70), (513, 65, 9, 17), (172, 70, 129, 131), (520, 200, 64, 128),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", TILES, ids=lambda c: "x".join(map(str, c)))
def test_linear_tiles(case, dtype):
    N, T, di, do = case
    if dtype == "bf16":
        di, do = max(di, 8) | 1, max(do, 8)
    say("linear tiles", case, dtype)
    g = torch.Generator().manual_seed(N + T)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    A = (torch.randn(N, T, di, generator=g) * 3).to(td)
    B = (torch.randn(N, T, do, generator=g) / 7).to(td)
    gW, gb, sq = linear(A, B, 1)
    A64, B64 = A.double(), B.double()
    ref = 1.5 * torch.bmm(B64.transpose(1, 2).contiguous(), A64).numpy()
    mag = 1.5 * torch.bmm(B64.abs().transpose(1, 2).contiguous(), A64.abs()).numpy()
    assert (abs(gW - ref) <= (T + 8) * 2.0 ** -24 * mag).all()
    assert (abs(gb - 1.5 * B64.sum(1).numpy()) <= (T + 8) * 2.0 ** -24 * 1.5 * B64.abs().sum(1).numpy()).all()
    sref = (gW.astype(np.float64) ** 2).sum((1, 2)) + (gb.astype(np.float64) ** 2).sum(1)
    assert (abs(sq - sref) <= 1e-5 * sref).all()      # 64 + log2-deep trees of positive terms


@pytest.mark.parametrize("case", [(200, 100, 400), (193, 70, 128), (100, 130, 130), (16, 64, 17)], ids=str)
def test_linear_result_does_not_depend_on_batch(case):
    """The tiles depend on the batch; a sample's gradients and norm do not, bit for bit."""
    T, di, do = case
    say("linear batches", case)
    g = torch.Generator().manual_seed(23)
    A, B = torch.randn(300, T, di, generator=g), torch.randn(300, T, do, generator=g)
    whole = linear(A, B, 0)
    for n in (1, 20):
        part = linear(A[:n].contiguous(), B[:n].contiguous(), 0)
        for a, b in zip(whole, part):
            np.testing.assert_array_equal(a[:n], b)


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.4e38])
def test_linear_non_finite(value):
    """A value that bf16 cannot hold reaches exactly the outputs it reaches in plain fp32 sums."""
    N, T, di, do = 2, 40, 70, 140
    say("linear non-finite", value)
    g = torch.Generator().manual_seed(5)
    A, B = torch.randn(N, T, di, generator=g), torch.randn(N, T, do, generator=g) / 100
    A[1, 33, 69] = value
    B[1, 33, 3] = 0.0
    gW, gb, sq = linear(A, B, 0, scale=1.0)
    ref = np.einsum("nti,ntj->nij", B.double().numpy(), A.double().numpy())
    with np.errstate(over="ignore"):
        np.testing.assert_array_equal(np.isnan(gW), np.isnan(ref))
        np.testing.assert_array_equal(np.isinf(gW), np.isinf(ref.astype(np.float32)))
    ok = np.isfinite(ref)
    mag = np.einsum("nti,ntj->nij", abs(B.double().numpy()), abs(A.double().numpy()))
    assert (abs(gW[ok] - ref[ok]) <= (T + 8) * 2.0 ** -24 * mag[ok]).all()
    assert np.isfinite(sq[0]) and not np.isfinite(sq[1])


def test_linear_small_magnitudes():
    """Backprops near the smallest normal numbers keep fp32's accuracy: their
    lowest bits lie below bf16's smallest subnormal."""
    N, T, di, do = 1, 32, 64, 128
    g = torch.Generator().manual_seed(6)
    A, B = torch.randn(N, T, di, generator=g), torch.randn(N, T, do, generator=g) * 2.0 ** -105
    say("linear small magnitudes")
    gW, _, _ = linear(A, B, 0, scale=1.0)
    ref = np.einsum("nti,ntj->nij", B.double().numpy(), A.double().numpy())
    mag = np.einsum("nti,ntj->nij", abs(B.double().numpy()), abs(A.double().numpy()))
    assert (abs(gW - ref) <= (T + 8) * 2.0 ** -24 * mag + 2.0 ** -140).all()


def test_linear_bias_error():
    """The bias gradient adds a stage's rows up before they join its sum.  A rounding is 0.42 * 2^-24 (rms) of
    its partial sum.  Over T = 256, the squares of a thread's 8 partial sums (4.4 of the whole's), a stage's 4 rows
    in pairs (2) and 8 row groups in pairs (3) give 0.42 * 2^-24 * sqrt(9.4) = 0.8e-7; a quarter more is
    allowed.  (Row after row, 32 of a thread and then 8 groups, gives 1.1e-7.)"""
    N, T, di, do = 64, 256, 100, 400
    say("linear bias error")
    g = torch.Generator().manual_seed(19)
    A, B = torch.randn(N, T, di, generator=g), torch.randn(N, T, do, generator=g)
    _, gb, _ = linear(A, B, 0, scale=1.0)
    ref = B.double().numpy().sum(1)
    assert np.linalg.norm(gb - ref) <= 0.97e-7 * np.linalg.norm(ref)


def small_feature_scales(n, e):
    """2^e for every second feature, 1 for the others."""
    return torch.where(torch.arange(n) % 2 == 1, 2.0 ** e, 1.0).double()


@pytest.mark.parametrize("e", [-114, -120, -126, -133, -140])
def test_linear_tiny_values(e):
    """Features of any size, subnormal ones among them, keep fp32's bits: the roundings of the sums alone
    are left, of which each is at most 2^-24 and K + 8 add in quadrature over independent terms."""
    N, T, di, do = 2, 64, 66, 130
    say("linear tiny values", e)
    g = torch.Generator().manual_seed(16)
    A = (torch.randn(N, T, di, generator=g).double() * small_feature_scales(di, e)).float()
    B = torch.randn(N, T, do, generator=g) * 2.0 ** 60
    gW, _, _ = linear(A, B, 0, scale=1.0)
    ref = np.einsum("nti,ntj->nij", B.double().numpy(), A.double().numpy())
    for j in (0, 1):
        err, size = gW[:, :, j::2] - ref[:, :, j::2], ref[:, :, j::2]
        assert np.linalg.norm(err) <= (T + 8) ** 0.5 * 2.0 ** -24 * np.linalg.norm(size)


@pytest.mark.parametrize("e", [-120, -133])
def test_conv_tiny_values(e):
    N, ci, co, H = 2, 40, 36, 14
    say("conv tiny values", e)
    g = torch.Generator().manual_seed(17)
    X = (torch.randn(N, ci, H, H, generator=g).double() * small_feature_scales(ci, e)[:, None, None]).float()
    GY = torch.randn(N, co, H, H, generator=g) * 2.0 ** 60
    gW, _, _ = conv(X, GY, 3, 1, 1, 0, 1.0)
    ref = conv_reference(X, GY, 3, 1, 1, 1.0)[0].reshape(N, co, ci, 9)
    err = gW.reshape(N, co, ci, 9) - ref
    for j in (0, 1):
        assert np.linalg.norm(err[:, :, j::2]) <= (H * H + 8) ** 0.5 * 2.0 ** -24 * np.linalg.norm(ref[:, :, j::2])


@pytest.mark.parametrize("value", [2.0 ** 103, 2.0 ** 104, 1e35])
def test_linear_large_values(value):
    """On both sides of the magnitude that can be split, with ordinary results."""
    N, T, di, do = 2, 40, 70, 140
    say("linear large values", value)
    g = torch.Generator().manual_seed(18)
    A, B = torch.randn(N, T, di, generator=g), torch.randn(N, T, do, generator=g) * 2.0 ** -60
    A[1, 33, 69] = value
    gW, _, sq = linear(A, B, 0, scale=1.0)
    ref = np.einsum("nti,ntj->nij", B.double().numpy(), A.double().numpy())
    mag = np.einsum("nti,ntj->nij", abs(B.double().numpy()), abs(A.double().numpy()))
    assert (abs(gW - ref) <= (T + 8) * 2.0 ** -24 * mag).all()
    assert np.isfinite(sq).all()


# N, Cin, Cout, H, W, k, stride, pad: shapes that the automatic choice gives the
# bf16-matrix kernel, at the edges of its channel blocks (32, 64), units of
# eight columns, row chunks, tap groups and shifts
CONVS = [
    (2, 32, 64, 16, 16, 3, 1, 1), (3, 24, 33, 15, 17, 3, 1, 1), (1, 65, 40, 13, 24, 3, 1, 0), (1, 33, 64, 20, 9, 3, 1, 2),
    (1, 25, 10, 56, 56, 3, 1, 1), (2, 40, 130, 13, 16, 3, 1, 1), (1, 31, 64, 33, 40, 3, 2, 1), (2, 64, 64, 18, 23, 3, 2, 0),
    (1, 24, 32, 28, 30, 3, 1, 1), (1, 25, 10, 56, 63, 3, 1, 1), (1, 33, 64, 20, 24, 3, 1, 2),
]
CONVS_BF16 = CONVS + [
    (3, 24, 40, 27, 27, 5, 2, 2), (2, 40, 24, 17, 18, 5, 1, 0), (1, 24, 24, 19, 21, 7, 1, 3), (2, 26, 33, 21, 26, 4, 2, 1),
    (1, 30, 64, 14, 15, 2, 1, 0), (2, 64, 32, 25, 25, 3, 3, 1), (1, 32, 32, 32, 32, 9, 2, 4),
    # several tap groups, with rows of GY that fill their units exactly
    (2, 24, 40, 32, 32, 5, 2, 2), (2, 24, 40, 31, 31, 5, 2, 2), (2, 32, 64, 32, 32, 4, 2, 1), (1, 64, 64, 32, 32, 7, 2, 3),
    (2, 32, 64, 15, 15, 4, 1, 2), (2, 32, 64, 14, 14, 5, 1, 3), (1, 32, 64, 48, 48, 5, 3, 1), (1, 32, 32, 13, 13, 6, 1, 4),
]
# shapes on the other side of that choice, by their grid or their size
CONVS_OTHER = [
    (2, 33, 31, 20, 9, 3, 1, 2), (1, 64, 64, 12, 63, 3, 1, 1), (2, 40, 130, 11, 11, 3, 1, 1), (300, 32, 64, 12, 12, 3, 1, 1),
    (2, 25, 70, 10, 57, 3, 1, 1), (2, 40, 24, 13, 14, 5, 1, 0), (2, 64, 32, 9, 9, 3, 3, 1), (2, 32, 64, 16, 16, 5, 2, 2),
    (2, 32, 64, 16, 16, 4, 2, 1), (2, 32, 64, 24, 24, 5, 3, 1), (6, 27, 5, 37, 63, 3, 1, 1), (3, 116, 31, 7, 8, 5, 1, 2),
]


def conv(X, GY, k, stride, pad, shift, scale=1.5):
    N, ci, H, W = X.shape
    co, ho, wo = GY.shape[1:]
    dt = dp.dtype_of(X)
    x, y = placed(X, shift), placed(GY, shift)
    n = N * co * ci * k * k
    gW = torch.full((n + shift + 64,), 7.0, device=DEV)
    gb = torch.full((N * co + 64,), 7.0, device=DEV)
    sq = torch.full((N,), 7.0, device=DEV)
    geom = (k, k, stride, stride, pad, pad)
    ws = torch.empty(max(dp.dp_grad_sample_conv2d_workspace_bytes(N, ci, H, W, co, *geom), 4), dtype=torch.uint8,
                     device=DEV)
    dp.dp_grad_sample_conv2d(x, y, dt, N, ci, H, W, co, ho, wo, *geom, 1, 1, 1, scale, gW[shift:], gb, sq, None, ws)
    torch.cuda.synchronize()
    assert (gW[:shift] == 7).all() and (gW[shift + n:] == 7).all() and (gb[N * co:] == 7).all(), "wrote outside"
    return (gW[shift:shift + n].reshape(N, co, ci * k * k).cpu().numpy(), gb[:N * co].reshape(N, co).cpu().numpy(),
            sq.cpu().numpy())


def conv_reference(X, GY, k, stride, pad, scale=1.5):
    """The gradients and the sums of the terms' magnitudes, in 64 bits."""
    y = GY.double().flatten(2)
    u = torch.nn.functional.unfold(X.double(), k, padding=pad, stride=stride).transpose(1, 2)
    return scale * torch.bmm(y, u).numpy(), scale * torch.bmm(y.abs(), u.abs()).numpy(), scale * y.sum(2).numpy()


def check_conv(dtype, case, shift):
    N, ci, co, H, W, k, st, pad = case
    say("conv", case, dtype, "shift", shift)
    g = torch.Generator().manual_seed(ci * 100 + H)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    ho, wo = (H + 2 * pad - k) // st + 1, (W + 2 * pad - k) // st + 1
    X = torch.randn(N, ci, H, W, generator=g).to(td)
    GY = (torch.randn(N, co, ho, wo, generator=g) / 5).to(td)
    gW, gb, sq = conv(X, GY, k, st, pad, shift)
    ref, mag, rb = conv_reference(X, GY, k, st, pad)
    bound = (ho * wo + 8) * 2.0 ** -24
    assert (abs(gW - ref) <= bound * mag).all()
    assert (abs(gb - rb) <= bound * 1.5 * GY.double().abs().sum((2, 3)).numpy()).all()
    sref = (gW.astype(np.float64) ** 2).sum((1, 2)) + (gb.astype(np.float64) ** 2).sum(1)
    assert (abs(sq - sref) <= 1e-5 * sref).all()
    return gW, X, GY


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("dtype,case", [("f32", c) for c in CONVS] + [("bf16", c) for c in CONVS_BF16],
                         ids=lambda c: c if isinstance(c, str) else "x".join(map(str, c)))
def test_conv_edges(dtype, case, shift):
    gW, X, GY = check_conv(dtype, case, shift)
    # the kernel ran: sums in the order of the fp32 matrix units differ from its own somewhere
    before = dp.dp_conv2d_set_path(dp.DP_CONV_ROWS)
    try:
        other = conv(X, GY, case[5], case[6], case[7], shift)[0]
    finally:
        dp.dp_conv2d_set_path(before)
    assert not np.array_equal(gW, other), "not the bf16-matrix kernel"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CONVS_OTHER, ids=lambda c: "x".join(map(str, c)))
def test_conv_other_side_of_the_choice(dtype, case):
    check_conv(dtype, case, 0)


@pytest.mark.parametrize("dtype,case", [("f32", (6, 184, 26, 36, 57, 3, 1, 1)), ("f32", (12, 42, 11, 13, 63, 3, 1, 1)),
                                        ("f32", (9, 32, 69, 19, 45, 3, 3, 1)), ("bf16", (149, 116, 31, 7, 8, 5, 1, 2)),
                                        ("bf16", (98, 160, 89, 8, 8, 5, 1, 2))],
                         ids=lambda c: c if isinstance(c, str) else "x".join(map(str, c)))
def test_conv_choice_is_not_the_slower_kernel(dtype, case):
    """Layers that the bf16-matrix kernel takes two to four times as long for: the choice is within a third of
    the best kernel that can be forced."""
    N, ci, co, H, W, k, st, pad = case
    say("conv choice", dtype, case)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    ho, wo = (H + 2 * pad - k) // st + 1, (W + 2 * pad - k) // st + 1
    X, GY = torch.randn(N, ci, H, W, device=DEV).to(td), torch.randn(N, co, ho, wo, device=DEV).to(td)
    gW, gb, sq = torch.empty(N, co, ci * k * k, device=DEV), torch.empty(N, co, device=DEV), torch.empty(N, device=DEV)
    geom = (k, k, st, st, pad, pad)
    ws = torch.empty(max(dp.dp_grad_sample_conv2d_workspace_bytes(N, ci, H, W, co, *geom), 4), dtype=torch.uint8, device=DEV)
    times = {}
    for path in (dp.DP_CONV_TILED, dp.DP_CONV_ROWS, dp.DP_CONV_AUTO):
        before = dp.dp_conv2d_set_path(path)
        try:
            for _ in range(4):
                s, e = torch.cuda.Event(True), torch.cuda.Event(True)
                s.record()
                for _ in range(10):
                    dp.dp_grad_sample_conv2d(X, GY, dp.dtype_of(X), N, ci, H, W, co, ho, wo, *geom, 1, 1, 1, 1.0, gW, gb,
                                             sq, None, ws)
                e.record()
                torch.cuda.synchronize()
                times[path] = min(times.get(path, 1e9), s.elapsed_time(e) * 100)
        finally:
            dp.dp_conv2d_set_path(before)
    print("[case] us", times, file=sys.stderr, flush=True)
    assert times[dp.DP_CONV_AUTO] <= 1.33 * min(times.values())


@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3.4e38])
def test_conv_non_finite(value):
    N, ci, co, H, k = 2, 40, 36, 14, 3
    say("conv non-finite", value)
    g = torch.Generator().manual_seed(9)
    X, GY = torch.randn(N, ci, H, H, generator=g), torch.randn(N, co, H, H, generator=g) / 100
    X[1, 39, 0, 13] = value                  # a corner: only some taps reach it
    GY[1, 5] = 0.0
    gW, gb, sq = conv(X, GY, k, 1, 1, 0, 1.0)
    # in 64 bits the padding's zeros must not meet the value: sum tap by tap
    ref, mag = conv_terms(X, GY, k, 1, 1)
    with np.errstate(over="ignore"):
        np.testing.assert_array_equal(np.isnan(gW), np.isnan(ref))
        np.testing.assert_array_equal(np.isinf(gW), np.isinf(ref.astype(np.float32)))
    ok = np.isfinite(ref)
    assert (abs(gW[ok] - ref[ok]) <= (H * H + 8) * 2.0 ** -24 * mag[ok]).all()
    assert np.isfinite(sq[0]) and not np.isfinite(sq[1])


def conv_terms(X, GY, k, stride, pad):
    """Per tap the sums over the positions inside the input alone, and the sums of their magnitudes, in 64 bits."""
    N, ci, H, W = X.shape
    co, ho, wo = GY.shape[1:]
    x, y = X.double().numpy(), GY.double().numpy()
    ref, mag = np.zeros((N, co, ci, k, k)), np.zeros((N, co, ci, k, k))
    with np.errstate(invalid="ignore", over="ignore"):
        for u in range(k):
            for v in range(k):
                rows = [o for o in range(ho) if 0 <= o * stride + u - pad < H]
                cols = [o for o in range(wo) if 0 <= o * stride + v - pad < W]
                a = x[:, :, [o * stride + u - pad for o in rows]][:, :, :, [o * stride + v - pad for o in cols]]
                b = y[:, :, rows][:, :, :, cols]
                a, b = a.reshape(N, ci, -1), b.reshape(N, co, -1)
                ref[:, :, :, u, v] = np.einsum("nop,ncp->noc", b, a)
                mag[:, :, :, u, v] = np.einsum("nop,ncp->noc", abs(b), abs(a))
    return ref.reshape(N, co, -1), mag.reshape(N, co, -1)


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3e38])
@pytest.mark.parametrize("dtype,case", [("f32", (2, 40, 36, 14, 13, 3, 1, 1)), ("f32", (1, 33, 64, 21, 22, 3, 2, 1)),
                                        ("bf16", (2, 40, 36, 14, 13, 3, 1, 0)), ("bf16", (2, 24, 40, 32, 32, 5, 2, 2)),
                                        ("bf16", (1, 64, 33, 15, 15, 4, 1, 2))],
                         ids=lambda c: c if isinstance(c, str) else "x".join(map(str, c)))
def test_conv_sums_again(dtype, case, value):
    """Values that the bf16 sums cannot take reach exactly the outputs they reach in plain fp32 sums, and all
    other outputs keep the bound."""
    N, ci, co, H, W, k, st, pad = case
    say("conv sums again", dtype, case, value)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(20)
    ho, wo = (H + 2 * pad - k) // st + 1, (W + 2 * pad - k) // st + 1
    X = torch.randn(N, ci, H, W, generator=g).to(td)
    GY = (torch.randn(N, co, ho, wo, generator=g) / 1000).to(td)
    X[0, ci - 1, 0, W - 1] = X[0, 3, H // 2, 0] = value      # a corner and an edge: only some taps reach them
    GY[0, 5] = 0.0
    gW, gb, sq = conv(X, GY, k, st, pad, 0, 1.0)
    ref, mag = conv_terms(X, GY, k, st, pad)
    np.testing.assert_array_equal(np.isnan(gW), np.isnan(ref))
    np.testing.assert_array_equal(np.isinf(gW), np.isinf(ref))
    ok = np.isfinite(ref)
    assert (gW[np.isinf(ref)] == ref[np.isinf(ref)]).all()
    assert (abs(gW[ok] - ref[ok]) <= (ho * wo + 8) * 2.0 ** -24 * mag[ok]).all()
    assert np.isfinite(sq[1:]).all() and not np.isfinite(sq[0])


@pytest.mark.parametrize("kind", ["linear", "conv", "conv_bf16"])
def test_non_finite_cost(kind):
    """A batch with non-finite samples takes the fp32 matrix units, not one multiply-add per lane and position:
    a pass over memory and MFMAs of a sixteenth of the rate, so some ten times the ordinary pass at most."""
    say("non-finite cost", kind)
    dt = dp.DP_BF16 if kind == "conv_bf16" else dp.DP_F32
    td = torch.bfloat16 if dt == dp.DP_BF16 else torch.float32
    if kind == "linear":
        N, T, di, do = 64, 256, 100, 400
        a, b = torch.randn(N, T, di, device=DEV), torch.randn(N, T, do, device=DEV)
        gW, gb = torch.empty(N, do, di, device=DEV), torch.empty(N, do, device=DEV)
        ws = torch.empty(dp.dp_grad_sample_linear_workspace_bytes(N, T, di, do, dt), dtype=torch.uint8, device=DEV)
    else:
        N, ci, co, H = 256, 64, 128, 16
        a, b = torch.randn(N, ci, H, H, device=DEV).to(td), torch.randn(N, co, H, H, device=DEV).to(td)
        gW, gb = torch.empty(N, co, ci * 9, device=DEV), torch.empty(N, co, device=DEV)
        geom = (3, 3, 1, 1, 1, 1)
        ws = torch.empty(max(dp.dp_grad_sample_conv2d_workspace_bytes(N, ci, H, H, co, *geom), 4), dtype=torch.uint8,
                         device=DEV)
    sq = torch.empty(N, device=DEV)

    def call():
        if kind == "linear":
            dp.dp_grad_sample_linear(a, b, dt, N, T, di, do, 1.0, gW, gb, sq, None, ws)
        else:
            dp.dp_grad_sample_conv2d(a, b, dt, N, ci, H, H, co, H, H, *geom, 1, 1, 1, 1.0, gW, gb, sq, None, ws)

    def us():
        best = 1e9
        for _ in range(5):
            s, e = torch.cuda.Event(True), torch.cuda.Event(True)
            s.record()
            for _ in range(5):
                call()
            e.record()
            torch.cuda.synchronize()
            best = min(best, s.elapsed_time(e) * 200)
        return best

    call()
    ordinary = us()
    a.view(N, -1)[:, 77] = float("nan")
    worst = us()
    print("[case] ordinary %.1f us, every sample with a NaN %.1f us" % (ordinary, worst), file=sys.stderr, flush=True)
    assert worst <= 20 * ordinary
