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
    lowest parts are subnormal in bf16."""
    N, T, di, do = 1, 32, 64, 128
    g = torch.Generator().manual_seed(6)
    A, B = torch.randn(N, T, di, generator=g), torch.randn(N, T, do, generator=g) * 2.0 ** -105
    say("linear small magnitudes")
    gW, _, _ = linear(A, B, 0, scale=1.0)
    ref = np.einsum("nti,ntj->nij", B.double().numpy(), A.double().numpy())
    mag = np.einsum("nti,ntj->nij", abs(B.double().numpy()), abs(A.double().numpy()))
    assert (abs(gW - ref) <= (T + 8) * 2.0 ** -24 * mag + 2.0 ** -140).all()
