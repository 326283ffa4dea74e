"""dp_grad_sample_groupnorm at the edges of its plane sizes (lanes per channel,
loads in flight, tails), alignments and the size from which it reads past the caches."""
import sys

import numpy as np
import pytest
import torch

from paper_2109_12298_amd import binding as dp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("N,C,P", [(2, 3, 1), (3, 17, 3), (2, 16, 64), (2, 18, 65), (1, 5, 255), (2, 4, 257), (1, 4, 260),
                                   (2, 3, 511), (2, 3, 515), (2, 3, 516), (1, 2, 1025), (1, 3, 2051), (3, 2, 4096),
                                   (200, 64, 1024)])
def test_planes(N, C, P, shift, dtype):
    print("[case] groupnorm", N, C, P, shift, dtype, file=sys.stderr, flush=True)
    g = torch.Generator(device=DEV).manual_seed(P)
    bx, bb = (torch.randn(N * C * P + shift, generator=g, device=DEV).to(dtype)[shift:] for _ in range(2))
    gg, gb, sq = torch.full((N, C), 7.0, device=DEV), torch.full((N, C), 7.0, device=DEV), torch.zeros(N, device=DEV)
    ws = torch.empty(max(dp.dp_grad_sample_groupnorm_workspace_bytes(N, C, P), 4), dtype=torch.uint8, device=DEV)
    dp.dp_grad_sample_groupnorm(bx, bb, dp.dtype_of(bx), N, C, P, 1.5, gg, gb, sq, None, ws)
    torch.cuda.synchronize()
    x, b = bx.reshape(N, C, P).double(), bb.reshape(N, C, P).double()
    bound = (P + 8) * 2.0 ** -24 * 1.5       # P products and sums, each rounded once
    assert ((gg - 1.5 * (x * b).sum(2)).abs() <= bound * (x * b).abs().sum(2)).all()
    assert ((gb - 1.5 * b.sum(2)).abs() <= bound * b.abs().sum(2)).all()
    ref = (gg.double() ** 2 + gb.double() ** 2).sum(1)
    np.testing.assert_allclose(sq.double().cpu().numpy(), ref.cpu().numpy(), rtol=1e-5)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,C,P", [(2, 3, 66), (2, 17, 127), (2, 16, 128), (2, 3, 130), (2, 3, 544), (2, 3, 1026), (2, 3, 1284),
                                   (300, 64, 1088), (500, 64, 576)])
def test_tails(N, C, P, dtype):
    """What a step of the loop leaves over, in planes read through and (the largest) past the caches, and the
    planes read by single elements."""
    test_planes(N, C, P, 0, dtype)
    test_planes(N, C, P, 1, dtype)
