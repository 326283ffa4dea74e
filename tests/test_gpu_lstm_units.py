"""dp_lstm_backward over the numbers of units per lane group and of row pieces:
hidden sizes at the edges of both, at most one workgroup per CU and more."""
import numpy as np
import pytest
import torch

import oracle
from compare import assert_g12
from paper_2109_12298_amd import binding as dp
from test_gpu_lstm import lstm_case, run_device, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("N", [3, 260])
@pytest.mark.parametrize("H", [2, 7, 8, 9, 16, 17, 24, 31, 32, 33, 47, 48, 49, 63, 64, 65, 72, 81, 95, 96, 97, 105, 127])
def test_units_and_pieces(N, H):
    T = 8                                    # a ring of six steps and two more
    say("lstm units", N, H)
    few = lstm_case(min(N, 4), T, 3, H, H % 2 == 0, True, seed=H)
    rep = -(-N // few[0].shape[0])
    case = [None if a is None else a if k == 2 else np.tile(a, (rep,) + (1,) * (a.ndim - 1))[:N]
            for k, a in enumerate(few)]
    got = run_device(*case)
    ref = oracle.lstm_backward(few[0], few[1], few[2], dh_out=few[3], dh_last=few[4])
    for n in range(N):
        # sums of 4H products and 8 chained steps: 1e-5 is fifty times what they show
        assert_g12(got[n], ref[n % len(ref)], 1e-5, "delta n=%d" % n)


@pytest.mark.parametrize("N,H", [(3, 20), (3, 100), (300, 96)])
def test_cell_gradient_is_one_rounding_per_step(N, H):
    """dc_t = dc_{t+1} f_{t+1} + dh_t o (1 - tanh^2 c_t), the chain over all steps, rounds once per step: with
    o = 1, c = 0 and no recurrent weights dh passes through exactly, and delta_i = dc / 4 at g = 1, i = 1 / 2."""
    T = 40
    say("lstm cell gradient", N, H)
    g = torch.Generator().manual_seed(31)
    gates = torch.ones(N, T, 4 * H)
    gates[:, :, :H] = 0.5
    gates[:, :, H:2 * H] = torch.rand(N, T, H, generator=g)
    dh = torch.randn(N, T, H, generator=g)
    delta = torch.full((N, T, 4 * H), 7.0, device=DEV)
    dp.dp_lstm_backward(gates.to(DEV), torch.zeros(N, T, H, device=DEV), torch.zeros(4 * H, H, device=DEV), dh.to(DEV), None,
                        N, T, H, delta, None)
    got = delta.cpu().numpy()[:, :, :H]
    f, h = gates[:, :, H:2 * H].numpy().astype(np.longdouble), dh.numpy().astype(np.longdouble)
    dc = np.zeros((N, H), np.float32)
    for t in range(T - 1, -1, -1):
        dc = (h[:, t] + (dc.astype(np.longdouble) * f[:, t + 1] if t + 1 < T else 0)).astype(np.float32)
        np.testing.assert_array_equal(got[:, t], dc / 4)
