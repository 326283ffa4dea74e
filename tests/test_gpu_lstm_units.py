"""dp_lstm_backward over the numbers of units per lane group and of row pieces:
hidden sizes at the edges of both, at most one workgroup per CU and more."""
import numpy as np
import pytest

import oracle
from compare import assert_g12
from test_gpu_lstm import lstm_case, run_device, say

pytestmark = pytest.mark.gpu


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
