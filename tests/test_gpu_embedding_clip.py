"""Clipped sum of CSR embedding gradients: the one-launch scan against the
laid-out index, bit for bit, and against 64-bit sums, at the edges of chunks of
samples, of the ids a workgroup owns and of the range the scan covers.

A cap beyond 256 rows per sample takes the laid-out index, so the same rows
are given once under each cap.  Bound per element against 64 bits: a chain of
up to N products and sums, each rounded relative to sum |c x| at most, and the
factor itself (a division and a sum): (N + 4) * 2^-24 * sum |c x|.
"""
import sys

import numpy as np
import pytest
import torch

from paper_2109_12298_amd import binding as dp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def clipped(rp, uq, rows, norm, cap, N, V, D, shift):
    """The clipped sum with room for cap rows, and the status flags."""
    u = torch.full((cap,), -1, dtype=torch.int64, device=DEV)
    r = torch.full((cap * D + shift,), float("nan"), device=DEV)
    k = min(cap, len(uq))
    u[:k] = torch.from_numpy(uq[:k]).to(DEV)
    r[shift:shift + k * D] = torch.from_numpy(rows[:k].reshape(-1)).to(DEV)
    out = torch.full((V * D + 64,), 7.0, device=DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    ws = torch.empty(dp.dp_clip_accumulate_embedding_workspace_bytes(N, V), dtype=torch.uint8, device=DEV)
    dp.dp_clip_accumulate_embedding(torch.from_numpy(rp).to(DEV), u, r[shift:], cap, torch.from_numpy(norm).to(DEV),
                                    1.0, N, V, D, out, status, ws)
    torch.cuda.synchronize()
    assert (out[V * D:] == 7).all(), "wrote outside sum"
    return out[:V * D].reshape(V, D).cpu().numpy(), int(status.item())


CASES = [  # N, V, D, rows per sample at most
    (1, 1, 4, 1), (3, 50, 5, 9), (63, 255, 100, 130), (64, 256, 36, 200), (65, 257, 300, 66), (130, 32768, 8, 129),
    (70, 32769, 12, 256), (2, 65536, 260, 250), (129, 1000, 1, 256), (5, 65537, 4, 40),
]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("bad", [False, True])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_scan_against_index(case, bad, shift):
    N, V, D, most = case
    print("[case]", case, "bad", bad, "shift", shift, file=sys.stderr, flush=True)
    rng = np.random.default_rng([N, V, D])
    ids, rp = [], [0]
    for n in range(N):
        u = 0 if n == 1 else int(rng.integers(1, min(most, V) + 1))      # sample 1 holds none
        v = np.concatenate([[V - 1], rng.choice(V - 1, u - 1, replace=False)]) if u else np.zeros(0)
        ids.append(v.astype(np.int64))                                   # in no order, the last id in every sample
        rp.append(rp[-1] + u)
    uq, rp = np.concatenate(ids), np.array(rp, dtype=np.int64)
    if bad:
        uq[len(uq) // 2] = V if N % 2 else -1
    rows = rng.standard_normal((len(uq), D), dtype=np.float32)
    norm = (rng.random(N, dtype=np.float32) * 3).astype(np.float32)
    norm[N // 2] = -1.0                                                  # a padding row
    few, many = len(uq), 256 * N + 1
    got, st = clipped(rp, uq, rows, norm, few, N, V, D, shift)
    ref, st_ref = clipped(rp, uq, rows, norm, many, N, V, D, shift)
    assert few <= 256 * N
    assert st == st_ref == (dp.DP_FLAG_BAD_INDEX if bad else 0)
    assert (got.view(np.int32) == ref.view(np.int32)).all()
    c = np.where(norm < 0, 0.0, np.minimum(1.0, 1.0 / (norm.astype(np.float64) + 1e-6)))
    want, mag = np.zeros((V, D)), np.zeros((V, D))
    for n in range(N):
        for k in range(rp[n], rp[n + 1]):
            if 0 <= uq[k] < V:
                want[uq[k]] += c[n] * rows[k]
                mag[uq[k]] += c[n] * abs(rows[k])
    assert (abs(got - want) <= (N + 4) * 2.0 ** -24 * mag).all()


def test_rows_beyond_cap_are_left_out():
    rp, uq = np.array([0, 3, 5], dtype=np.int64), np.array([0, 2, 3, 1, 2], dtype=np.int64)
    rows = np.arange(20, dtype=np.float32).reshape(5, 4)
    got, st = clipped(rp, uq, rows, np.full(2, 0.5, np.float32), 4, 2, 4, 4, 0)
    assert st == dp.DP_FLAG_CAP
    assert (got == rows[[0, 3, 1, 2]]).all()
