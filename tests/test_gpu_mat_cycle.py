"""The materialised cost read once per cycle (k_mat_cycle, k_mat_cols): lanes large
enough for it at every column layout (256 and 512 threads, 4 to 32 columns each),
with row and column counts off the 64-row items, ragged lanes whose sizes fall
below the window's, zero masses, and the modes that share the launches, against
the float64 oracle. The cost is float32, so potentials and residuals keep the bars
of the float32 parity tests."""

import numpy as np
import pytest

from paper_2607_24741_amd import workloads as wl
from tests.gpu_support import FP32_BAND, compare, log, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _window(sizes, n_max, m_max, seed, d=40):
    rng = np.random.default_rng([seed, n_max, m_max])
    W = len(sizes)
    X = np.full((W, n_max, d), np.nan, np.float32)
    Y = np.full((W, m_max, d), np.nan, np.float32)
    A = np.full((W, n_max), np.nan, np.float32)
    B = np.full((W, m_max), np.nan, np.float32)
    N = np.array([s[0] for s in sizes], np.int32)
    M = np.array([s[1] for s in sizes], np.int32)
    for t in range(W):
        X[t, :N[t]] = rng.standard_normal((N[t], d)) / np.sqrt(d)
        Y[t, :M[t]] = rng.standard_normal((M[t], d)) / np.sqrt(d) + 0.05
        a, b = rng.gamma(1.0, size=N[t]) + 1e-3, rng.gamma(1.0, size=M[t]) + 1e-3
        if N[t] > 3 and M[t] > 3:
            a[N[t] // 2] = 0.0
            b[M[t] // 3] = 0.0
        A[t, :N[t]], B[t, :M[t]] = a / a.sum(), b / b.sum()
    return wl.Workload(name="mat", X=X, Y=Y, a=A, b=B, eps=np.full(W, 0.06, np.float32), n=N, m=M,
                       tol=1e-4, max_iter=12)


@pytest.mark.parametrize("n,m", [(12300, 1024), (6310, 2000), (3601, 3500), (1601, 8000), (1025, 12290)])
def test_every_column_layout_against_the_oracle(n, m):
    # one full lane and a ragged one
    w = _window([(n, m), (n // 3 + 5, m - 131)], n, m, seed=3)
    log(f"[case] one pass n={n} m={m}")
    got = run_gpu(w, 1e-9, max_iter=5)
    ref = run_oracle(w, 1e-9, max_iter=5)
    rep = compare(w, got, ref, 1e-9, max_iter=5, band=FP32_BAND)
    assert rep["max_pot_err"] <= 3e-5


def test_decisions_modes_and_width():
    w = _window([(3600, 3500), (2000, 3001), (3599, 64), (1, 3500)], 3600, 3500, seed=4)
    log("[case] one pass: decisions, modes, width")
    got = run_gpu(w, 3e-3, max_iter=60)
    ref = run_oracle(w, 3e-3, max_iter=60)
    compare(w, got, ref, 3e-3, max_iter=60, band=FP32_BAND)
    # a lane's bits depend neither on its co-lanes nor on the mode it runs in
    one = wl.Workload(name="one", X=w.X[1:2], Y=w.Y[1:2], a=w.a[1:2], b=w.b[1:2], eps=w.eps[1:2],
                      n=w.n[1:2], m=w.m[1:2], tol=3e-3, max_iter=60)
    alone = run_gpu(one, 3e-3, max_iter=60)
    logical = run_gpu(w, 3e-3, max_iter=60, mode="logical")
    shadow = run_gpu(w, 3e-3, max_iter=60, flags=1)
    for k in ("f", "g", "residual", "depth"):
        assert np.array_equal(alone[k][0], got[k][1]), k
        assert np.array_equal(logical[k], got[k]), k
        assert np.array_equal(shadow[k], got[k]), k
    assert shadow["stats"].missed_ready == 0 and shadow["stats"].screen_discrepancy < 1e-6
    guard = run_gpu(w, 3e-3, max_iter=60, flags=64)
    assert np.abs(guard["depth"] - got["depth"]).max() <= 1
