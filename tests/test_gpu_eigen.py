"""Eigen-solve of the refresh where its launch or its accuracy has an edge: matrices of up to 64 rows beside longer ones (one
launch, whose workgroups hold them in one group of 64 rows or two), and leading eigenvalues close to the line below which the
tridiagonal path declines."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import make_gpu_ctx
from oracle import tgrad_oracle as O
from paper_2501_02379_amd import synth, tgrad as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,ranks", [
    ((75, 24, 7), (18, 6, 2)), ((65, 64, 3), (20, 21, 2)), ((128, 16, 17), (9, 15, 16)), ((66, 63, 2), (5, 62, 1)),
    ((64, 48, 33), (63, 1, 32)), ((127, 2, 9), (11, 1, 8))])
def test_short_modes_beside_long_ones(shape, ranks):
    print("[case] eigen-solve", shape, ranks, flush=True)
    g = synth.small_case(shape, 31, outlier_frac=(1, 100))
    ctx = make_gpu_ctx(T, shape, ranks, 0, refresh_every=0)
    for _ in range(2):                             # the second refresh finds the first one's results in the work buffers
        ctx.tgrad_refresh_factors(T.to_device_grad(g))
        factors = [ctx.tgrad_get_state(T.STATE_FACTOR0 + n).astype(np.complex128) for n in range(len(shape))]
        for n, (U, r) in enumerate(zip(factors, ranks)):
            assert ctx.tgrad_get_state(T.STATE_EIG_INFO0 + n)[2] == 0, n
            gram = ctx.tgrad_get_state(T.STATE_GRAM0 + n)
            lam, V = np.linalg.eigh(gram)
            lam, V = lam[::-1], V[:, ::-1]
            top = V[np.abs(V).argmax(0), np.arange(V.shape[1])]
            V = V * (np.abs(top) / top)
            # both sides solve the same float64 matrix: backward errors of n 2^-53 |A| over the gap, and the factor's rounding
            gap = np.array([min(abs(lam[k] - lam[j]) for j in range(len(lam)) if j != k) for k in range(r)])
            bound = 2.0 ** -24 + 8 * shape[n] * 2.0 ** -53 * lam[0] / gap
            assert np.all(np.abs(U - V[:, :r]).max(0) <= 4 * bound), (n, np.abs(U - V[:, :r]).max(0), bound)
    ctx.tgrad_destroy()


@pytest.mark.parametrize("n", [16, 64, 100, 128])
def test_close_leading_eigenvalues(n):
    """Eigenvalues 1 and 1 - 4e-7 of the spectral radius: four times the line.  The shift of the inverse iteration is 3e-11 off at
    most, so the three solves leave (3e-11 / 4e-7)^3 < 1e-12 of the neighbour; errors of n 2^-53 over the gap are below 4e-8 on
    each side, the factor's rounding 6e-8: four times their sum."""
    print("[case] close pair", n, flush=True)
    rng = np.random.default_rng(n)
    q = [np.linalg.qr(rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n)))[0] for _ in range(2)]
    sv = np.concatenate(([1.0, 1.0 - 2e-7], 0.9 - 0.5 * np.arange(n - 2) / n))
    g = ((q[0] * sv) @ q[1].conj().T).astype(np.complex64)
    ctx = make_gpu_ctx(T, (n, n), (3, 3), 0, refresh_every=0)
    ctx.tgrad_refresh_factors(T.to_device_grad(g))
    for mode, x in enumerate((g, g.T)):
        assert ctx.tgrad_get_state(T.STATE_EIG_INFO0 + mode)[2] == 0, mode
        lam, V = np.linalg.eigh(x.astype(np.complex128) @ x.astype(np.complex128).conj().T)
        assert 2e-7 < (lam[-1] - lam[-2]) / lam[-1] < 8e-7
        V = V[:, ::-1][:, :3]
        top = V[np.abs(V).argmax(0), np.arange(3)]
        U = ctx.tgrad_get_state(T.STATE_FACTOR0 + mode)
        assert np.max(np.abs(U - V * (np.abs(top) / top))) < 4 * (8e-8 + 6e-8), mode
    ctx.tgrad_destroy()
