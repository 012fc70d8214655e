"""The last mode alone on 16-row units (ranks above 16, or above 32 in the mode before, matrices, slabs of fewer than four rows): steps
against the oracle at the edges of the units, of the size classes and of the lines to the kernels for other shapes."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import check_parity, make_gpu_ctx, run_both, run_both_bf16_weights
from oracle import tgrad_oracle as O
from paper_2501_02379_amd import synth, tgrad as T

pytestmark = pytest.mark.gpu

# shape, ranks, share of entries in the support
SHAPES = [
    ((5, 3, 2), (3, 2, 1), 0.1),                        # shortest rows, one unit of 15
    ((6, 5, 3, 3), (3, 3, 2, 2), 0.5),                  # odd rows, an odd number of elements in the last unit
    ((5, 3, 16), (3, 2, 15), 0.02),                     # one quad of elements, two column tiles
    ((7, 3, 17), (3, 2, 16), 1.0),                      # two quads; everything in the support (more than 64 entries per 32 rows)
    ((31, 24), (31, 10), 0.02),                         # a matrix (its core would be diagonal): last class of three pieces
    ((33, 25), (33, 17), 0.3),                          # ... and the first of five; three column tiles
    ((7, 11, 40), (3, 4, 20), 0.5),
    ((7, 11, 41), (3, 4, 32), 0.02),                    # seven pieces, four column tiles
    ((6, 13, 56), (3, 5, 25), 0.02),
    ((6, 13, 57), (3, 5, 17), 0.05),                    # nine pieces
    ((5, 9, 69), (3, 4, 24), 0.02), ((5, 9, 72), (3, 4, 32), 0.2),
    ((5, 9, 73), (3, 4, 18), 0.02),                     # longer rows: the 32 x 32 kernels
    ((33, 31, 17, 33), (4, 5, 6, 17), 0.01),            # workgroups of 4 wavefronts, a unit each; the last of 15 rows and an odd count
    ((40, 30, 40, 24), (4, 5, 34, 9), 0.01),            # rank 9 of many rows
    ((40, 30, 40, 12), (4, 5, 34, 8), 0.01),            # rank 8 of many rows: the update of the 32 x 32 kernels
    ((20, 20, 40, 13), (4, 5, 34, 6), 0.05),            # 16000 rows: a wavefront for every unit
    ((64, 60, 51, 6), (4, 5, 34, 3), 0.05),             # 195840 short rows: the 32 x 32 kernels
    ((64, 61, 51, 5), (4, 5, 34, 2), 0.05),             # 199104: several short units per wavefront
]

# The same where every wavefront takes more than three units: both sets of registers, each of them requested again, and support
# ranges, rows of z and LDS slices handed on.  256 compute units hold what LDS has room for: 3 workgroups of 4 wavefronts at rows
# of 39 and rank 20 (4 with bf16 gradients), 2 (3) at 55 and 17, one of 8 (2 of 4) from 69 on.  More than 64 entries of the
# support in every 32 rows; the last unit has 3, 13, 13 and 13 rows, an odd number of elements where rows are odd.
LONG = [((59, 59, 59, 39), (4, 5, 6, 20), 0.1), ((53, 53, 53, 55), (4, 5, 6, 17), 0.06), ((47, 47, 45, 69), (4, 5, 6, 24), 0.05),
        ((47, 47, 45, 72), (4, 5, 6, 32), 0.05)]


def _weights(shape, seed):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * 0.02


@pytest.mark.parametrize("dt", ["c64", "cbf16"])
@pytest.mark.parametrize("shape,ranks,share", SHAPES)
def test_rows(shape, ranks, share, dt):
    print("[case] rows", shape, ranks, share, dt, flush=True)
    grads = [synth.small_case(shape, 600 + t, outlier_frac=(1, 100), dtype=dt) for t in range(4)]
    W0 = _weights(shape, 8).astype(np.complex64)
    info = run_both(T, shape, ranks, int(np.ceil(share * np.prod(shape))), grads, W0, refresh_every=3, lr=2e-3, weight_decay=0.01,
                    grad_dtype=T.TGRAD_CBF16 if dt == "cbf16" else T.TGRAD_C64)
    assert all(info["omega_equal"])
    check_parity(info, W0)


@pytest.mark.parametrize("shape,ranks,share", [SHAPES[0], SHAPES[1], SHAPES[3], SHAPES[5], SHAPES[8], SHAPES[11], SHAPES[13]])
def test_rows_bf16_weights(shape, ranks, share):
    """Four-element pieces of W (bounds as in test_bf16_weights_single_steps)."""
    print("[case] rows, bf16 weights", shape, ranks, share, flush=True)
    grads = [synth.small_case(shape, 700 + t, outlier_frac=(1, 100)) for t in range(3)]
    info = run_both_bf16_weights(T, shape, ranks, int(np.ceil(share * np.prod(shape))), grads,
                                 O.complex_to_bf16_pairs(_weights(shape, 9)), resync=True, refresh_every=3, lr=2e-3, weight_decay=0.01)
    for worst, frac in info["stats"]:
        assert worst <= 1
        assert frac <= max(5e-3, 2.0 / (2 * int(np.prod(shape))))


@pytest.mark.parametrize("dt", ["c64", "cbf16"])
@pytest.mark.parametrize("shape,ranks,share", LONG)
def test_rows_many_units(shape, ranks, share, dt):
    print("[case] rows, many units", shape, ranks, dt, flush=True)
    grads = [synth.small_case(shape, 610 + t, outlier_frac=(1, 100), dtype=dt) for t in range(2)]
    W0 = _weights(shape, 11).astype(np.complex64)
    info = run_both(T, shape, ranks, int(np.ceil(share * np.prod(shape))), grads, W0, refresh_every=3, lr=2e-3, weight_decay=0.01,
                    grad_dtype=T.TGRAD_CBF16 if dt == "cbf16" else T.TGRAD_C64)
    assert all(info["omega_equal"])
    check_parity(info, W0)


@pytest.mark.parametrize("shape,ranks,share", LONG)
def test_rows_many_units_bf16_weights(shape, ranks, share):
    print("[case] rows, many units, bf16 weights", shape, ranks, flush=True)
    grads = [synth.small_case(shape, 710 + t, outlier_frac=(1, 100)) for t in range(2)]
    info = run_both_bf16_weights(T, shape, ranks, int(np.ceil(share * np.prod(shape))), grads,
                                 O.complex_to_bf16_pairs(_weights(shape, 12)), resync=True, refresh_every=3, lr=2e-3, weight_decay=0.01)
    for worst, frac in info["stats"]:
        assert worst <= 1 and frac <= 5e-3


@pytest.mark.parametrize("order", [T.TGRAD_ORDER_LR_US, T.TGRAD_ORDER_SUM])
def test_rows_in_the_other_orders(order):
    """The low-rank part sees the full gradient: nothing is removed, and the sparse values are gathered elsewhere."""
    shape, ranks = (7, 11, 40), (3, 4, 20)
    print("[case] rows, order", order, flush=True)
    grads = [synth.small_case(shape, 800 + t, outlier_frac=(1, 100)) for t in range(3)]
    W0 = _weights(shape, 10).astype(np.complex64)
    info = run_both(T, shape, ranks, 120, grads, W0, refresh_every=3, lr=2e-3, order=order)
    assert all(info["omega_equal"])
    check_parity(info, W0)


def _float32_products(x, c):
    """Rows of x times c (complex) by chains of float32 multiply-adds, one rounding each."""
    parts = []
    for a, b in (((1, c.real), (-1, c.imag)), ((1, c.imag), (1, c.real))):
        acc = np.zeros((x.shape[0], c.shape[1]), np.float32)
        for k in range(x.shape[1]):
            for (sign, f), v in ((a, x[:, k].real), (b, x[:, k].imag)):
                acc = (acc + sign * v.astype(np.float64)[:, None] * f[k].astype(np.float64)).astype(np.float32)
        parts.append(acc)
    return parts[0] + 1j * parts[1]


@pytest.mark.parametrize("K,r", [(2, 1), (3, 1), (4, 1), (4, 2), (5, 2), (3, 3), (8, 2), (8, 4), (16, 3), (16, 16), (17, 9),
                                 (20, 20), (24, 18), (33, 32), (72, 20)])
def test_no_further_from_64_bits_than_float32_multiply_adds(K, r):
    """Both products of the last mode alone: modes 1 and 2 are left as they are (identity factors, whose products are exact), the
    update divides by 1 (V = 0, eps = 1, no gradient) and starts from zero weights.  3 %: three times what the error of some
    8000 rounded numbers scatters, and the order of a sum moves less."""
    print("[case] rows, error", K, r, flush=True)
    shape, ranks = (32, 64, K), (32, 64, r)
    rng = np.random.default_rng(100 * K + r)
    g, m = ((rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64) for s in (shape, ranks))
    U = np.linalg.qr(rng.standard_normal((K, r)) + 1j * rng.standard_normal((K, r)))[0].astype(np.complex64)

    def step(grad, core_m):
        ctx = make_gpu_ctx(T, shape, ranks, 0, lr=1.0, beta1=0.5, beta2=0.5, eps=1.0, refresh_every=0)
        ctx.tgrad_set_state(T.STATE_STEP, 1000)
        ctx.tgrad_set_state(T.STATE_INDICES, np.zeros(0))
        for n, u in enumerate((np.eye(32), np.eye(64), U)):
            ctx.tgrad_set_state(T.STATE_FACTOR0 + n, u)
        ctx.tgrad_set_state(T.STATE_CORE_M, core_m)
        w = T.to_device_weight(np.zeros(shape, np.complex64))
        ctx.tgrad_step(w, T.to_device_grad(grad))
        core = ctx.tgrad_get_state(T.STATE_CORE_G)
        ctx.tgrad_destroy()
        return core, T.weight_to_host(w)

    def error(got, x, c):
        want = x.astype(np.complex128) @ c.astype(np.complex128)
        return np.linalg.norm(got.reshape(want.shape) - want) / np.linalg.norm(want)

    x = g.reshape(-1, K)
    assert error(step(g, np.zeros(ranks))[0], x, U.conj()) <= 1.03 * error(_float32_products(x, U.conj()), x, U.conj())
    x = (np.float32(-0.5) * m).reshape(-1, r)              # what the core's half of M is expanded from
    assert error(step(np.zeros(shape, np.complex64), m)[1], x, U.T) <= 1.03 * error(_float32_products(x, U.T), x, U.T)
