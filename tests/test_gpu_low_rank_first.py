"""Low rank first: the expansions that the update and the compressed gradient have both, in one launch or in two."""
import numpy as np
import pytest

from paper_2501_02379_amd import synth
from paper_2501_02379_amd import tgrad as T
from helpers import check_parity, run_both

pytestmark = pytest.mark.gpu

# shape, ranks, launches of residual kernels in a step: those of mode 1, of the modes that only this part expands, the gather
CASES = [
    ((40, 40, 8, 8), (17, 3, 4, 3), 3),              # pairs of columns
    ((40, 30, 7, 9), (17, 11, 3, 3), 3),             # an odd number of columns: the second of the two at an odd place
    ((20, 12, 10, 8, 5), (17, 5, 4, 3, 3), 3),       # two such expansions, each into the other half of the room
    ((20, 18, 24, 80), (17, 5, 7, 20), 2),           # last mode alone: modes 2 and 3 for both
    ((18, 6, 5, 4), (18, 6, 5, 4), 4),               # no: the two do not fit the residual's room
    ((34, 40, 48, 40), (17, 5, 40, 40), 4),          # no: 54400 columns
]


@pytest.mark.parametrize("shape,ranks,residual", CASES)
def test_expansions_of_both_parts(shape, ranks, residual):
    print("[case]", shape, ranks, flush=True)
    rng = np.random.default_rng(31)
    grads = [synth.small_case(shape, 900 + t, outlier_frac=(1, 100)) for t in range(3)]
    W0 = ((rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * 0.02).astype(np.complex64)
    k = int(np.prod(shape)) // 100 + 3
    info = run_both(T, shape, ranks, k, grads, W0, refresh_every=4, lr=2e-3, lam=0.7, alpha=1.2, order=T.TGRAD_ORDER_LR_US)
    assert all(info["omega_equal"])
    check_parity(info, W0)
    ctx = info["ctx"]
    ctx.tgrad_set_profiling(True)
    ctx.tgrad_step(T.to_device_weight(W0), T.to_device_grad(grads[0]))
    times = ctx.tgrad_get_kernel_times()
    assert times["residual"]["launches"] == residual and times["core"]["launches"] == 1
    ctx.tgrad_destroy()
