"""GPU: closing traces where the rule takes tiles -- every string on eight or nine sites,
with short K ranges and with split ones, 32- and 64-bit environments -- against
the dense statevector (sparse sums, which take pairs, are in test_gpu_gram_pairs)."""

import numpy as np
import pytest

from tests.test_gpu_env_merged import _state
from tests.test_gpu_gram_pairs import _values

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,sites,D", [(16, 8, 32), (16, 8, 100), (16, 8, 128), (18, 9, 16)])
def test_dense_sums(gpu_lib, n, sites, D):
    from paper_2303_03681_amd import binding
    rng = np.random.default_rng(D)
    m = _state(binding, n, D, rng)
    codes = np.zeros((4 ** sites, n), np.uint8)
    codes[:, 4:4 + sites] = np.array(np.unravel_index(np.arange(4 ** sites), (4,) * sites)).T
    plan = binding.PauliSum(codes, rng.standard_normal(len(codes)))
    pick = rng.choice(len(codes), 200, replace=False)
    ref = _values(m.to_statevector(), codes[pick])
    for prec, tol in (("c128", 1e-12), ("c64", 1e-6), ("split_f16", 1e-6)):  # a few ulps per transfer product
        m.set_timing(True)
        _, per = m.expect(plan, prec, per_term=True)
        t = m.timing()
        err = np.abs(per[pick] - ref).max()
        print(f"n={n} D={D} {prec}: {err:.1e}, close work {t['close_tile_flops'] / t['close_flops']:.2f} of needed",
              flush=True)
        assert err <= tol
    m.close()
