"""GPU: a cutoff of zero (only the bond cap truncates) keeps singular values
that are round-off.  Their vectors must not count a direction that is kept
already: the two-site matrix is reproduced to rounding all the same."""

import numpy as np
import pytest

from tests.test_gpu_fused_lq import _gate, _reference

pytestmark = pytest.mark.gpu


def _blocks(rng, dl, dm, dr):
    """Sites of block-sparse form, as particle number conservation gives them:
    every row of C~ has one element, many rows in each of dm columns."""
    b0 = np.zeros((2, dl, dm), complex)
    for s in range(2):
        b0[s, np.arange(dl), np.arange(dl) % dm] = rng.standard_normal(dl) + 1j * rng.standard_normal(dl)
    b1 = np.zeros((2, dm, dr), complex)
    b1[0, np.arange(dm), np.arange(dm)] = 1.0
    lam = np.logspace(0, -2, dl)
    return b0, b1, lam / np.linalg.norm(lam)


@pytest.mark.parametrize("cutoff", [0.0, 1e-30])
@pytest.mark.parametrize("fused,n,D,dl,dm,dr", [(True, 14, 128, 64, 20, 64), (True, 14, 128, 64, 9, 17),
                                                (True, 14, 128, 20, 7, 33), (False, 22, 128, 64, 20, 64),
                                                (False, 22, 128, 128, 24, 100), (False, 22, 256, 90, 70, 256)])
def test_round_off_directions(gpu_lib, fused, n, D, dl, dm, dr, cutoff):
    from paper_2303_03681_amd import binding
    b0, b1, lam = _blocks(np.random.default_rng([dl, dm, dr]), dl, dm, dr)
    s, _, kept, Ak = _reference(D, np.eye(4), b0, b1, lam)
    bl, br, got = _gate(binding, n, n // 2 - 1, D, np.eye(4), b0, b1, lam, 0, fused, cutoff)
    P = np.tile(lam, 2)[:, None] * (bl.reshape(2 * dl, -1) @ br.transpose(1, 0, 2).reshape(-1, 2 * dr))
    err = np.linalg.norm(P - Ak)
    print(f"fused {fused} {2 * dl}x{2 * dr} rank {dm}: k={len(got)}, |d A| {err:.1e}", flush=True)
    assert np.abs(got[:dm] - s[:dm] / kept).max() <= 1e-12
    assert err <= 1e-12 + 16 * max(2 * dl, 2 * dr) * 2.0 ** -53
