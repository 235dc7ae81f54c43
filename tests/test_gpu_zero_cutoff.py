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


# Algorithm 1 on C~ itself: small matrices, and larger ones under a lowered sweep limit
@pytest.mark.parametrize("cutoff", [0.0, 1e-30])
@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("dl,dm,dr,sweeps", [(16, 5, 16, 0), (4, 3, 30, 0), (64, 9, 17, 59), (64, 20, 64, 59)])
def test_round_off_directions_direct(gpu_lib, fused, dl, dm, dr, sweeps, cutoff):
    from paper_2303_03681_amd import binding
    b0, b1, lam = _blocks(np.random.default_rng([dl, dm, dr]), dl, dm, dr)
    s, _, kept, Ak = _reference(128, np.eye(4), b0, b1, lam)
    bl, br, got = _gate(binding, 14, 6, 128, np.eye(4), b0, b1, lam, sweeps, fused, cutoff)
    P = np.tile(lam, 2)[:, None] * (bl.reshape(2 * dl, -1) @ br.transpose(1, 0, 2).reshape(-1, 2 * dr))
    err = np.linalg.norm(P - Ak)
    print(f"fused {fused} {2 * dl}x{2 * dr} rank {dm}: k={len(got)}, |d A| {err:.1e}", flush=True)
    assert np.abs(got[:dm] - s[:dm] / kept).max() <= 1e-12
    assert err <= 1e-12 + 16 * max(2 * dl, 2 * dr) * 2.0 ** -53


@pytest.mark.parametrize("fused", [True, False])
def test_uccsd_chain_keeps_its_state(gpu_lib, fused):
    """A window of the UCCSD chain on 10 qubits at the full bond dimension 32:
    nothing but round-off is truncated, whatever the cutoff."""
    from oracle import dense_apply_gates, dense_product_state
    from paper_2303_03681_amd import binding
    from workloads import fuse_gates, pack_gates
    from workloads.circuits import uccsd_gates, uccsd_n_params
    n = 10
    bits = np.array([1] * 5 + [0] * 5, np.uint8)
    theta = np.random.default_rng(8).uniform(-0.1, 0.1, size=uccsd_n_params(n, 5, window=5))
    gates = fuse_gates(uccsd_gates(n, 5, theta, window=5), n)[:300]
    psi = np.asarray(dense_apply_gates(dense_product_state(bits), gates)).reshape(-1)
    m = binding.Mps(n, 32, 0.0, bits=bits)
    m.set_fused_gates(fused)
    m.apply_gates(*pack_gates(gates))
    v = m.to_statevector()
    m.canonicalize()
    w = m.to_statevector()
    m.close()
    err = 1.0 - abs(np.vdot(psi, v)) / np.linalg.norm(v)
    print(f"fused {fused}: 1 - overlap {err:.1e}, norm - 1 {np.linalg.norm(v) - 1:.1e}", flush=True)
    # 300 gates, each within its tolerance above of the exact product; the overlap is quadratic in them
    assert err <= 1e-12
    assert abs(np.linalg.norm(v) - 1.0) <= 300 * 2e-12
    assert 1.0 - abs(np.vdot(psi, w)) / np.linalg.norm(w) <= 1e-12  # in exact canonical form too
