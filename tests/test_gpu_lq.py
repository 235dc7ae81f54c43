"""GPU: the LQ-preconditioned gate SVD (batched path) on shapes at the edges of
its blocks and dispatch, against LAPACK and against the direct iteration (which
handles with a lowered sweep limit keep)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N, Q = 22, 10  # the gate acts on sites 10 and 11


def _site(rng, dl, dr):
    """Random right-orthonormal tensor (2, dl, dr) where 2 dr >= dl."""
    a = rng.standard_normal((max(dl, 2 * dr), dl)) + 1j * rng.standard_normal((max(dl, 2 * dr), dl))
    q = np.linalg.qr(a)[0].conj().T[:, :2 * dr]
    return np.ascontiguousarray(q.reshape(dl, 2, dr).transpose(1, 0, 2))


def _run(binding, D, u, sites, sweeps):
    m = binding.Mps(N, D, 1e-14, max_jacobi_sweeps=sweeps)
    m.set_fused_gates(False)
    for q, (b, lam) in enumerate(sites):
        m.import_site(Q + q, b, lam)
    m.apply_gate(Q, Q + 1, u)
    bl, _ = m.export_site(Q)
    br, lam = m.export_site(Q + 1)
    m.close()
    return bl, br, lam


# (D, dl, dm, dr, decades of lambda): side lengths around 64 rows, the 16-row
# blocks, the 128 / 256 / 512 / 1024 row lengths, tall and wide matrices, and
# ranks far below both sides (dm small)
@pytest.mark.parametrize("D,dl,dm,dr,decades", [
    (128, 12, 100, 128, 2),
    (128, 33, 40, 65, 3),
    (128, 64, 128, 64, 6),
    (128, 65, 128, 63, 2),
    (128, 128, 16, 128, 1),
    (128, 128, 128, 12, 2),
    (256, 129, 200, 128, 2),
    (256, 256, 256, 256, 6),
    (256, 72, 256, 200, 12),
    (512, 257, 300, 255, 2),
    (512, 100, 512, 512, 2),
    (512, 512, 64, 100, 2),
    (64, 64, 30, 16, 2),
    (64, 9, 40, 30, 1),
    # the rows of the larger half of lambda all parallel (negative decades)
    (128, 128, 24, 12, -1),
    (128, 60, 100, 70, -2),
])
def test_gate_svd_vs_lapack_and_direct(gpu_lib, D, dl, dm, dr, decades):
    from paper_2303_03681_amd import binding
    rng = np.random.default_rng([dl, dm, dr])
    lam = np.logspace(0, -abs(decades), dl)
    lam /= np.linalg.norm(lam)
    b0, b1 = _site(rng, dl, dm), _site(rng, dm, dr)
    if decades < 0:
        b0[:, :dl // 2] = b0[:, :1]
    lam_m = np.ones(dm) / np.sqrt(dm)
    u = np.linalg.qr(rng.standard_normal((4, 4)) + 1j * rng.standard_normal((4, 4)))[0]
    sites = [(b0, lam), (b1, lam_m)]
    theta = np.einsum("alm,bmr->ablr", b0, b1)
    C = np.einsum("cdab,ablr->cldr", u.reshape(2, 2, 2, 2), theta).reshape(2 * dl, 2 * dr)
    A = np.tile(lam, 2)[:, None] * C
    uu, s, vh = np.linalg.svd(A, full_matrices=False)
    k = max(1, min(D, int((s > 1e-14 * np.linalg.norm(s)).sum())))
    kept = np.linalg.norm(s[:k])
    Ak = (uu[:, :k] * s[:k]) @ vh[:k] / kept
    # round-off of the factorisations n 2^-53, over the gap of the cut for the subspace
    n = max(2 * dl, 2 * dr)
    eps = 16 * n * 2.0 ** -53
    gap = (s[k - 1] - (s[k] if k < len(s) else 0.0)) / s[0]
    tol = 1e-12 + eps / max(gap, eps)
    print(f"D={D} {2 * dl}x{2 * dr} rank bound {4 * dm}: k={k}, gap {gap:.1e}, tol {tol:.1e}", flush=True)
    for sweeps in (0, 59):  # preconditioned, direct
        bl, br, got = _run(binding, D, u, sites, sweeps)
        V = br.transpose(1, 0, 2).reshape(k, 2 * dr)
        P = np.tile(lam, 2)[:, None] * (bl.reshape(2 * dl, k) @ V)
        d_orth = np.abs(V @ V.conj().T - np.eye(k)).max()
        print(f"  sweeps limit {sweeps or 60}: |dlam| {np.abs(got - s[:k] / kept).max():.1e}, orthonormality "
              f"{d_orth:.1e}, |d A_k| {np.linalg.norm(P - Ak):.1e}", flush=True)
        assert got.shape == (k,) and bl.shape == (2, dl, k) and br.shape == (2, k, dr)
        assert np.abs(got - s[:k] / kept).max() <= 1e-12
        if s[k - 1] > 1e-10 * s[0]:
            assert d_orth <= 1e-12
        assert np.linalg.norm(P - Ak) <= tol


def test_budget_without_room_takes_the_direct_iteration(gpu_lib):
    """A budget that the direct iteration fits stays enough for a layer of gates."""
    from paper_2303_03681_amd import binding
    rng = np.random.default_rng(3)
    n, D = 16, 80
    gates = [(q, np.linalg.qr(rng.standard_normal((4, 4)) + 1j * rng.standard_normal((4, 4)))[0])
             for layer in range(8) for start in (0, 1) for q in range(start, n - 1, 2)]
    q0 = [q for q, _ in gates]
    u = np.zeros((len(gates), 16, 2))
    for i, (_, g) in enumerate(gates):
        u[i, :, 0], u[i, :, 1] = g.ravel().real, g.ravel().imag
    held = {}
    out = []
    for sweeps, budget in ((59, 0), (0, None), (0, 0)):
        # 4 bytes per gate of a batch for the 60th sweep's rotation counters
        m = binding.Mps(n, D, 1e-14, max_jacobi_sweeps=sweeps,
                        hbm_budget_bytes=held[59] + 4 * (n // 2) if budget is None else 0)
        m.set_fused_gates(False)
        m.apply_gates(q0, np.array(q0) + 1, u)
        held.setdefault(sweeps, m.device_bytes())
        out.append((m.bond_dims(), np.concatenate([m.export_site(q)[1] for q in range(n)])))
        m.close()
    for dims, lam in out[1:]:
        assert list(dims) == list(out[0][0])
        assert np.abs(lam - out[0][1]).max() <= 1e-9
