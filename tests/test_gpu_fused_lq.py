"""GPU: the fused gate's SVD at the edges of its register layouts and rules --
preconditioned and, with a lowered sweep limit, on C~ itself -- against LAPACK;
and the orthonormality of V^+ on spectra over twelve decades, fused and batched."""

import numpy as np
import pytest

from tests.test_gpu_lq import _site

pytestmark = pytest.mark.gpu

# both outer bonds of the gate on sites 6 and 7 of 14 have capacity 64 (the
# fused limit), the bond between them min(D, 128)
N, Q = 14, 6


def _gate(binding, n, q, D, u, b0, b1, lam, sweeps, fused, cutoff=1e-14):
    m = binding.Mps(n, D, cutoff, max_jacobi_sweeps=sweeps)
    m.set_fused_gates(fused)
    m.import_site(q, b0, lam)
    m.import_site(q + 1, b1, np.ones(b0.shape[2]) / np.sqrt(b0.shape[2]))
    m.apply_gate(q, q + 1, u)
    bl, _ = m.export_site(q)
    br, got = m.export_site(q + 1)
    m.close()
    return bl, br, got


def _reference(D, u, b0, b1, lam, cutoff=1e-14):
    theta = np.tensordot(b0, b1, ([2], [1]))  # [a][l][b][r]
    c = np.tensordot(u.reshape(2, 2, 2, 2), theta, ([2, 3], [0, 2])).transpose(0, 2, 1, 3)  # [c][l][d][r]
    A = np.tile(lam, 2)[:, None] * c.reshape(2 * len(lam), -1)
    uu, s, vh = np.linalg.svd(A, full_matrices=False)
    k = max(1, min(D, int((s > cutoff * np.linalg.norm(s)).sum())))
    kept = np.linalg.norm(s[:k])
    return s, k, kept, (uu[:, :k] * s[:k]) @ vh[:k] / kept


def _inputs(rng, dl, dm, dr, decades):
    lam = np.logspace(0, -abs(decades), dl)
    lam /= np.linalg.norm(lam)
    b0, b1 = _site(rng, dl, dm), _site(rng, dm, dr)
    if decades < 0:  # the rows of the larger half of lambda all parallel
        b0[:, :dl // 2] = b0[:, :1]
    u = np.linalg.qr(rng.standard_normal((4, 4)) + 1j * rng.standard_normal((4, 4)))[0]
    return u, b0, b1, lam


# (D, dl, dm, dr, decades of lambda) of the 2 dl x 2 dr matrix: sides around 32,
# 64 and 128 in all three layouts, square, wide, tall (also with more than 64
# columns, and tall enough to be factorised at fewer than 32 x 32 elements),
# kept ranks 64 and 65, ranks far below both sides
@pytest.mark.parametrize("D,dl,dm,dr,decades", [
    (128, 16, 20, 16, 2),
    (128, 16, 20, 17, 2),
    (128, 17, 20, 16, 3),
    (128, 31, 60, 32, 2),
    (128, 32, 40, 32, 6),
    (128, 32, 50, 33, 2),
    (128, 33, 50, 32, 2),
    (128, 33, 64, 33, 3),
    (128, 64, 128, 64, 6),
    (65, 64, 65, 64, 1),
    (64, 64, 64, 64, 1),
    (128, 64, 16, 64, 1),
    (128, 64, 100, 33, 2),
    (128, 45, 100, 64, 2),
    (128, 5, 40, 64, 1),
    (128, 30, 20, 7, 1),
    (128, 64, 20, 3, 1),
    (128, 64, 2, 1, 1),
    (128, 40, 5, 41, 2),
    (128, 64, 24, 12, -1),
    (128, 60, 100, 50, -2),
    (128, 48, 128, 56, 12),
])
def test_fused_gate_vs_lapack(gpu_lib, D, dl, dm, dr, decades):
    from paper_2303_03681_amd import binding
    u, b0, b1, lam = _inputs(np.random.default_rng([dl, dm, dr]), dl, dm, dr, decades)
    s, k, kept, Ak = _reference(D, u, b0, b1, lam)
    # round-off of the factorisations n 2^-53, over the gap of the cut for the subspace
    eps = 16 * max(2 * dl, 2 * dr) * 2.0 ** -53
    gap = (s[k - 1] - (s[k] if k < len(s) else 0.0)) / s[0]
    tol = 1e-12 + eps / max(gap, eps)
    print(f"D={D} {2 * dl}x{2 * dr} rank bound {4 * dm}: k={k}, gap {gap:.1e}, tol {tol:.1e}", flush=True)
    for sweeps in (0, 59):  # preconditioned, direct
        bl, br, got = _gate(binding, N, Q, D, u, b0, b1, lam, sweeps, True)
        V = br.transpose(1, 0, 2).reshape(-1, 2 * dr)
        P = np.tile(lam, 2)[:, None] * (bl.reshape(2 * dl, -1) @ V)
        assert got.shape == (k,) and bl.shape == (2, dl, k) and br.shape == (2, k, dr)
        d_orth = np.abs(V @ V.conj().T - np.eye(k)).max()
        print(f"  sweeps limit {sweeps or 60}: |dlam| {np.abs(got - s[:k] / kept).max():.1e}, orthonormality "
              f"{d_orth:.1e}, |d A_k| {np.linalg.norm(P - Ak):.1e}", flush=True)
        assert np.abs(got - s[:k] / kept).max() <= 1e-12
        if sweeps == 0 or s[k - 1] > 1e-10 * s[0]:
            assert d_orth <= 1e-12
        assert np.linalg.norm(P - Ak) <= tol


# V^+ of the preconditioned gate, fused and batched, is orthonormal whatever
# the grading: Z Q1 is so to eps sigma_1 / sigma_k only, the last pass mends it
@pytest.mark.parametrize("fused,n,D,dl,dm,dr", [(True, 14, 128, 64, 128, 64), (True, 14, 128, 64, 100, 20),
                                                (False, 22, 128, 64, 128, 64), (False, 22, 256, 72, 256, 200),
                                                (False, 22, 512, 300, 200, 150)])
def test_orthonormal_over_twelve_decades(gpu_lib, fused, n, D, dl, dm, dr):
    from paper_2303_03681_amd import binding
    u, b0, b1, lam = _inputs(np.random.default_rng([dl, dm, dr, 7]), dl, dm, dr, 12)
    _, br, got = _gate(binding, n, n // 2 - 1, D, u, b0, b1, lam, 0, fused)
    k = len(got)
    V = br.transpose(1, 0, 2).reshape(k, 2 * dr)
    d = np.abs(V @ V.conj().T - np.eye(k)).max()
    print(f"fused {fused} {2 * dl}x{2 * dr}: k={k}, sigma_k / sigma_1 {got[-1] / got[0]:.1e}, "
          f"orthonormality {d:.1e}", flush=True)
    assert d <= 1e-12
