"""GPU: handles with and without an HBM budget in one call: what one of them has
no room for does not change another's results."""

import numpy as np
import pytest

from tests.test_gpu_env_merged import _plan, _state

pytestmark = pytest.mark.gpu


def _gates(n, layers, rng):
    q0 = [q for _ in range(layers) for start in (0, 1) for q in range(start, n - 1, 2)]
    u = np.zeros((len(q0), 16, 2))
    for i in range(len(q0)):
        g = np.linalg.qr(rng.standard_normal((4, 4)) + 1j * rng.standard_normal((4, 4)))[0]
        u[i, :, 0], u[i, :, 1] = g.ravel().real, g.ravel().imag
    return np.array(q0), np.array(q0) + 1, u


def _equal(a, b):
    assert list(a.bond_dims()) == list(b.bond_dims())
    for q in range(a.n):
        for x, y in zip(a.export_site(q), b.export_site(q)):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("tight_first", [False, True])
def test_gates_of_a_batch(gpu_lib, tight_first):
    """Bonds above the fused limit; the budget fits the direct iteration only."""
    from paper_2303_03681_amd import binding
    n, D = 16, 96
    lists = [_gates(n, 7, np.random.default_rng(k)) for k in range(2)]
    probe = binding.Mps(n, D, 1e-14, max_jacobi_sweeps=59)
    binding.apply_gates_multi([probe], [lists[1]])
    budget = probe.device_bytes() + 8192  # counters of a batch of two
    probe.close()
    make = [lambda: binding.Mps(n, D, 1e-14), lambda: binding.Mps(n, D, 1e-14, hbm_budget_bytes=budget)]
    alone = [f() for f in make]
    for m, g in zip(alone, lists):
        binding.apply_gates_multi([m], [g])
    mixed = [f() for f in make]
    order = [1, 0] if tight_first else [0, 1]
    binding.apply_gates_multi([mixed[i] for i in order], [lists[i] for i in order])
    for a, b in zip(mixed, alone):
        _equal(a, b)
    print(f"held: free {mixed[0].device_bytes()}, budget {budget} held {mixed[1].device_bytes()}", flush=True)
    assert mixed[1].device_bytes() <= budget
    for m in alone + mixed:
        m.close()


def test_expectations_together(gpu_lib):
    """Passes with GEMM1 outputs of their own (no budget) and shared ones."""
    from paper_2303_03681_amd import binding
    rng = np.random.default_rng(11)
    budgets = [0, 1 << 30, 0, 1 << 30]
    sizes = [(10, 24), (12, 40), (12, 70), (9, 9)]
    states = [_state(binding, n, D, rng, hbm_budget_bytes=b) for (n, D), b in zip(sizes, budgets)]
    plans = [_plan(binding, n, 200, rng) for n, _ in sizes]
    for prec in ("c128", "c64", "split_bf16"):
        single = [m.expect(p, prec, per_term=True) for m, p in zip(states, plans)]
        for pick in ([0, 1, 2, 3], [1, 0], [3, 2, 1], [0, 2]):
            e, per = binding.expect_multi([states[i] for i in pick], [plans[i] for i in pick], prec, per_term=True)
            for k, i in enumerate(pick):
                assert e[k] == single[i][0] and np.array_equal(per[k], single[i][1]), (prec, pick, i)
        print(prec, [round(s[0], 9) for s in single], flush=True)
    for m in states:
        m.close()


# more distinct parents at the middle sites than fit the 1 GiB of GEMM1 outputs
# (512 of 2 MiB in c128, 1024 of 1 MiB in c64): several chunks a depth, both passes merged
@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_chunks_of_parents(gpu_lib, prec):
    from paper_2303_03681_amd import binding
    rng = np.random.default_rng(12)
    n, D = 18, 256
    m = _state(binding, n, D, rng)
    plan = _plan(binding, n, 3000, rng)
    lpar, lsite, _ = plan.export()["left"]
    most = max(len(np.unique(lpar[lsite == s])) for s in np.unique(lsite))
    print(f"{prec}: bonds up to {m.bond_dims().max()}, {most} distinct parents at a site", flush=True)
    assert most > (1 << 30) // (2 * D * D * (16 if prec == "c128" else 8))
    e, per = m.expect(plan, prec, per_term=True)
    m.set_env_tile(1)  # one launch per half, chunk and pass
    e1, per1 = m.expect(plan, prec, per_term=True)
    assert e == e1 and np.array_equal(per, per1)
    m.close()
    b = _state(binding, n, D, np.random.default_rng(12), hbm_budget_bytes=64 << 30)
    e2, per2 = b.expect(plan, prec, per_term=True)  # shared GEMM1 outputs
    b.close()
    assert e2 == e and np.array_equal(per2, per)
