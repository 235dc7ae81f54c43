"""GPU: environment updates merged over passes and states, and the kernel that
runs a small update in one workgroup, against one GEMM launch per half and site
(a forced tile): the same products in the same order, so every value is equal
bit for bit.  Bonds just below, at and above the 16-wide tiles, the 32 and 64
limits; state copies by one launch."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _state(binding, n, D, rng, **kw):
    m = binding.Mps(n, D, 1e-14, **kw)
    q0, us = [], []
    for _ in range(D.bit_length() + 1):
        for start in (0, 1):
            for q in range(start, n - 1, 2):
                q0.append(q)
                us.append(np.linalg.qr(rng.standard_normal((4, 4)) + 1j * rng.standard_normal((4, 4)))[0])
    u = np.zeros((len(us), 16, 2))
    for i, g in enumerate(us):
        u[i, :, 0], u[i, :, 1] = g.ravel().real, g.ravel().imag
    m.apply_gates(q0, np.array(q0) + 1, u)
    return m


def _copy(binding, m, D, **kw):
    c = binding.Mps(m.n, D, 1e-14, **kw)
    c.copy_from(m)
    return c


def _plan(binding, n, count, rng):
    codes = np.unique(rng.integers(0, 4, size=(count, n)).astype(np.uint8), axis=0)
    return binding.PauliSum(codes, rng.standard_normal(len(codes)))


@pytest.mark.parametrize("n,D", [(3, 1), (5, 3), (9, 15), (9, 16), (10, 17), (11, 31), (11, 32), (12, 33), (13, 63),
                                 (13, 64), (14, 65)])
@pytest.mark.parametrize("canonical", [False, True])
def test_merged_equals_one_by_one(gpu_lib, n, D, canonical):
    from paper_2303_03681_amd import binding
    rng = np.random.default_rng([n, D])
    m = _state(binding, n, D, rng)
    if canonical:
        m.canonicalize()
    plan = _plan(binding, n, 150, rng)
    kinds = [{}, {"hbm_budget_bytes": 1 << 30}]  # with a budget the passes stay apart
    for prec in ("c128", "c64", "split_f16"):
        one = _copy(binding, m, D)
        one.set_env_tile(0)
        e0, p0 = one.expect(plan, prec, per_term=True)
        for kw in kinds:
            c = _copy(binding, m, D, **kw)
            e, p = c.expect(plan, prec, per_term=True)
            assert e == e0 and np.array_equal(p, p0), (prec, kw)
            c.close()
        one.close()
    c = _copy(binding, m, D)
    assert np.array_equal(c.bond_dims(), m.bond_dims())
    for q in range(n):
        for a, b in zip(c.export_site(q), m.export_site(q)):
            assert np.array_equal(a, b)
    print(f"n={n} D={D} canonical={canonical}: bonds {m.bond_dims().tolist()}", flush=True)
    c.close()
    m.close()


@pytest.mark.parametrize("count", [1, 2, 31, 33, 70])  # segments of a launch: 2 .. 140, around 64
def test_many_states(gpu_lib, count):
    from paper_2303_03681_amd import binding
    rng = np.random.default_rng(count)
    base = [(_state(binding, n, D, rng), D, _plan(binding, n, k, rng))
            for n, D, k in ((4, 4, 20), (7, 9, 1), (8, 16, 60), (10, 33, 30))]
    pick = [base[i % len(base)] for i in range(count)]
    states = [_copy(binding, m, D) for m, D, _ in pick]
    single = [m.expect(p, "c128", per_term=True) for m, _, p in base]
    e, per = binding.expect_multi(states, [p for _, _, p in pick], "c128", per_term=True)
    for i in range(count):
        assert e[i] == single[i % len(base)][0]
        assert np.array_equal(per[i], single[i % len(base)][1])
    print(f"{count} states", flush=True)
    for m in states:
        m.close()
    for m, _, p in base:
        m.close()
        p.close()


# updates in the 64 x 64 and 128 x 64 tiles against the 32 x 32 ones: bonds at
# their edges, K not a multiple of the chunk, enough strings for 1024 tiles
@pytest.mark.parametrize("n,D,count", [(13, 7, 40), (14, 63, 60), (14, 64, 3000), (15, 65, 60), (16, 127, 300),
                                       (16, 128, 1500), (16, 129, 300), (17, 200, 200)])
def test_tiles_agree(gpu_lib, n, D, count):
    from paper_2303_03681_amd import binding
    rng = np.random.default_rng([n, D, count])
    m = _state(binding, n, D, rng)
    plan = _plan(binding, n, count, rng)
    for prec in ("c128", "c64"):
        out = []
        for tile in (-1, 0, 1):
            m.set_env_tile(tile)
            out.append(m.expect(plan, prec, per_term=True))
        print(f"n={n} D={D} {prec}: bonds up to {m.bond_dims().max()}, E {out[0][0]:.12f}", flush=True)
        for e, p in out[:2]:
            assert e == out[2][0] and np.array_equal(p, out[2][1])
    m.close()
    plan.close()
