"""Host orchestration against a stand-in for the HIP runtime (fake_hip.cpp):
which workspaces are allocated, when, and what happens without room for the
optional ones.  Each test runs in a process of its own, so that the stand-in
never meets the real runtime."""

import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, json, sys
sys.modules["torch"] = None
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
for f in ("fake_mallocs", "fake_frees", "fake_blocks", "fake_launches"):
    getattr(fake, f).restype = ctypes.c_longlong
fake.fake_used.restype = ctypes.c_size_t
fake.fake_set_capacity.argtypes = [ctypes.c_size_t]
import numpy as np
from paper_2303_03681_amd import binding

def layers(n, count):
    q0 = [q for _ in range(count) for s in (0, 1) for q in range(s, n - 1, 2)]
    u = np.zeros((len(q0), 16, 2))
    u[:, :, 0] = np.eye(4).ravel()
    return np.array(q0), np.array(q0) + 1, u

def preconditioned():
    return fake.fake_blocks(b"14lq_rank_kernel")

def direct():
    return fake.fake_blocks(b"15finalize_kernel")
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    out = tmp_path_factory.mktemp("fake") / "fake_hip.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_2303_03681_amd", "csrc"),
                    os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", str(out)], check=True)

    def run(script):
        res = subprocess.run([sys.executable, "-c", PRELUDE + script, str(out)], capture_output=True, text=True,
                             cwd=ROOT, timeout=120)
        assert res.returncode == 0, res.stdout + res.stderr
        return json.loads(res.stdout.splitlines()[-1])

    return run


SOLO = """
n, D = 16, 80
g, one = layers(n, 6), layers(n, 1)
m = binding.Mps(n, D, 1e-14, max_jacobi_sweeps=59)
m.set_fused_gates(False)
m.apply_gates(*g)
held = m.device_bytes() + 4 * (n // 2)  # the 60th sweep's rotation counters
m.close()
"""


@pytest.mark.parametrize("fused", [False, True])
def test_no_room_costs_no_allocations(fake, fused):
    """A budget (or a device) that fits the direct iteration and part of the
    factors: once the workspaces stand, a layer of gates allocates nothing."""
    r = fake(SOLO + f"""
out = []
side = 2 * 80
per = 2 * side * side * 16
for extra in (0, per // 2, per + per // 2, 3 * per, 7 * per + 4000):
    m = binding.Mps(n, D, 1e-14, hbm_budget_bytes=held + extra)
    m.set_fused_gates({fused})
    m.apply_gates(*g)
    a, f = fake.fake_mallocs(), fake.fake_frees()
    for _ in range(4):
        m.apply_gates(*one)
    out.append((fake.fake_mallocs() - a, fake.fake_frees() - f))
    m.close()
m = binding.Mps(n, D, 1e-14)
m.set_fused_gates({fused})
fake.fake_set_capacity(fake.fake_used() - m.device_bytes() + held + 3 * per)
m.apply_gates(*g)
a, f = fake.fake_mallocs(), fake.fake_frees()
for _ in range(4):
    m.apply_gates(*one)
out.append((fake.fake_mallocs() - a, fake.fake_frees() - f))
print(json.dumps(out))
""")
    # without a budget the device refuses: one attempt per batch size (7 or 8 gates) at the most
    assert r[:-1] == [[0, 0]] * 5
    assert r[-1][0] <= 2 and r[-1][1] == 0


def test_a_budget_is_its_own_handles_matter(fake):
    """One handle of a batch has no room for the factors: its gate is iterated
    directly, the others' are preconditioned as they are alone."""
    r = fake("""
n, D = 16, 80
g, one = layers(n, 6), layers(n, 1)
held = {}
def batch(budgets):
    ms = [binding.Mps(n, D, 1e-14, hbm_budget_bytes=b) for b in budgets]
    binding.apply_gates_multi(ms, [g] * len(ms))
    p, d = preconditioned(), direct()
    binding.apply_gates_multi(ms, [one] * len(ms))
    out = (preconditioned() - p, direct() - d)
    held[len(ms)] = [m.device_bytes() for m in ms]
    for m in ms:
        m.close()
    return out
alone = batch([0])
pair = batch([0, 0])
m = binding.Mps(n, D, 1e-14, max_jacobi_sweeps=59)
binding.apply_gates_multi([m], [g])
tight = m.device_bytes() + 8192  # a batch of three has its counters at the first handle
m.close()
print(json.dumps([alone, pair, batch([tight]), batch([0, tight]), batch([tight, 0]), batch([0, tight, 0])]))
""")
    alone, pair, tight, *mixed = r
    gates = sum(alone)
    assert alone[0] > 0 and pair == [2 * alone[0], 2 * alone[1]]
    assert tight == [0, gates]
    for m, k in zip(mixed, (1, 1, 2)):
        assert m == [k * alone[0], k * alone[1] + gates]


FULL = """
def state(n, D, **kw):
    m = binding.Mps(n, D, 1e-14, **kw)
    m.set_fused_gates(False)
    m.apply_gates(*layers(n, 8))
    return m

def strings(n, count):
    codes = np.unique(np.random.default_rng(n).integers(0, 4, size=(count, n)).astype(np.uint8), axis=0)
    return binding.PauliSum(codes, np.ones(len(codes)))

def room(extra):
    fake.fake_set_capacity(fake.fake_used() + extra)

n, D = 16, 80
m = state(n, D, max_jacobi_sweeps=59)
need = m.device_bytes()
m.close()
"""


def test_idle_handles_give_optional_workspaces_back(fake):
    """A handle that fitted beside another one without its optional workspaces
    (the factors, the second pass' GEMM1 outputs) fits beside one with them."""
    r = fake(FULL + """
a = state(n, D)
bare = need + 4 * (n // 2)                 # the 60th sweep's rotation counters
pre = a.device_bytes() - bare
room(need - pre // 2)
b = state(n, D, max_jacobi_sweeps=59)      # takes the factors back
out = [pre, a.device_bytes() - bare]
room(1 << 30)
p = preconditioned()
a.apply_gates(*layers(n, 1))
out += [a.device_bytes() - bare - pre, preconditioned() - p]
a.canonicalize()
plan = strings(n, 400)
a.expect(plan, "c128")
held = a.device_bytes()
b.close()
room(need - pre - (1 << 20))               # the factors alone would not do
b = state(n, D, max_jacobi_sweeps=59)
out += [held - a.device_bytes() - pre]
b.close()
room(held)
out += [a.expect(plan, "c128"), held - a.device_bytes()]
a.close()
out += [fake.fake_used()]
print(json.dumps(out))
""")
    pre, left, back, again, more, e, missing, used = r
    assert pre > 1 << 20 and left == 0
    assert back == 0 and again > 0
    assert more > 1 << 20
    assert e == 0.0 and missing == pre  # the GEMM1 outputs are back, the factors wait for gates
    assert used == 0


def test_full_device_shares_gemm1_outputs(fake):
    """No room for GEMM1 outputs per pass: the expectation runs with shared ones,
    as under a budget, and repeats without allocating."""
    r = fake(FULL + """
plan = strings(n, 400)
held = []
for kw in ({"hbm_budget_bytes": 1 << 34}, {}):
    m = state(n, D, **kw)
    m.canonicalize()
    before = m.device_bytes()
    m.expect(plan, "c128")
    held.append(m.device_bytes() - before)
    m.close()
m = state(n, D, max_jacobi_sweeps=59)
m.canonicalize()
before = m.device_bytes()
room((held[0] + held[1]) // 2)
m.expect(plan, "c128")
held.append(m.device_bytes() - before)
a = fake.fake_mallocs()
m.expect(plan, "c128")
binding.expect_multi([m], [plan], "c128")
print(json.dumps(held + [fake.fake_mallocs() - a]))
""")
    shared, apart, full, again = r
    assert apart > shared + (1 << 20)
    assert full == shared and again == 0


def test_threads_on_a_full_device(fake):
    """Handles of several threads take each other's optional workspaces back:
    every call succeeds or reports no memory, and the books balance."""
    r = fake(FULL + """
import threading
plan = strings(n, 200)
ms = [state(n, D) for _ in range(4)]
for m in ms:
    m.canonicalize()
room(500 << 20)
bad, done = [], [0] * 4
def work(i):
    rng = np.random.default_rng(i)
    for k in range(60):
        try:
            if rng.random() < 0.5:
                ms[i].apply_gates(*layers(n, 1))
                ms[i].canonicalize()
            elif rng.random() < 0.7:
                assert ms[i].expect(plan, "c128") == 0.0
            else:
                x = state(n, D)
                x.close()
            done[i] += 1
        except binding.MpsError as e:
            if e.name != "MPS_ERR_OOM":
                bad.append(str(e))
t = [threading.Thread(target=work, args=(i,)) for i in range(4)]
[x.start() for x in t]
[x.join() for x in t]
held = sum(m.device_bytes() for m in ms) - fake.fake_used()
[m.close() for m in ms]
print(json.dumps([bad, done, held, fake.fake_used()]))
""")
    bad, done, held, used = r
    assert bad == [] and min(done) > 0
    assert held == 0 and used == 0


@pytest.mark.parametrize("qubits,bond,strings", [(12, 32, 2000), (16, 64, 4000), (24, 64, 6000), (32, 128, 8000),
                                                 (40, 128, 8000)])
def test_serving_estimate_is_an_upper_one(fake, qubits, bond, strings):
    """Device memory of a served fragment whose bonds are all at their cap."""
    r = fake(f"""
fake.fake_set_capacity(1 << 36)
from paper_2303_03681_amd import serving
from workloads.configs import build_serving_fragments
frag = serving.Fragment.from_dict(build_serving_fragments(1, 1, qubits=({qubits},), bonds=({bond},),
                                                          max_strings={strings})[0])
back = serving.GpuBackend.__new__(serving.GpuBackend)
back.binding, back.prec, back.plans = binding, "c64", {{}}
server = serving.Server([frag], back, hbm_budget=1 << 40)
m = back.create(frag)
binding.apply_gates_multi([m], [layers({qubits}, 10)])
try:
    back.expect_many([(m, frag)])
except binding.MpsError as e:  # the stand-in computes no norm
    assert e.name == "MPS_ERR_NONFINITE"
print(json.dumps([server._need(frag), m.device_bytes(), int(m.bond_dims().max()), back.plan_updates(frag)]))
""")
    est, held, most, updates = r
    print(f"{qubits} qubits D = {bond}: estimate {est / 1e6:.1f} MB, held {held / 1e6:.1f} MB, {updates} updates")
    assert most == bond
    assert held <= est <= 3 * held


@pytest.mark.parametrize("D,prec", [(8, "c128"), (32, "c64"), (33, "c128"), (80, "c64"), (16, "split_f16")])
def test_environment_launches_are_counted_as_made(fake, D, prec):
    """mps_timing.env_launches against the launches of the environment kernels,
    alone and together with another state."""
    r = fake(FULL + f"""
def made():
    return fake.fake_launches(b"env_small_kernel") + fake.fake_launches(b"EnvG")
a, b = state(16, {D}), state(16, {D})
for m in (a, b):
    m.canonicalize()
plan, other = strings(16, 400), strings(16, 90)
out = []
for run in (lambda: a.expect(plan, "{prec}"), lambda: binding.expect_multi([a, b], [plan, other], "{prec}")):
    a.set_timing(True)
    before = made()
    run()
    out += [made() - before, a.timing()["env_launches"]]
print(json.dumps(out))
""")
    assert r[0] > 0 and r[2] > 0
    assert r[1] == r[0] and r[3] == r[2]


CLOSES = """
def exchange(n, count):
    rng = np.random.default_rng(n)
    idx = np.sort(np.argsort(rng.random((count, n)), axis=1)[:, :4], axis=1)
    cols, rows = np.arange(n), np.arange(count)
    p, q, r, s = (idx[:, k:k + 1] for k in range(4))
    codes = 3 * (((cols > p) & (cols < q)) | ((cols > r) & (cols < s))).astype(np.uint8)
    for k in range(4):
        codes[rows, idx[:, k]] = 1 + rng.integers(0, 2, count)
    codes = np.unique(codes, axis=0)
    return binding.PauliSum(codes, np.ones(len(codes)))

def dense(n, sites):  # every string on the middle sites
    codes = np.zeros((4 ** sites, n), np.uint8)
    codes[:, (n - sites) // 2:(n - sites) // 2 + sites] = np.array(np.unravel_index(np.arange(4 ** sites), (4,) * sites)).T
    return binding.PauliSum(codes, np.ones(len(codes)))
"""


@pytest.mark.parametrize("n,D,count,prec,pairs", [(48, 32, 220000, "c128", False), (48, 32, 220000, "c64", True),
                                                  (48, 32, 3000, "c128", True), (40, 64, 200000, "c128", False),
                                                  (12, 32, 200, "c64", True), (16, 32, 8, "c128", False),
                                                  (16, 128, 8, "c128", False), (18, 16, 9, "c64", False)])
def test_closes_are_chosen_for_all_bonds_together(fake, n, D, count, prec, pairs):
    """Sums whose bonds each have few tiles but together fill the chip (48 qubits
    D = 32, 200,001 strings: 0.25 ms as tiles, 0.37 as pairs in c128, 0.34 and
    0.17 in c64) are not split up as if every bond's tiles ran by themselves."""
    r = fake(FULL + CLOSES + f"""
m = state({n}, {D})
m.canonicalize()
plan = exchange({n}, {count}) if {count} > 99 else dense({n}, {count})
m.expect(plan, "{prec}")
print(json.dumps([fake.fake_blocks(b"gram_pairs"), fake.fake_blocks(b"GramTileP") + fake.fake_blocks(b"GramSplitP")]))
""")
    print(f"{n} qubits D = {D} {count} {prec}: {r[0]} pair groups, {r[1]} tile blocks")
    assert (r[0] > 0) == pairs and (r[1] == 0) == pairs
