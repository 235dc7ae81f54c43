"""Performance cases of the MPS energy evaluation: what a VQE program asks of it.

Every case is one call sequence on handles a program keeps (the MPSs and the
compiled Pauli sums); inputs are drawn from the seed.  The families:

  ansatz     prefix-cached UCCSD step: copy the state after an unchanged
             circuit prefix, apply a window of the (sequential) UCCSD gate
             chain, evaluate the energy.  Small molecules, 8 .. 12 qubits.
  fragments  the same for several fragments at once through the multi-state
             calls (gradient shifts, the serving mix).
  layer      hardware-efficient ansatz: one more brickwork layer on a state
             whose bonds are at the cap, then the energy.
  expect     the energy of a state the handle has not seen, in each precision
             of the environments.
  canonical  the gauge restored (exact Schmidt values), then the energy.
  rdm        the fragment 2-RDM that follows an energy in a DMET loop.

Values that were asked for in a 32-bit (c64) or split 16-bit environment
precision are handed on as 32-bit numbers, those of c128 as 64-bit numbers.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2303_03681_amd import binding
from workloads.circuits import (
    brickwork_gates, fuse_gates, pack_gates, uccsd_gates, uccsd_n_params,
)
from workloads.rdm import two_rdm_rows

WINDOW = 5  # consecutive orbitals an excitation of the windowed UCCSD spans


def listed():
    return [
        # a small molecule (8 spin orbitals): every call is latency
        {"name": "ansatz 8q D16", "kind": "ansatz", "n": 8, "bond": 16, "skip": 200, "gates": 48,
         "strings": 361, "prec": "c128"},
        # a 12-orbital fragment, bonds up to 64, no truncation at the cap
        {"name": "ansatz 12q D64", "kind": "ansatz", "n": 12, "bond": 64, "skip": 600, "gates": 40,
         "strings": 1819, "prec": "c128"},
        # 16 fragments (or parameter-shifted copies) advancing together
        {"name": "fragments 16 x 10q D32", "kind": "fragments", "count": 16, "n": 10, "bond": 32, "skip": 200,
         "gates": 32, "strings": 875, "prec": "c128"},
        # brickwork on 24 qubits at the bond dimension of the serving mix
        {"name": "layer 24q D64", "kind": "layer", "n": 24, "bond": 64, "strings": 4096, "prec": "c128"},
        # odd sizes: neither the qubits nor the bond are round numbers
        {"name": "layer 31q D150", "kind": "layer", "n": 31, "bond": 150, "strings": 1500, "prec": "c64"},
        # the quoted benchmark's bond dimension
        {"name": "layer 36q D256", "kind": "layer", "n": 36, "bond": 256, "strings": 4096, "prec": "c128"},
        # the largest: rows of 1024 elements in every gate of the middle
        {"name": "layer 28q D512", "kind": "layer", "n": 28, "bond": 512, "strings": 512, "prec": "c64"},
        # a fragment's energy: many short launches
        {"name": "expect 16q D32 c128", "kind": "expect", "n": 16, "bond": 32, "strings": 5793, "prec": "c128"},
        # a chain of orbitals at a middle bond dimension
        {"name": "expect 40q D128 c64", "kind": "expect", "n": 40, "bond": 128, "strings": 16384, "prec": "c64"},
        # the quoted benchmark's state: double precision and split 16-bit environments
        {"name": "expect 50q D256 c128", "kind": "expect", "n": 50, "bond": 256, "strings": 8192, "prec": "c128"},
        {"name": "expect 50q D256 split_f16", "kind": "expect", "n": 50, "bond": 256, "strings": 32768,
         "prec": "split_f16"},
        # a 20-qubit fragment brought to exact canonical form
        {"name": "canonical 20q D64", "kind": "canonical", "n": 20, "bond": 64, "strings": 2048, "prec": "c128"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ansatz", "fragments", "layer", "layer", "expect", "expect", "canonical", "rdm"])
    if kind in ("ansatz", "fragments"):
        n = rng.choice([8, 10, 12])
        c = {"kind": kind, "n": n, "bond": 64 if n == 12 else rng.choice([32, 64]), "skip": rng.randint(60, 500),
             "gates": rng.randint(16, 64), "strings": _log_int(rng, 64, 1500), "prec": rng.choice(["c128", "c64"])}
        if kind == "fragments":
            c["count"] = _log_int(rng, 3, 24)
        return c
    if kind == "layer":
        bond = _log_int(rng, 24, 320)
        n = rng.randint(max(14, 2 * math.ceil(math.log2(bond)) + 2), 40 if bond <= 200 else 28)
        return {"kind": kind, "n": n, "bond": bond, "strings": _log_int(rng, 256, 4096),
                "prec": rng.choice(["c128", "c64", "split_f16", "split_bf16"])}
    if kind == "expect":
        n = rng.randint(12, 48)
        return {"kind": kind, "n": n, "bond": _log_int(rng, 16, 224), "strings": _log_int(rng, 256, 16384),
                "prec": rng.choice(["c128", "c64", "split_f16", "split_bf16"])}
    if kind == "canonical":
        return {"kind": kind, "n": rng.randint(12, 26), "bond": _log_int(rng, 16, 96),
                "strings": _log_int(rng, 256, 2048), "prec": rng.choice(["c128", "c64"])}
    return {"kind": "rdm", "n": rng.choice([6, 8, 10]), "bond": rng.choice([32, 64]), "skip": rng.randint(60, 400),
            "prec": rng.choice(["c128", "c64"])}


# ---------------------------------------------------------------- inputs

def _strings(rng, n, count):
    """The identity and `count` distinct strings of the Jordan-Wigner forms
    (Z, ZZ, hopping with parity string and optional Z, four-index exchange
    with parity strings), with coefficients like those of molecular sums."""
    out = np.zeros((0, n), np.uint8)
    for _ in range(8):
        m = 2 * count
        cols = np.arange(n)[None, :]
        idx = np.sort(np.argsort(rng.random((m, n)), axis=1)[:, :4], axis=1)
        p, q, r, s = (idx[:, k:k + 1] for k in range(4))
        form = rng.choice(4, size=(m, 1), p=[0.02, 0.04, 0.14, 0.8])
        letters = 1 + rng.integers(0, 2, size=(m, 4)).astype(np.uint8)
        letters[:, 3] = 1 + (letters[:, :3] == 2).sum(axis=1) % 2  # an even number of Y
        codes = np.zeros((m, n), np.uint8)
        for k, site in enumerate((p, q, r, s)):
            codes[cols == site] = letters[:, k]
        parity = ((cols > p) & (cols < q)) | ((cols > r) & (cols < s))
        codes[(form == 3) & parity] = 3
        hop = np.where(cols == p, letters[:, :1], 0) + np.where(cols == q, letters[:, :1], 0)
        hop = np.where((cols > p) & (cols < q), 3, hop)
        hop = np.where((cols == r) & (letters[:, 1:2] == 1), 3, hop)
        codes = np.where(form == 2, hop, codes)
        codes = np.where(form == 1, 3 * ((cols == p) | (cols == q)), codes)
        codes = np.where(form == 0, 3 * (cols == p), codes).astype(np.uint8)
        out = np.unique(np.concatenate([out, codes]), axis=0)
        if len(out) >= count:
            break
    out = out[np.sort(rng.choice(len(out), size=min(count, len(out)), replace=False))]
    weight = (out != 0).sum(axis=1)
    coeffs = rng.normal(0.0, 0.02, size=len(out)) + np.where(weight <= 2, rng.normal(0.0, 0.2, size=len(out)), 0.0)
    return (np.concatenate([np.zeros((1, n), np.uint8), out]), np.concatenate([[-2.0 - rng.random()], coeffs]))


def _uccsd(rng, case):
    """Prefix and window of the windowed UCCSD circuit with angles U(-0.1, 0.1)."""
    n = case["n"]
    bits = np.zeros(n, np.uint8)
    bits[:n // 2] = 1
    theta = rng.uniform(-0.1, 0.1, size=uccsd_n_params(n, n // 2, window=WINDOW))
    gates = fuse_gates(uccsd_gates(n, n // 2, theta, window=WINDOW), n)
    skip = min(case["skip"], max(0, len(gates) - case.get("gates", 0)))
    return bits, gates[:skip], gates[skip:skip + case.get("gates", 0)]


def _brickwork(rng, case):
    """Layers that bring the bonds to the cap, and one layer more."""
    n = case["n"]
    bits = (np.arange(n) % 2).astype(np.uint8)
    layers = min(n // 2, math.ceil(math.log2(case["bond"]))) + 1
    angles = rng.uniform(-math.pi, math.pi, size=(layers + 1, n, 2))
    return (bits, fuse_gates(brickwork_gates(n, angles[:layers]), n),
            fuse_gates(brickwork_gates(n, angles[layers:]), n))


def _circuit(case, rng):
    return _uccsd(rng, case) if case["kind"] in ("ansatz", "fragments", "rdm") else _brickwork(rng, case)


def _cutoff(case):
    return 1e-10 if case["kind"] in ("ansatz", "fragments", "rdm") else 1e-14


def _one(case, rng):
    bits, prefix, window = _circuit(case, rng)
    stream = torch.cuda.current_stream().cuda_stream
    base, work = (binding.Mps(case["n"], case["bond"], _cutoff(case), bits=bits, stream=stream) for _ in range(2))
    s = {"base": base, "work": work, "prefix": pack_gates(prefix), "gates": pack_gates(window)}
    if case["kind"] == "rdm":
        s["rows"] = two_rdm_rows(case["n"])
        s["plan"] = binding.PauliSum(s["rows"].strings.codes, s["rows"].strings.coeffs)
    else:
        s["plan"] = binding.PauliSum(*_strings(rng, case["n"], case["strings"]))
    return s


def prepare(case, seed):
    rngs = [np.random.default_rng([seed, k]) for k in range(case.get("count", 1))]
    parts = [_one(case, r) for r in rngs]
    if len(parts) == 1:
        parts[0]["base"].apply_gates(*parts[0]["prefix"])
    else:
        binding.apply_gates_multi([s["base"] for s in parts], [s["prefix"] for s in parts],
                                  stream=torch.cuda.current_stream().cuda_stream)
    return {"case": case, "parts": parts}


# ---------------------------------------------------------------- one pass

def _values(case, energy, per_term):
    t = np.float64 if case["prec"] == "c128" else np.float32
    return {"energy": np.asarray(energy, t), "per_term": np.asarray(per_term, t)}


def run(state):
    case, parts = state["case"], state["parts"]
    kind, prec = case["kind"], case["prec"]
    for s in parts:
        s["work"].copy_from(s["base"])
    if kind == "fragments":
        works = [s["work"] for s in parts]
        binding.apply_gates_multi(works, [s["gates"] for s in parts],
                                  stream=torch.cuda.current_stream().cuda_stream)
        e, per = binding.expect_multi(works, [s["plan"] for s in parts], prec, per_term=True)
        return _values(case, e, np.concatenate(per))
    s = parts[0]
    w = s["work"]
    if kind == "rdm":
        r = s["rows"]
        out = w.expect_rows(s["plan"], r.row_ptr, r.cols, r.vals, prec)
        return {"rows": out.astype(np.float64 if prec == "c128" else np.float32)}
    if kind in ("ansatz", "layer"):
        w.apply_gates(*s["gates"])
    if kind == "canonical":
        w.canonicalize()
    out = _values(case, *w.expect(s["plan"], prec, per_term=True))
    if kind in ("layer", "canonical"):
        out |= {"norm": np.float64(w.norm()), "bond_dims": w.bond_dims()}
    if kind == "layer":
        out["discarded"] = np.float64(w.discarded_weight())
    return out


# ---------------------------------------------------------------- the least a pass needs

def _caps(case):
    n = case["n"]
    return [min(case["bond"], 2 ** min(b, n - b)) for b in range(n + 1)]


def work(case):
    n, D = case["n"], _caps(case)
    sites = 16.0 * sum(2 * D[q] * D[q + 1] for q in range(n))
    prec_bytes = 16.0 if case["prec"] == "c128" else 8.0
    bytes_, flops = 2 * sites, 0.0  # the copy of the state
    if case["kind"] in ("ansatz", "fragments", "layer"):
        each = []
        for q in range(n - 1):
            a, b, m = 2 * D[q], 2 * D[q + 2], D[q + 1]
            lo, hi = min(a, b), max(a, b)
            # two-site product, SVD (values and one side: 4 (2 hi lo^2 + 11 lo^3)), site update
            each.append(8.0 * a * b * m + 4.0 * (2 * hi * lo * lo + 11.0 * lo ** 3) + 8.0 * a * b * m)
        if case["kind"] == "layer":
            flops += sum(each)
            bytes_ += 2 * sites
        else:
            flops += case["gates"] * sum(each) / len(each)
            bytes_ += case["gates"] * 2 * sites / n * 2
    if case["kind"] == "canonical":
        for q in range(n):
            a, b = 2 * D[q], D[q + 1]
            flops += 8.0 * a * b * b + 4.0 * (2 * a * b * b) + 4.0 * (2 * max(D[q], 2 * b) * D[q] ** 2 + 11.0 * D[q] ** 3)
        bytes_ += 4 * sites
    # boundary environments of both sides, then about one transfer update per
    # three strings (shared prefixes and suffixes) at the mean bond
    update = [16.0 * D[q] * D[q + 1] * (D[q] + D[q + 1]) for q in range(n)]
    strings = case.get("strings", 3 * n ** 3 / 2)
    flops += 2 * sum(update) + strings / 3 * sum(update) / n + 4.0 * strings * sum(d * d for d in D) / n
    bytes_ += sites + strings / 3 * prec_bytes * 2 * sum(d * d for d in D) / n + 8.0 * strings
    k = case.get("count", 1)
    return {"bytes": k * bytes_, "flops": k * flops}


# ---------------------------------------------------------------- 64-bit reference

def _dense_state(n, bits, gates):
    psi = np.zeros(2 ** n, complex)
    psi[int("".join(str(int(b)) for b in bits), 2)] = 1.0
    for g in gates:
        k = 1 if g.q1 < 0 else 2
        x = psi.reshape(2 ** g.q0, 2 ** k, -1)
        psi = np.einsum("ij,ajb->aib", g.u, x).reshape(-1)
    return psi


def _truncated_state(n, bond, cutoff, bits, gates):
    """The same circuit on a matrix product state with LAPACK's SVD (Hastings
    update, cap and cutoff, kept values renormalised)."""
    B = [np.zeros((2, 1, 1), complex) for _ in range(n)]
    for q in range(n):
        B[q][int(bits[q]), 0, 0] = 1.0
    lam = [np.ones(1) for _ in range(n + 1)]
    lost = 0.0
    for g in gates:
        q = g.q0
        if g.q1 < 0:
            B[q] = np.tensordot(g.u, B[q], 1)
            continue
        dl, dr = B[q].shape[1], B[q + 1].shape[2]
        theta = (B[q].reshape(2 * dl, -1) @ B[q + 1].transpose(1, 0, 2).reshape(B[q].shape[2], 2 * dr))
        theta = theta.reshape(2, dl, 2, dr).transpose(0, 2, 1, 3).reshape(4, -1)
        C = (g.u @ theta).reshape(2, 2, dl, dr).transpose(0, 2, 1, 3).reshape(2 * dl, 2 * dr)
        _, sv, vh = np.linalg.svd(np.tile(lam[q], 2)[:, None] * C, full_matrices=False)
        k = max(1, min(bond, int((sv > cutoff * np.linalg.norm(sv)).sum())))
        kept = np.linalg.norm(sv[:k])
        lost += (sv[k:] ** 2).sum() / (sv ** 2).sum()
        B[q] = (C @ vh[:k].conj().T / kept).reshape(2, dl, k)
        B[q + 1] = np.ascontiguousarray(vh[:k].reshape(k, 2, dr).transpose(1, 0, 2))
        lam[q + 1] = sv[:k] / kept
    psi = np.ones((1, 1), complex)
    for t in B:
        psi = np.tensordot(psi, t, ([1], [1])).reshape(-1, t.shape[2])
    return psi.reshape(-1), [1] + [t.shape[2] for t in B], lost


def _pauli_values(psi, codes):
    """Re <psi|P|psi> / <psi|psi> of every string on the dense state."""
    n = codes.shape[1]
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    v = torch.from_numpy(np.ascontiguousarray(psi)).to(dev)
    idx = torch.arange(v.numel(), device=dev)
    bit = 2 ** np.arange(n - 1, -1, -1, dtype=np.int64)
    norm = float((v.real ** 2 + v.imag ** 2).sum())
    out = []
    for c in codes:
        x = int(bit[(c == 1) | (c == 2)].sum())
        z = int(bit[(c == 2) | (c == 3)].sum())
        par = idx & z
        for sh in (32, 16, 8, 4, 2, 1):
            par = par ^ (par >> sh)
        sign = (1 - 2 * (par & 1)).to(torch.float64)
        # P|j> = i^{#Y} (-1)^{|j & z|} |j ^ x>
        amp = (v[idx ^ x].conj() * v * sign).sum()
        out.append(complex(amp) * 1j ** int((c == 2).sum()))
    return np.array(out).real / norm


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    brick = kind in ("layer", "expect", "canonical")
    if n > 24 or (brick and case["bond"] > 96) or case.get("strings", 0) * 2 ** n > 2 ** 36:
        return None
    energies, values = [], []
    dims, lost, norm = None, None, None
    for k in range(case.get("count", 1)):
        rng = np.random.default_rng([seed, k])
        bits, prefix, window = _circuit(case, rng)
        gates = prefix + (window if kind in ("ansatz", "fragments", "layer") else [])
        if brick:
            psi, dims, lost = _truncated_state(n, case["bond"], _cutoff(case), bits, gates)
            norm = np.linalg.norm(psi)
        else:
            psi = _dense_state(n, bits, gates)
        if kind == "rdm":
            r = two_rdm_rows(n)
            val = _pauli_values(psi, r.strings.codes)
            return {"rows": np.add.reduceat(np.append(r.vals * val[r.cols], 0.0), r.row_ptr[:-1])
                    * (np.diff(r.row_ptr) > 0)}
        codes, coeffs = _strings(rng, n, case["strings"])
        values.append(_pauli_values(psi, codes))
        energies.append(math.fsum(coeffs * values[-1]))
    out = {"energy": np.array(energies) if kind == "fragments" else np.float64(energies[0]),
           "per_term": np.concatenate(values)}
    if kind in ("layer", "canonical"):
        out |= {"norm": np.float64(norm), "bond_dims": None}
    if kind == "layer":
        out["discarded"] = np.float64(lost)
    return out
