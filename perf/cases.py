"""The work that programs built on this library have it do, as timed cases.

``listed()`` names the cases, ``draw()`` gives others of the same ranges,
``prepare()`` builds what a program holds before the call (Hamiltonians,
ansatz programs, batches, angles, device buffers), ``run()`` makes one pass
through the public entry points, ``work()`` counts what a pass cannot do
without, and ``exact()`` gives the same outputs from a plain float64
simulation in torch that shares no code with the library.

Kinds of pass:

* ``single``: ``energy_grad`` of one Hamiltonian (the step of a VQE, and with
  ``grad`` off the energy a line search asks for);
* ``batch``: ``Batch.energy_grad_device`` over many problems of one or several
  qubit counts (bond-stretch scans, data sets of geometries);
* ``pool``: ``pool_gradient``, the operation every ADAPT round starts with;
* ``pairs``: a batch of pUCCD problems on hard-core bosons;
* ``state``: the statevector calls (prepare, apply an ansatz, expectation);
* ``rotations``: ``energy_grad`` of a program of Pauli rotations, which leaves
  the particle-number sector and runs on full complex vectors;
* ``mlp``: training steps of the warm-start network from given weights.
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

TUNING_CACHE = os.path.join("paper_2311_01242_amd", "tuning_cache.json")


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # the smallest VQE: every step of its optimiser is one such call
        {"name": "vqe4", "kind": "single", "ansatz": "uccsd", "mapping": "jw", "n": 4, "ne": 2, "grad": True},
        # the warm-start scan's geometries: plain VQE on 16 qubits, one call per BFGS step
        {"name": "vqe16", "kind": "single", "ansatz": "uccsd", "mapping": "jw", "n": 16, "ne": 8, "grad": True},
        # an energy without a gradient, as a line search or a potential-energy curve asks for
        {"name": "energy20", "kind": "single", "ansatz": "uccsd", "mapping": "jw", "n": 20, "ne": 10, "grad": False},
        # the largest single instance: 24 qubits, 1,818 angles
        {"name": "single24", "kind": "single", "ansatz": "uccsd", "mapping": "jw", "n": 24, "ne": 12, "grad": True},
        # a bond-stretch scan: 20 geometries of 12 qubits per step
        {"name": "scan12", "kind": "batch", "ansatz": "uccsd", "mapping": "jw", "states": 20, "n_min": 12,
         "n_max": 12, "tuned": False},
        # the headline batch: 512 problems of 12 to 20 qubits, launch parameters from the shipped tuning cache
        {"name": "batch512", "kind": "batch", "ansatz": "uccsd", "mapping": "jw", "states": 512, "n_min": 12,
         "n_max": 20, "tuned": True},
        # generalised pair excitations, odd and even qubit counts, no tuning run beforehand
        {"name": "kupccgsd64", "kind": "batch", "ansatz": "kupccgsd2", "mapping": "jw", "states": 64, "n_min": 11,
         "n_max": 18, "tuned": False},
        # one ADAPT round on 20 qubits: 16 operators in the ansatz, the pool of all 875
        {"name": "adapt20", "kind": "pool", "n": 20, "ne": 10, "operators": 16},
        # pUCCD at 11 orbitals and 7 pairs, 512 geometries per step
        {"name": "puccd11", "kind": "pairs", "n": 11, "ne": 7, "states": 512},
        # a full statevector for a program that goes on with it, and its energy
        {"name": "state18", "kind": "state", "n": 18, "ne": 9},
        # arbitrary Pauli rotations (a circuit that conserves nothing) with the adjoint gradient
        {"name": "rotations14", "kind": "rotations", "n": 14, "ne": 7, "gates": 400, "params": 120},
        # the warm-start network at its 16-qubit shapes
        {"name": "mlp16", "kind": "mlp", "features": 37, "hidden": 256, "outputs": 360, "samples": 160, "steps": 40},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    limit = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["single", "single", "single", "batch", "batch", "batch", "pool", "pairs", "state",
                           "rotations", "mlp"])
        if kind == "single":
            n = rng.randint(4, 23)
            ne = max(2, min(n - 2, n // 2 + rng.choice([0, 0, 0, -1, 1])))
            c = {"kind": kind, "ansatz": rng.choice(["uccsd", "uccsd", "trotter2", "kupccgsd2"]), "mapping": "jw",
                 "n": n, "ne": ne, "grad": rng.random() < 0.75}
            if c["ansatz"] == "uccsd" and n <= 16 and rng.random() < 0.25:
                c["mapping"] = "bk"
        elif kind == "batch":
            lo = rng.randint(6, 20)
            c = {"kind": kind, "ansatz": rng.choice(["uccsd", "uccsd", "trotter2", "kupccgsd2"]), "mapping": "jw",
                 "states": _log_int(rng, 2, 512), "n_min": lo, "n_max": min(20, lo + rng.choice([0, 0, 2, 5, 8])),
                 "tuned": False}
        elif kind == "pool":
            n = rng.randint(8, 21)
            c = {"kind": kind, "n": n, "ne": n // 2, "operators": rng.randint(1, 24)}
        elif kind == "pairs":
            n = rng.randint(4, 12)
            c = {"kind": kind, "n": n, "ne": rng.randint(1, n - 1), "states": _log_int(rng, 1, 512)}
        elif kind == "state":
            n = rng.randint(6, 20)
            c = {"kind": kind, "n": n, "ne": n // 2}
        elif kind == "rotations":
            n = rng.randint(5, 16)
            gates = _log_int(rng, 20, 600)
            c = {"kind": kind, "n": n, "ne": n // 2, "gates": gates, "params": rng.randint(gates // 4, gates)}
        else:
            n = rng.randint(8, 20)
            ns, o, v = (n + 1) // 2, (n // 2) // 2, (n + 1) // 2 - (n // 2) // 2
            c = {"kind": kind, "features": 1 + ns * (ns + 1) // 2, "hidden": rng.choice([64, 128, 256, 300]),
                 "outputs": max(3, o * o * v * v), "samples": _log_int(rng, 8, 160), "steps": rng.randint(1, 40)}
        if _cost(c) <= limit:
            return c


# ---------------------------------------------------------------- the programs

def _excitations(n, ne, ansatz):
    """(annihilated..., created...) spin orbitals of every gate, with its parameter and angle factor."""
    if ansatz == "kupccgsd2":
        layer = [(p, q) for q in range(n) for p in range(q) if (p - q) % 2 == 0]
        layer += [(2 * p, 2 * p + 1, 2 * q, 2 * q + 1) for q in range(n // 2) for p in range(q)]
        return [(e, k * len(layer) + j, 1.0) for k in range(2) for j, e in enumerate(layer)], 2 * len(layer)
    occ, vir = range(ne), range(ne, n)
    ops = [(i, a) for a in vir for i in occ if (i - a) % 2 == 0]
    for a in vir:
        for b in range(a + 1, n):
            for i in occ:
                for j in range(i + 1, ne):
                    if i % 2 + j % 2 == a % 2 + b % 2:
                        ops.append((i, j, a, b))
    if ansatz == "trotter2":
        return [(e, j, 0.5) for _ in range(2) for j, e in enumerate(ops)], len(ops)
    return [(e, j, 1.0) for j, e in enumerate(ops)], len(ops)


def _sizes(case):
    """(n, n_e) of every state of a case."""
    if case["kind"] != "batch":
        return [(case["n"], case["ne"])] * case.get("states", 1)
    span = case["n_max"] - case["n_min"] + 1
    if case["tuned"]:   # the benchmark's batch: its counts are the tuning cache's keys
        return [(int(n), int(n) // 2) for n in
                np.random.default_rng(3).integers(case["n_min"], case["n_max"] + 1, size=case["states"])]
    return [(n, n // 2) for n in (case["n_min"] + (5 * i) % span for i in range(case["states"]))]


def _comb(n, k):
    return math.comb(n, k) if 0 <= k <= n else 0


def _sector(n, ne):
    """(alpha orbitals, beta orbitals, alpha electrons, beta electrons)."""
    return (n + 1) // 2, n // 2, (ne + 1) // 2, ne // 2


def _gate_pairs(n, ne, ansatz):
    """Amplitude pairs that the program's gates rotate within the reference's sector."""
    total, (oa, ob, na, nb) = 0, _sector(n, ne)
    kinds = {}
    for e, _, _ in _excitations(n, ne, ansatz)[0]:
        ka = sum(1 for p in e if p % 2 == 0) // 2
        kinds[(ka, len(e) // 2 - ka)] = kinds.get((ka, len(e) // 2 - ka), 0) + 1
    for (ka, kb), cnt in kinds.items():
        total += cnt * _comb(oa - 2 * ka, na - ka) * _comb(ob - 2 * kb, nb - kb)
    return total


def _h_elements(n, ne):
    """Nonzero matrix elements of a two-body Hamiltonian within the sector."""
    oa, ob, na, nb = _sector(n, ne)
    sa, sb = na * (oa - na), nb * (ob - nb)
    per = 1 + sa + sb + sa * sb + _comb(na, 2) * _comb(oa - na, 2) + _comb(nb, 2) * _comb(ob - nb, 2)
    return per * _comb(oa, na) * _comb(ob, nb)


def _integral_count(n):
    m = ((n + 1) // 2) * ((n + 1) // 2 + 1) // 2
    return m + m * (m + 1) // 2


def work(case):
    kind = case["kind"]
    if kind == "mlp":
        f, h, o, b, steps = (case[k] for k in ("features", "hidden", "outputs", "samples", "steps"))
        weights = f * h + h * h + h * o
        params = weights + 2 * h + o
        # each step: forward and weight gradients of three layers, input gradients of two
        return {"bytes": 4.0 * (2 * params + b * (f + o) + steps), "flops": steps * b * (6.0 * weights - 2.0 * f * h)}
    if kind == "pairs":
        n, k, S = case["n"], case["ne"], case["states"]
        m = k * (n - k)
        gate, elements = m * _comb(n - 2, k - 1), _comb(n, k) * (1 + m)
        return {"bytes": 8.0 * S * (2 * m + 1 + n * n), "flops": S * (6.0 * gate + 2.0 * elements + 16.0 * gate)}
    if kind == "rotations":
        n, m = case["n"], case["gates"]
        # per rotation 8 flops an amplitude forward, 2 vectors and a product of them in reverse
        terms = sum(_h_elements(n, ne) for ne in range(2, n - 1)) / max(1, _comb(n, n // 2))
        return {"bytes": 8.0 * (2 * case["params"] + 1 + _integral_count(n)) + 16.0 * m,
                "flops": (1 << n) * (m * 28.0) + 4.0 * terms * _comb(n, n // 2)}
    if kind == "state":
        n, ne = case["n"], case["ne"]
        m = _excitations(n, ne, "uccsd")[1]
        return {"bytes": 16.0 * (1 << n) + 8.0 * (m + 1 + _integral_count(n)),
                "flops": 12.0 * _gate_pairs(n, ne, "uccsd") + 4.0 * _h_elements(n, ne)}
    if kind == "pool":
        n, ne = case["n"], case["ne"]
        gates = _excitations(n, ne, "uccsd")[1]
        pairs = _gate_pairs(n, ne, "uccsd")
        return {"bytes": 8.0 * (case["operators"] + gates + 1 + _integral_count(n)),
                "flops": 6.0 * pairs * case["operators"] / gates + 2.0 * _h_elements(n, ne) + 4.0 * pairs}
    out = {"bytes": 0.0, "flops": 0.0}
    counts = {}
    for s in _sizes(case):
        counts[s] = counts.get(s, 0) + 1
    for (n, ne), S in counts.items():
        pairs, m = _gate_pairs(n, ne, case["ansatz"]), _excitations(n, ne, case["ansatz"])[1]
        grad = case.get("grad", True)
        out["bytes"] += S * 8.0 * (m * (2 if grad else 1) + 1 + _integral_count(n))
        # a rotation of a pair: 6 flops; in reverse two of them and the pair's gradient part (4)
        out["flops"] += S * (6.0 * pairs + 2.0 * _h_elements(n, ne) + (16.0 * pairs if grad else 0.0))
    return out


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


# ------------------------------------------------------------------ the inputs

def _symmetric(rng, ns, std):
    m = np.triu(rng.normal(0.0, std, (ns, ns)))
    return m + np.triu(m, 1).T


def _eightfold(rng, ns, std):
    p, q = np.tril_indices(ns)
    m = len(p)
    v = np.tril(rng.normal(0.0, std, (m, m)))
    v = v + np.tril(v, -1).T
    idx = np.zeros((ns, ns), np.int64)
    idx[p, q] = idx[q, p] = np.arange(m)
    return v[idx.reshape(-1)][:, idx.reshape(-1)].reshape(ns, ns, ns, ns)


def _integrals(rng, ns):
    """One geometry: h ~ N(0, 0.5^2) symmetric with its diagonal lowered by 1, (pq|rs) ~ N(0, 0.1^2)."""
    return 0.0, _symmetric(rng, ns, 0.5) - np.eye(ns), _eightfold(rng, ns, 0.1)


def _problems(case, seed):
    """[(n, n_e, h0, h, g, theta)] of every state of a case."""
    rng = np.random.default_rng([seed, 17])
    kind, out, counts = case["kind"], [], {}
    for n, ne in _sizes(case):
        ns = n if kind == "pairs" else (n + 1) // 2
        h0, h, g = _integrals(rng, ns)
        if kind == "pairs":
            m = ne * (n - ne)
        elif kind == "pool":
            m = case["operators"]
        elif kind == "rotations":
            m = case["params"]
        else:
            if (n, ne) not in counts:
                counts[n, ne] = _excitations(n, ne, case.get("ansatz", "uccsd"))[1]
            m = counts[n, ne]
        out.append((n, ne, h0, h, g, rng.uniform(-0.1, 0.1, m)))
    return out


def _pool_choice(case, seed):
    pool = _excitations(case["n"], case["ne"], "uccsd")[1]
    return [int(k) for k in np.random.default_rng([seed, 23]).integers(0, pool, case["operators"])]


def _rotation_program(case, seed):
    """x, z masks, parameter and factor of every rotation: one- and two-qubit strings with a few wider ones."""
    rng = np.random.default_rng([seed, 29])
    n, k = case["n"], case["gates"]
    x, z = np.zeros(k, np.uint32), np.zeros(k, np.uint32)
    for i in range(k):
        width = int(min(n, rng.choice([1, 2, 2, 2, 4])))
        for q in rng.choice(n, width, replace=False):
            letter = int(rng.integers(1, 4))
            x[i] |= np.uint32((letter & 1) << int(q))
            z[i] |= np.uint32((letter >> 1) << int(q))
    param = np.concatenate([np.arange(case["params"]), rng.integers(0, case["params"], k - case["params"])])
    return x, z, param.astype(np.int32), rng.uniform(0.5, 1.5, k)


def _mlp_data(case, seed):
    rng = np.random.default_rng([seed, 31])
    x = rng.normal(0.0, 1.0, (case["samples"], case["features"])).astype(np.float32)
    y = rng.normal(0.0, 0.1, (case["samples"], case["outputs"])).astype(np.float32)
    widths = [case["features"], case["hidden"], case["hidden"], case["outputs"]]
    parts = []
    for fi, fo in zip(widths[:-1], widths[1:]):
        parts += [rng.normal(0.0, math.sqrt(2.0 / fi), fo * fi), np.zeros(fo)]
    return widths, np.concatenate(parts).astype(np.float32), x, y


def _make_ansatz(vq, n, ne, ansatz, mapping):
    if ansatz == "kupccgsd2":
        return vq.Ansatz.kupccgsd(n, ne, 2)
    if ansatz == "trotter2":
        return vq.Ansatz.uccsd_trotter(n, ne, 2)
    return vq.Ansatz.uccsd(n, ne) if mapping == "jw" else vq.Ansatz.uccsd_map(n, ne, mapping)


def prepare(case, seed):
    import paper_2311_01242_amd as vq
    kind = case["kind"]
    if kind == "mlp":
        from paper_2311_01242_amd.mlp import MLP
        widths, p0, x, y = _mlp_data(case, seed)
        return {"kind": kind, "net": MLP(widths), "p0": p0, "x": x, "y": y, "steps": case["steps"]}
    probs = _problems(case, seed)
    if kind in ("batch", "pairs"):
        hams, ans, made = [], [], {}
        for n, ne, h0, h, g, _ in probs:
            if kind == "pairs":
                hams.append(vq.Hamiltonian.pairs_from_integrals(n, h0, h, g))
            else:
                hams.append(vq.Hamiltonian.from_integrals(n, h0, h, g))
            if (n, ne) not in made:
                made[n, ne] = vq.Ansatz.puccd(n, ne) if kind == "pairs" else \
                    _make_ansatz(vq, n, ne, case["ansatz"], case["mapping"])
            ans.append(made[n, ne])
        nes, theta = [p[1] for p in probs], np.concatenate([p[5] for p in probs])
        if kind == "batch":
            for n in sorted({p[0] for p in probs}):   # the built-in launch parameters
                vq.set_tuning(n, True)
                vq.set_run_threads(n, True)
                vq.set_tile_cap(n, True)
            if case["tuned"]:
                from paper_2311_01242_amd import autotune
                autotune.autotune_batch(hams, ans, nes, theta, np.cumsum([0] + [p[5].size for p in probs]),
                                        cache=TUNING_CACHE)
        b = vq.Batch(hams, ans, nes)
        return {"kind": "batch", "batch": b, "theta": torch.tensor(theta, device="cuda"),
                "e": torch.empty(b.S, dtype=torch.float64, device="cuda"),
                "g": torch.empty(theta.size, dtype=torch.float64, device="cuda")}
    n, ne, h0, h, g, theta = probs[0]
    if kind == "single":
        H = vq.Hamiltonian.from_integrals_map(n, case["mapping"], h0, h, g)
        A = _make_ansatz(vq, n, ne, case["ansatz"], case["mapping"])
        return {"kind": kind, "H": H, "A": A, "ne": ne, "theta": theta, "grad": case["grad"]}
    H = vq.Hamiltonian.from_integrals(n, h0, h, g)
    if kind == "rotations":
        A = vq.Ansatz.from_rotations(n, case["params"], *_rotation_program(case, seed))
        return {"kind": "single", "H": H, "A": A, "ne": ne, "theta": theta, "grad": True}
    if kind == "pool":
        pool = vq.Ansatz.uccsd(n, ne)
        return {"kind": kind, "H": H, "A": pool.select(_pool_choice(case, seed)), "pool": pool, "ne": ne,
                "theta": theta}
    psi = torch.empty(1 << n, dtype=torch.complex128, device="cuda")
    return {"kind": kind, "H": H, "A": vq.Ansatz.uccsd(n, ne), "ne": ne, "theta": theta, "psi": psi,
            "state": vq.State.wrap(psi)}


def run(state):
    import paper_2311_01242_amd as vq
    kind = state["kind"]
    if kind == "single":
        e, g = vq.energy_grad(state["H"], state["A"], state["ne"], state["theta"], grad=state["grad"])
        return {"energy": e, "gradient": g} if state["grad"] else {"energy": e}
    if kind == "batch":
        state["batch"].energy_grad_device(state["theta"], state["e"], state["g"])
        return {"energy": state["e"], "gradient": state["g"]}
    if kind == "pool":
        e, g = vq.pool_gradient(state["H"], state["A"], state["pool"], state["ne"], state["theta"])
        return {"energy": e, "gradient": g}
    if kind == "state":
        s = state["state"]
        s.prepare_hf(state["ne"])
        s.apply_ansatz(state["A"], state["theta"])
        return {"energy": s.expectation(state["H"]), "psi": state["psi"]}
    net = state["net"]
    net.set_params(state["p0"])
    trace = net.train(state["x"], state["y"], state["steps"])
    return {"loss": trace, "params": net.get_params()}


# ---------------------------------------------- the same outputs in plain torch

def _parity(v):
    for s in (16, 8, 4, 2, 1):
        v = v ^ (v >> s)
    return v & 1


class _Space:
    """Occupation strings of a sector (or of the whole register), with their positions."""

    def __init__(self, n, keep, dev):
        b = torch.arange(1 << n, dtype=torch.int64, device=dev)
        self.bits = b[keep(b)]
        self.pos = torch.full((1 << n,), -1, dtype=torch.int64, device=dev)
        self.pos[self.bits] = torch.arange(self.bits.numel(), device=dev)
        self.dev, self.size = dev, self.bits.numel()

    def move(self, gone, made, signs=True):
        """Sources, targets and signs of the product of ladder operators that empties `gone` and fills `made`
        (rightmost first: a_gone[0], a_gone[1], ..., then a+_made[last], ..., a+_made[0])."""
        need = sum(1 << p for p in gone)
        fill = sum(1 << p for p in made)
        src = torch.nonzero((self.bits & need == need) & ((self.bits & ~need) & fill == 0)).reshape(-1)
        d, par = self.bits[src], torch.zeros(src.numel(), dtype=torch.int64, device=self.dev)
        for p in list(gone) + list(made)[::-1]:
            par += _parity(d & ((1 << p) - 1))
            d = d ^ (1 << p)
        s = (1 - 2 * (par & 1)).to(torch.float64)
        return src, self.pos[d], s if signs else torch.ones_like(s)


def _count(b, mask):
    c = torch.zeros_like(b)
    while mask:
        low = mask & -mask
        c += (b & low) != 0
        mask ^= low
    return c


def _fermion_space(n, ne, dev):
    a_mask = sum(1 << q for q in range(0, n, 2))
    b_mask = sum(1 << q for q in range(1, n, 2))
    return _Space(n, lambda b: (_count(b, a_mask) == (ne + 1) // 2) & (_count(b, b_mask) == ne // 2), dev)


def _h_apply(sp, n, probs, psi):
    """H psi of every row of psi [states, strings] from the integrals: with E_pq = sum over spin of a+_p a_q,
    H = h0 + sum_pq (h_pq - 1/2 sum_r (pr|rq)) E_pq + 1/2 sum_pqrs (pq|rs) E_pq E_rs; on an odd register the last
    orbital has no beta spin orbital, so the sum over r is taken spin by spin."""
    ns, out = (n + 1) // 2, torch.zeros_like(psi)
    moves = {(P, Q): sp.move((Q,), (P,)) for P in range(n) for Q in range(n) if (P - Q) % 2 == 0}
    step = max(1, int(3e9 // (16 * ns * ns * sp.size)))
    for s0 in range(0, len(probs), step):
        v = psi[s0:s0 + step]
        part = probs[s0:s0 + step]
        D = torch.zeros((v.shape[0], ns * ns, sp.size), dtype=psi.dtype, device=psi.device)
        for (P, Q), (src, dst, sg) in moves.items():
            D[:, (P // 2) * ns + Q // 2, dst] += sg * v[:, src]
        g = torch.tensor(np.stack([p[4].reshape(ns * ns, ns * ns) for p in part]), device=psi.device).to(psi.dtype)
        G = 0.5 * torch.bmm(g, D)
        del D
        acc = torch.stack([torch.as_tensor(p[2], dtype=psi.dtype, device=psi.device) * v[k]
                           for k, p in enumerate(part)])
        for (P, Q), (src, dst, sg) in moves.items():
            k = []
            for p in part:
                same = [r for r in range(ns) if 2 * r + P % 2 < n]
                k.append(p[3][P // 2, Q // 2] - 0.5 * sum(p[4][P // 2, r, r, Q // 2] for r in same))
            k = torch.tensor(k, dtype=psi.dtype, device=psi.device)[:, None]
            acc[:, dst] += sg * (G[:, (P // 2) * ns + Q // 2, src] + k * v[:, src])
        out[s0:s0 + step] = acc
    return out


def _pairs_apply(sp, n, probs, psi):
    out = torch.zeros_like(psi)
    occ = [((sp.bits >> p) & 1).to(torch.float64) for p in range(n)]
    moves = {(p, q): sp.move((q,), (p,), signs=False) for p in range(n) for q in range(n) if p != q}
    for k, (_, _, h0, h, g, _) in enumerate(probs):
        d = torch.full((sp.size,), float(h0), dtype=torch.float64, device=psi.device)
        for p in range(n):
            d += (2 * h[p, p] + g[p, p, p, p]) * occ[p]
            for q in range(p + 1, n):
                d += 2 * (2 * g[p, p, q, q] - g[p, q, q, p]) * occ[p] * occ[q]
        acc = d * psi[k]
        for (p, q), (src, dst, _) in moves.items():
            acc[dst] += float(g[p, q, p, q]) * psi[k, src]
        out[k] = acc
    return out


def _rotate(psi, move, c, s):
    src, dst, sg = move
    d, e = psi[:, src], psi[:, dst]
    psi[:, src], psi[:, dst] = c * d - sg * s * e, c * e + sg * s * d


def _evaluate(sp, probs, gates, moves, apply_h, grad, n_params):
    """Energies and gradients of the states `probs` that share one gate program."""
    S, dev = len(probs), sp.dev
    th = torch.tensor(np.stack([p[5] for p in probs]), device=dev)
    psi = torch.zeros((S, sp.size), dtype=torch.float64, device=dev)
    psi[:, sp.pos[(1 << probs[0][1]) - 1]] = 1.0
    cs = [(torch.cos(f * th[:, p])[:, None], torch.sin(f * th[:, p])[:, None]) for _, p, f in gates]
    for k in range(len(gates)):
        _rotate(psi, moves[k], *cs[k])
    lam = apply_h(psi)
    e = (psi * lam).sum(1)
    g = torch.zeros((S, n_params), dtype=torch.float64, device=dev)
    if grad:
        for k in reversed(range(len(gates))):
            src, dst, sg = moves[k]
            g[:, gates[k][1]] += 2 * gates[k][2] * (sg * (lam[:, dst] * psi[:, src] - lam[:, src] * psi[:, dst])).sum(1)
            _rotate(psi, moves[k], cs[k][0], -cs[k][1])
            _rotate(lam, moves[k], cs[k][0], -cs[k][1])
    return psi, e, g


def _exact_mlp(case, seed):
    widths, p, x, y = _mlp_data(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    p, x, y = (torch.tensor(v, dtype=torch.float64, device=dev) for v in (p, x, y))
    m, v, trace = torch.zeros_like(p), torch.zeros_like(p), []
    for t in range(1, case["steps"] + 1):
        q = p.clone().requires_grad_(True)
        a, o = x, 0
        for li, (fi, fo) in enumerate(zip(widths[:-1], widths[1:])):
            w, b = q[o:o + fi * fo].reshape(fo, fi), q[o + fi * fo:o + fi * fo + fo]
            o += fi * fo + fo
            a = a @ w.T + b
            if li < 2:
                a = torch.nn.functional.gelu(a)
        loss = ((a - y) ** 2).mean()
        (gr,) = torch.autograd.grad(loss, q)
        trace.append(loss.detach())
        m, v = 0.9 * m + 0.1 * gr, 0.999 * v + 0.001 * gr * gr
        p = p - 1e-3 * (m / (1 - 0.9 ** t)) / (torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
    return {"loss": torch.stack(trace).cpu().numpy(), "params": p.cpu().numpy()}


def _exact_rotations(case, probs, seed, dev):
    n, ne, _, _, _, theta = probs[0]
    sp = _Space(n, lambda b: b >= 0, dev)
    x, z, param, scale = _rotation_program(case, seed)
    units = (1, 1j, -1, -1j)

    def string(psi, k):   # P |b> = i^#Y (-1)^(b.z) |b ^ x>
        ph = units[bin(int(x[k] & z[k])).count("1") % 4] * (1 - 2 * _parity(sp.bits & int(z[k]))).to(psi.dtype)
        return (ph * psi)[sp.bits ^ int(x[k])]

    def rotate(psi, k, sign):
        a = 0.5 * sign * float(scale[k]) * float(theta[param[k]])
        return math.cos(a) * psi - 1j * math.sin(a) * string(psi, k)

    psi = torch.zeros(sp.size, dtype=torch.complex128, device=dev)
    psi[(1 << ne) - 1] = 1.0
    for k in range(case["gates"]):
        psi = rotate(psi, k, 1.0)
    lam = _h_apply(sp, n, probs, psi[None])[0]
    e = torch.vdot(psi, lam).real
    g = torch.zeros(case["params"], dtype=torch.float64, device=dev)
    for k in reversed(range(case["gates"])):
        g[int(param[k])] += float(scale[k]) * torch.vdot(lam, string(psi, k)).imag
        psi, lam = rotate(psi, k, -1.0), rotate(lam, k, -1.0)
    return {"energy": float(e), "gradient": g.cpu().numpy()}


def exact(case, seed):
    kind = case["kind"]
    if kind == "mlp":
        return _exact_mlp(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    probs = _problems(case, seed)
    if kind == "rotations":
        return _exact_rotations(case, probs, seed, dev)
    if kind in ("batch", "pairs"):
        E, G = torch.zeros(len(probs), dtype=torch.float64, device=dev), [None] * len(probs)
        for n, ne in sorted({(p[0], p[1]) for p in probs}):
            idx = [i for i, p in enumerate(probs) if (p[0], p[1]) == (n, ne)]
            part = [probs[i] for i in idx]
            if kind == "pairs":
                sp = _Space(n, lambda b: _count(b, (1 << n) - 1) == ne, dev)
                gates = [((i, a), (a - ne) * ne + i, 1.0) for a in range(ne, n) for i in range(ne)]
                moves, m = [sp.move(e[:1], e[1:], signs=False) for e, _, _ in gates], len(gates)
            else:
                sp = _fermion_space(n, ne, dev)
                gates, m = _excitations(n, ne, case["ansatz"])
                moves = [sp.move(e[:len(e) // 2], e[len(e) // 2:]) for e, _, _ in gates]
            apply_h = _pairs_apply if kind == "pairs" else _h_apply
            _, e, g = _evaluate(sp, part, gates, moves, lambda v: apply_h(sp, n, part, v), True, m)
            E[torch.tensor(idx, device=dev)] = e
            for i, row in zip(idx, g):
                G[i] = row
        return {"energy": E.cpu().numpy(), "gradient": torch.cat(G).cpu().numpy()}
    n, ne = probs[0][0], probs[0][1]
    sp = _fermion_space(n, ne, dev)
    ansatz = case.get("ansatz", "uccsd")
    gates, m = _excitations(n, ne, ansatz)
    pool = gates
    if kind == "pool":
        gates = [(gates[k][0], j, 1.0) for j, k in enumerate(_pool_choice(case, seed))]
        m = len(gates)
    moves = [sp.move(e[:len(e) // 2], e[len(e) // 2:]) for e, _, _ in gates]
    apply_h = lambda v: _h_apply(sp, n, probs, v)  # noqa: E731
    if kind == "single":
        _, e, g = _evaluate(sp, probs, gates, moves, apply_h, case["grad"], m)
        return {"energy": float(e[0]), "gradient": g[0].cpu().numpy()} if case["grad"] else {"energy": float(e[0])}
    psi, e, _ = _evaluate(sp, probs, gates, moves, apply_h, False, m)
    if kind == "state":
        full = torch.zeros(1 << n, dtype=torch.complex128, device=dev)
        full[sp.bits] = psi[0].to(torch.complex128)
        return {"energy": float(e[0]), "psi": full.cpu().numpy()}
    lam, g = apply_h(psi), []
    for exc, _, _ in pool:
        src, dst, sg = sp.move(exc[:len(exc) // 2], exc[len(exc) // 2:])
        g.append(2 * (sg * (lam[:, dst] * psi[:, src] - lam[:, src] * psi[:, dst])).sum())
    return {"energy": float(e[0]), "gradient": torch.stack(g).cpu().numpy()}
