"""The work this framework is timed on: calls of its public entry points over
the range of sizes they serve.

A case names a program family and its sizes. `prepare` loads the program(s)
into a context, as a user does once; `run` is one library call; `exact`
evaluates the same program with a plain batched torch state vector in complex128.

Families (the circuit shapes of the repository's benchmark):
  dynamic  layers of U on every qubit and CX pairs, measure / if / reset sites
           on the way, final measure-all (complex128, complex64, or with
           depolarizing noise per shot)
  state    the same without measurements: one shot, its state vector returned
  rus      random layers, then a repeat-until-success loop, measure-all; shots
           with equal histories share one state
  batch    many different rus circuits, some shots each, in one call
  energy   <H> of a hardware-efficient ansatz over a batch of parameter vectors
  grad     the same with the adjoint gradient
"""
import math

import numpy as np
import torch

from paper_2604_11599_amd import Context

TWO_PI = 2.0 * math.pi


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def _dyn(name, n, layers, sites, shots, c64=False, noise=0.0):
    return {"name": name, "kind": "dynamic", "n": n, "layers": layers, "sites": sites, "shots": shots, "c64": c64,
            "noise": noise}


def listed():
    return [
        # one shot of a protocol-sized program: the latency of a call
        _dyn("shots_3q_1", 3, 2, 1, 1),
        # a small test circuit with an odd shot count
        _dyn("shots_7q_257", 7, 11, 2, 257),
        # the usual validation run: 10 qubits, three feed-forward sites, 1000 shots
        _dyn("shots_10q_1000", 10, 20, 3, 1000),
        # the same under depolarizing noise, every shot with its own matrices
        _dyn("noisy_10q_1000", 10, 20, 3, 1000, noise=1e-3),
        # repeat-until-success, shared trajectories
        {"name": "rus_16q_1024", "kind": "rus", "n": 16, "layers": 12, "iters": 8, "shots": 1024},
        # the state vector of a circuit, for comparison with another simulator
        {"name": "state_20q", "kind": "state", "n": 20, "layers": 24},
        # wide circuits, every shot its own state
        _dyn("shots_24q_4", 24, 40, 4, 4),
        # the same in single precision
        _dyn("c64_25q_8", 25, 40, 4, 8, c64=True),
        # the headline width
        _dyn("shots_28q_4", 28, 40, 4, 4),
        # a queue of different circuits of 12 to 18 qubits, 16 shots each
        {"name": "batch_24", "kind": "batch", "n_lo": 12, "n_hi": 18, "count": 24, "layers": 12, "iters": 8,
         "shots": 16},
        # a line search of a variational run: energies alone, odd width
        {"name": "energy_17q_32", "kind": "energy", "n": 17, "layers": 6, "terms": 60, "batch": 32},
        # a gradient step of a variational run
        {"name": "grad_20q_64", "kind": "grad", "n": 20, "layers": 6, "terms": 60, "batch": 64},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["dynamic", "dynamic", "dynamic", "c64", "noise", "rus", "state", "batch", "energy", "grad"])
    if kind in ("dynamic", "c64"):
        n = rng.randint(3, 26)
        top = max(1, min(3000, (1 << 28) >> n))
        return {"kind": "dynamic", "n": n, "layers": rng.randint(4, 40), "sites": rng.randint(1, 4),
                "shots": log_int(1, top), "c64": kind == "c64", "noise": 0.0}
    if kind == "noise":
        n = rng.randint(3, 12)
        return {"kind": "dynamic", "n": n, "layers": rng.randint(4, 20), "sites": rng.randint(1, 3),
                "shots": log_int(16, 1000), "c64": False, "noise": rng.choice([1e-4, 1e-3, 1e-2])}
    if kind == "rus":
        return {"kind": "rus", "n": rng.randint(8, 17), "layers": rng.randint(4, 12), "iters": rng.randint(2, 8),
                "shots": log_int(64, 1024)}
    if kind == "state":
        return {"kind": "state", "n": rng.randint(5, 22), "layers": rng.randint(4, 40)}
    if kind == "batch":
        lo = rng.randint(6, 15)
        return {"kind": "batch", "n_lo": lo, "n_hi": lo + rng.randint(0, 3), "count": rng.randint(3, 24),
                "layers": rng.randint(4, 12), "iters": rng.randint(2, 8), "shots": rng.randint(1, 24)}
    n = rng.randint(6, 20)
    return {"kind": kind, "n": n, "layers": rng.randint(2, 6), "terms": rng.randint(10, 80),
            "batch": log_int(1, min(128, (1 << 26) >> n))}


# ---------------------------------------------------------------------------
# Programs as lists of statements: ("U", q, (a, b, c)), ("x", q), ("cx", a, b),
# ("rx" | "ry" | "rz", q, angle or parameter index), ("measure", q, bit),
# ("reset", q), ("if", (first bit, width, value), body, other),
# ("rus", q, bit, tries, body)
# ---------------------------------------------------------------------------
def _u(rng, q):
    return ("U", q, tuple(float(x) for x in rng.random(3) * TWO_PI))


def _brick(rng, n, layer):
    ops = [_u(rng, q) for q in range(n)]
    return ops + [("cx", a, a + 1) for a in range(layer % 2, n - 1, 2)]


def _matched(rng, n):
    perm = [int(x) for x in rng.permutation(n)]
    return [_u(rng, q) for q in range(n)] + [("cx", perm[2 * k], perm[2 * k + 1]) for k in range(n // 2)]


def _dynamic_ops(rng, n, layers, sites):
    """Up to 12 qubits: random pairs and a measure / if x / reset site after
    every few layers. Wider: brickwork, one site measuring `sites` qubits, an
    if on the register's value and an if/else on one bit. Then measure-all."""
    ops = []
    if n <= 12:
        at = {(k + 1) * layers // (sites + 1): k for k in range(sites)}
        for layer in range(1, layers + 1):
            ops += _matched(rng, n)
            if layer in at:
                m = int(rng.integers(n))
                r = (m + 1 + int(rng.integers(n - 1))) % n
                ops += [("measure", m, at[layer]), ("if", (at[layer], 1, 1), [("x", r)], []), ("reset", m)]
    else:
        for layer in range(layers):
            ops += _brick(rng, n, layer)
        mq = [int(x) for x in rng.choice(n, size=sites, replace=False)]
        ops += [("measure", q, i) for i, q in enumerate(mq)]
        a, b = (int(x) for x in rng.choice(n, size=2, replace=False))
        ops += [("if", (0, sites, 10 % (1 << sites)), [_u(rng, int(rng.integers(n))), ("cx", a, b),
                                                       _u(rng, int(rng.integers(n)))], [])]
        r, t = int(rng.integers(n)), float(rng.random() * TWO_PI)
        ops += [("if", (0, 1, 1), [("rx", r, t)], [("rz", r, t)])]
    return ops + [("measure", q, sites + q) for q in range(n)]


def _rus_ops(rng, n, layers, iters):
    a = int(rng.integers(n))
    ops = []
    for _ in range(layers):
        ops += _matched(rng, n)
    ops += [("rus", a, 0, iters, _matched(rng, n) + _matched(rng, n))]
    return ops + [("measure", q, 1 + q) for q in range(n)]


def _ansatz_ops(n, layers):
    ops = []
    for layer in range(layers):
        ops += [("ry", q, 2 * n * layer + q) for q in range(n)]
        ops += [("rz", q, 2 * n * layer + n + q) for q in range(n)]
        ops += [("cx", q, q + 1) for q in range(n - 1)]
    return ops


def _qasm(n, sites, ops, params=0):
    """OpenQASM 3 text of a statement list; its classical bits are a register c
    of the sites' bits, then, where there are any, f of the final measurement's."""
    def ang(x):
        return f"theta[{x}]" if isinstance(x, int) else repr(x)

    def bit(i):
        return f"c[{i}]" if i < sites else f"f[{i - sites}]"

    def line(op):
        if op[0] == "U":
            return f"U({', '.join(repr(x) for x in op[2])}) q[{op[1]}];"
        if op[0] in ("rx", "ry", "rz"):
            return f"{op[0]}({ang(op[2])}) q[{op[1]}];"
        if op[0] == "x":
            return f"x q[{op[1]}];"
        if op[0] == "cx":
            return f"cx q[{op[1]}], q[{op[2]}];"
        if op[0] == "measure":
            return f"{bit(op[2])} = measure q[{op[1]}];"
        if op[0] == "reset":
            return f"reset q[{op[1]}];"
        if op[0] == "if":
            lo, width, value = op[1]
            cond = f"c == {value}" if width > 1 else f"{bit(lo)} == {value}"
            other = " else { " + " ".join(map(line, op[3])) + " }" if op[3] else ""
            return f"if ({cond}) {{ " + " ".join(map(line, op[2])) + " }" + other
        _, a, flag, tries, body = op
        return (f"for uint i in [0:{tries - 1}] {{\n  {bit(flag)} = measure q[{a}];\n  if ({bit(flag)} == 0) break;\n"
                f"  reset q[{a}];\n  " + "\n  ".join(map(line, body)) + "\n}")

    head = ["OPENQASM 3.0;", 'include "stdgates.inc";']
    head += [f"input array[float[64], {params}] theta;"] if params else []
    head += [f"qubit[{n}] q;"] + ([f"bit[{sites}] c;", f"bit[{n}] f;"] if sites else [])
    return "\n".join(head + [line(op) for op in ops]) + "\n"


def _programs(case, seed):
    """(n, site bits, statements) of every program of the case."""
    rng = np.random.default_rng([seed, 7])
    k = case["kind"]
    if k == "dynamic":
        return [(case["n"], case["sites"], _dynamic_ops(rng, case["n"], case["layers"], case["sites"]))]
    if k == "state":
        return [(case["n"], 0, [op for layer in range(case["layers"]) for op in _brick(rng, case["n"], layer)])]
    if k == "rus":
        return [(case["n"], 1, _rus_ops(rng, case["n"], case["layers"], case["iters"]))]
    if k == "batch":
        widths = [case["n_lo"] + i % (case["n_hi"] - case["n_lo"] + 1) for i in range(case["count"])]
        return [(n, 1, _rus_ops(rng, n, case["layers"], case["iters"])) for n in widths]
    return [(case["n"], 0, _ansatz_ops(case["n"], case["layers"]))]


def _vqe_inputs(case, seed):
    """A random 2-local Pauli sum (N(0, 1) coefficients) and parameter vectors."""
    rng = np.random.default_rng([seed, 8])
    n, terms = case["n"], case["terms"]
    codes = np.zeros((terms, n), dtype=np.uint8)
    for t in range(terms):
        a, b = rng.choice(n, size=2, replace=False)
        codes[t, a], codes[t, b] = rng.integers(1, 4), rng.integers(1, 4)
    return (rng.standard_normal(terms), codes,
            rng.uniform(-math.pi, math.pi, size=(case["batch"], 2 * n * case["layers"])))


def prepare(case, seed):
    ctx = Context(0)
    state = {"kind": case["kind"], "ctx": ctx, "seed": seed}
    if case["kind"] in ("energy", "grad"):
        n = case["n"]
        state["prog"] = ctx.load(_qasm(n, 0, _programs(case, seed)[0][2], params=2 * n * case["layers"]))
        state["coeffs"], state["codes"], state["thetas"] = _vqe_inputs(case, seed)
        return state
    progs = [ctx.load(_qasm(*p), noise=case.get("noise", 0.0) > 0.0) for p in _programs(case, seed)]
    if case["kind"] == "batch":
        state["requests"] = [{"prog": p, "shots": case["shots"], "seed": seed * 1000 + i} for i, p in enumerate(progs)]
        return state
    state["prog"] = progs[0]
    state["shots"] = case.get("shots", 1)
    state["opts"] = {"complex64": case.get("c64", False), "depolarizing": case.get("noise", 0.0),
                     "share": case["kind"] == "rus", "state_out": case["kind"] == "state"}
    return state


def _shot_outputs(r):
    return {"creg": r.creg.view(np.int64), "record": r.record, "n_events": r.n_events.astype(np.int64),
            "record_prob": r.record_prob, "status": r.shot_status}


def _side_by_side(outs):
    """The outputs of many programs, each kind in one array."""
    return {k: None if outs[0][k] is None else np.concatenate([o[k].ravel() for o in outs]) for k in outs[0]}


def run(state):
    k = state["kind"]
    if k == "energy":
        return state["prog"].expval(state["thetas"], state["coeffs"], state["codes"])
    if k == "grad":
        return state["prog"].expval_grad(state["thetas"], state["coeffs"], state["codes"])
    if k == "batch":
        return _side_by_side([_shot_outputs(r) for r in state["ctx"].run_batch(state["requests"])])
    r = state["prog"].run_shots(state["shots"], seed=state["seed"], **state["opts"])
    return r.state if k == "state" else _shot_outputs(r)


# ---------------------------------------------------------------------------
# Work: 14 flops per amplitude for a complex 2x2 product, and the state written
# once and read once (the measurement, the Hamiltonian, or the caller's copy)
# ---------------------------------------------------------------------------
def _rotations(ops):
    return sum(1 if op[0] in ("U", "rx", "ry", "rz") else _rotations(op[4]) / 2 if op[0] == "rus" else 0 for op in ops)


def work(case):
    by = fl = 0.0
    shots = case.get("shots", 1) * case.get("batch", 1)
    for n, _, ops in _programs(case, 0):
        amps = float(1 << n) * shots
        factor = 3.0 if case["kind"] == "grad" else 1.0  # forward, and psi and lambda back
        fl += 14.0 * _rotations(ops) * amps * factor
        by += (8.0 if case.get("c64") else 16.0) * amps * 2.0 * factor
    return {"bytes": by, "flops": fl}


# ---------------------------------------------------------------------------
# Plain evaluation in complex128
# ---------------------------------------------------------------------------
def _mulhi(a, b):
    m = np.uint64(0xFFFFFFFF)
    s = np.uint64(32)
    a0, a1, b0, b1 = a & m, a >> s, b & m, b >> s
    t = a1 * b0 + ((a0 * b0) >> s)
    return a1 * b1 + (t >> s) + ((a0 * b1 + (t & m)) >> s)


def _uniform(seed, shots, counter, word):
    """Uniforms of Philox4x64-10: one counter (4 arrays) and word per shot."""
    with np.errstate(over="ignore"):
        k0 = np.full(shots, seed, dtype=np.uint64)
        k1 = np.arange(shots, dtype=np.uint64)
        c = [np.broadcast_to(np.asarray(x, dtype=np.uint64), (shots,)).copy() for x in counter]
        m0, m1 = np.uint64(0xD2E7470EE14C6C93), np.uint64(0xCA5A826395121157)
        for _ in range(10):
            h0, l0, h1, l1 = _mulhi(c[0], m0), c[0] * m0, _mulhi(c[2], m1), c[2] * m1
            c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
            k0, k1 = k0 + np.uint64(0x9E3779B97F4A7C15), k1 + np.uint64(0xBB67AE8584CAA73B)
    w = np.stack(c)[np.asarray(word), np.arange(shots)]
    return (w >> np.uint64(11)).astype(np.float64) * 2.0 ** -53


def _pair(psi, n, q):
    v = psi.view(psi.shape[0], 1 << (n - 1 - q), 2, 1 << q)
    return v[:, :, 0], v[:, :, 1]


def _apply(psi, n, q, m, mask=None):
    """The 2x2 matrix m (numbers, or one per state) on qubit q, in place."""
    a, b = _pair(psi, n, q)
    col = [x if not torch.is_tensor(x) else x.view(-1, 1, 1) for x in m]
    x0, x1 = col[0] * a + col[1] * b, col[2] * a + col[3] * b
    if mask is not None:
        x0, x1 = torch.where(mask.view(-1, 1, 1), x0, a), torch.where(mask.view(-1, 1, 1), x1, b)
    a.copy_(x0)
    b.copy_(x1)


def _cx(psi, n, c, t, mask=None):
    hi, lo = max(c, t), min(c, t)
    v = psi.view(psi.shape[0], 1 << (n - 1 - hi), 2, 1 << (hi - lo - 1), 2, 1 << lo)
    a, b = (v[:, :, 1, :, 0], v[:, :, 1, :, 1]) if c == hi else (v[:, :, 0, :, 1], v[:, :, 1, :, 1])
    x, y = a.clone(), b.clone()
    if mask is not None:
        mk = mask.view(-1, 1, 1, 1)
        x, y = torch.where(mk, x, y), torch.where(mk, y, x)
    a.copy_(y)
    b.copy_(x)


def _matrix(op):
    if op[0] == "x":
        return 0.0, 1.0, 1.0, 0.0
    if op[0] == "U":
        t, p, l = op[2]
        c, s = math.cos(t / 2), math.sin(t / 2)
        ex = lambda a: complex(math.cos(a), math.sin(a))  # noqa: E731
        return c, -ex(l) * s, ex(p) * s, ex(p + l) * c
    c, s = math.cos(op[2] / 2), math.sin(op[2] / 2)
    return {"rx": (c, -1j * s, -1j * s, c), "ry": (c, -s, s, c), "rz": (complex(c, -s), 0.0, 0.0, complex(c, s))}[op[0]]


class _Shots:
    """Every shot of one program side by side, psi [shots, 2^n]."""

    def __init__(self, n, sites, shots, seed, noise=0.0):
        self.n, self.shots, self.seed, self.noise = n, shots, seed, noise
        self.psi = torch.zeros(shots, 1 << n, dtype=torch.complex128, device="cuda")
        self.psi[:, 0] = 1.0
        self.bits = np.zeros((shots, sites + n), dtype=np.int64)
        self.events = np.zeros(shots, dtype=np.int64)
        self.prob = np.ones(shots)
        self.statement = 0

    def _mask(self, act):
        return None if act.all() else torch.from_numpy(act).cuda()

    def _project(self, q, act, flip):
        u = _uniform(self.seed, self.shots, (self.events // 4 + 1, 0, 0, 0), self.events % 4)
        a, b = _pair(self.psi, self.n, q)
        p0 = (a.real ** 2 + a.imag ** 2).sum((1, 2)).cpu().numpy()
        p1 = (b.real ** 2 + b.imag ** 2).sum((1, 2)).cpu().numpy()
        one = u >= p0 / (p0 + p1)
        p = np.where(one, p1, p0)
        scale = 1.0 / np.sqrt(p)
        k0, k1 = (torch.from_numpy(np.where(act, np.where(o, scale, 0.0), 1.0)).cuda().view(-1, 1, 1)
                  for o in (~one, one))
        a.mul_(k0)
        b.mul_(k1)
        self.prob = np.where(act, self.prob * (p / (p0 + p1)), self.prob)
        self.events = self.events + act
        if flip and (act & one).any():
            _apply(self.psi, self.n, q, _matrix(("x",)), torch.from_numpy(act & one).cuda())
        return one

    def _depolarize(self, qubits, act):
        for k, q in enumerate(qubits):
            u = _uniform(self.seed, self.shots, (self.statement, 0, k, 1), np.zeros(self.shots, dtype=np.int64))
            for i, m in enumerate([(0.0, 1.0, 1.0, 0.0), (0.0, -1j, 1j, 0.0), (1.0, 0.0, 0.0, -1.0)]):
                hit = act & (u >= i * self.noise / 3.0) & (u < (i + 1) * self.noise / 3.0)
                if hit.any():
                    _apply(self.psi, self.n, q, m, torch.from_numpy(hit).cuda())

    def run(self, ops, act=None):
        act = np.ones(self.shots, dtype=bool) if act is None else act
        for op in ops:
            if op[0] in ("U", "x", "rx", "ry", "rz", "cx"):
                if act.any():
                    if op[0] == "cx":
                        _cx(self.psi, self.n, op[1], op[2], self._mask(act))
                    else:
                        _apply(self.psi, self.n, op[1], _matrix(op), self._mask(act))
                    if self.noise:
                        self._depolarize(op[1:3] if op[0] == "cx" else op[1:2], act)
                self.statement += 1
            elif op[0] == "measure":
                one = self._project(op[1], act, False)
                self.bits[act, op[2]] = one[act]
            elif op[0] == "reset":
                self._project(op[1], act, True)
            elif op[0] == "if":
                lo, width, value = op[1]
                hit = (self.bits[:, lo:lo + width] == [(value >> i) & 1 for i in range(width)]).all(1)
                self.run(op[2], act & hit)
                self.run(op[3], act & ~hit)
            else:
                _, a, bit, tries, body = op
                live = act.copy()
                for _ in range(tries):
                    if not live.any():
                        break
                    self.run([("measure", a, bit)], live)
                    live &= self.bits[:, bit] == 1
                    if live.any():
                        self.run([("reset", a)] + body, live)
        return self


def _rotation(kind, t):
    """Matrices of ry / rz for angles t [batch], as four tensors."""
    c, s, z = torch.cos(t / 2), torch.sin(t / 2), torch.zeros_like(t)
    if kind == "ry":
        return [torch.complex(x, z) for x in (c, -s, s, c)]
    zero = torch.complex(z, z)
    return [torch.complex(c, -s), zero, zero, torch.complex(c, s)]


def _hamiltonian(psi, n, coeffs, codes):
    i = torch.arange(1 << n, device="cuda")
    out = torch.zeros_like(psi)
    for c, row in zip(coeffs, codes):
        x = sum(1 << q for q in range(n) if row[q] in (1, 2))
        z = [q for q in range(n) if row[q] in (2, 3)]
        sign = torch.ones(1 << n, dtype=torch.float64, device="cuda")
        for q in z:  # of the source index i ^ x
            sign = sign * (1.0 - 2.0 * (((i ^ x) >> q) & 1).to(torch.float64))
        out += psi[:, i ^ x] * (sign * (c * 1j ** int(np.sum(row == 2))))
    return out


def _vqe(case, seed):
    coeffs, codes, thetas = _vqe_inputs(case, seed)
    n, ops = case["n"], _ansatz_ops(case["n"], case["layers"])
    th = torch.from_numpy(thetas).cuda()
    psi = torch.zeros(len(thetas), 1 << n, dtype=torch.complex128, device="cuda")
    psi[:, 0] = 1.0
    for op in ops:
        if op[0] == "cx":
            _cx(psi, n, op[1], op[2])
        else:
            _apply(psi, n, op[1], _rotation(op[0], th[:, op[2]]))
    lam = _hamiltonian(psi, n, coeffs, codes)
    energy = (psi.real * lam.real + psi.imag * lam.imag).sum(1).cpu().numpy()
    if case["kind"] == "energy":
        return energy
    grad = np.zeros(thetas.shape)
    for op in reversed(ops):
        if op[0] == "cx":
            _cx(psi, n, op[1], op[2])
            _cx(lam, n, op[1], op[2])
            continue
        # dE = 2 Re <lambda| (-i P / 2) |psi> with both after the rotation
        (a, b), (la, lb) = _pair(psi, n, op[1]), _pair(lam, n, op[1])
        if op[0] == "ry":
            v = (la.conj() * b - lb.conj() * a).sum((1, 2)) * -0.5
        else:
            v = (la.conj() * a - lb.conj() * b).sum((1, 2)) * -0.5j
        grad[:, op[2]] = 2.0 * v.real.cpu().numpy()
        for s in (psi, lam):
            _apply(s, n, op[1], _rotation(op[0], -th[:, op[2]]))
    return energy, grad


def exact(case, seed):
    if case["kind"] in ("energy", "grad"):
        return _vqe(case, seed)
    if case["kind"] == "dynamic" and case["shots"] << case["n"] > 1 << 28:
        return None  # about a minute of plain gates
    out = []
    for i, (n, sites, ops) in enumerate(_programs(case, seed)):
        key = seed * 1000 + i if case["kind"] == "batch" else seed
        s = _Shots(n, sites, case.get("shots", 1), key, case.get("noise", 0.0)).run(ops)
        if case["kind"] == "state":
            return s.psi[0].cpu().numpy()
        out.append({"creg": None, "record": None, "n_events": None, "record_prob": s.prob, "status": None})
    return _side_by_side(out)
