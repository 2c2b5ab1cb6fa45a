"""Measured workloads of the library, through the entry points that a program calls.

Each case is a dict of plain values; ``kind`` names the path:

* ``rref``      GF(2) elimination of a matrix, optionally with its transform;
* ``pauli``     commutation table of a set of Pauli strings;
* ``evaluate``  parameterized evaluation: two parity products, then the phase-pair product;
* ``single``    one diagram simplified and read back (latency);
* ``batch``     a prepared batch of diagrams simplified in one launch, greedy or learned;
* ``sample``    detector sampling;
* ``train``     one optimiser step of the scoring network;
* ``extract``   flow layers and circuits of a batch of diagrams.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2604_01059_amd import zx

DEV = "cuda"
GATES = 1536  # room for the gates of one circuit of the extraction cases, on average


def listed():
    return [
        # the benchmark matrix: full-rank elimination, the largest one in use
        {"name": "rref 4096x16384", "kind": "rref", "m": 4096, "n_cols": 16384, "density": 0.5, "transform": False},
        # a parameter basis of a reduced diagram: small, ragged, with the row combinations
        {"name": "rref 300x1000 T", "kind": "rref", "m": 300, "n_cols": 1000, "density": 0.05, "transform": True},
        # the whole commutation table of the benchmark
        {"name": "pauli 65536x1024", "kind": "pauli", "n": 65536, "qubits": 1024},
        # amplitudes of a large compiled circuit for many parameter settings
        {"name": "evaluate 4096x65536", "kind": "evaluate", "terms": 4096, "settings": 65536, "params": 1024,
         "any_phase": False},
        # the same for a small circuit and a handful of thousand settings, sizes off every tile
        {"name": "evaluate 300x5000", "kind": "evaluate", "terms": 300, "settings": 5000, "params": 200,
         "any_phase": False},
        # interactive use: one diagram of 8 qubits and 64 spiders, result on the host
        {"name": "single 8q 64", "kind": "single", "qubits": 8, "per_qubit": 8, "density": 0.1},
        # the batched workload: 4096 uneven diagrams
        {"name": "batch 4096", "kind": "batch", "count": 4096, "q_lo": 4, "q_hi": 64, "m_lo": 4, "m_hi": 16,
         "learned": False},
        # one large diagram
        {"name": "batch 1 of 4160", "kind": "batch", "count": 1, "q_lo": 260, "q_hi": 260, "m_lo": 16, "m_hi": 16,
         "learned": False},
        # learned schedule over diagrams of 32 to 128 qubits (the proposal's evaluation set)
        {"name": "learned 512", "kind": "batch", "count": 512, "q_lo": 32, "q_hi": 128, "m_lo": 4, "m_hi": 16,
         "learned": True},
        # shots of a distance-7, 7-round memory experiment
        {"name": "sample d7 2^24", "kind": "sample", "d": 7, "rounds": 7, "p": 1e-3, "shots": 1 << 24},
        # a training step of the proposal network: 128 states of 16 candidates
        {"name": "train 128x16", "kind": "train", "states": 128, "per_state": 16},
        # circuits of 20 qubits out of their diagrams
        {"name": "extract 1024", "kind": "extract", "count": 1024, "qubits": 20, "depth": 21},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["rref", "rref", "pauli", "evaluate", "evaluate", "single", "batch", "batch", "learned",
                       "sample", "train", "extract"])
    if kind == "rref":
        m, n = _log_int(rng, 40, 4096), _log_int(rng, 64, 16384)
        # of a tall matrix the reduced rows alone say little: the row combinations are what is asked for
        return {"kind": kind, "m": m, "n_cols": n, "density": rng.choice([0.5, 0.5, 0.05]),
                "transform": n < m + 64 or rng.random() < 0.2}
    if kind == "pauli":
        return {"kind": kind, "n": _log_int(rng, 100, 65536), "qubits": _log_int(rng, 20, 1024)}
    if kind == "evaluate":
        return {"kind": kind, "terms": _log_int(rng, 20, 4096), "settings": _log_int(rng, 64, 65536),
                "params": _log_int(rng, 16, 1024), "any_phase": rng.random() < 0.25}
    if kind == "single":
        return {"kind": kind, "qubits": rng.randint(4, 32), "per_qubit": rng.randint(4, 16),
                "density": rng.uniform(0.05, 0.3)}
    if kind == "batch" and rng.random() < 0.3:
        q = rng.randint(100, 260)
        return {"kind": kind, "count": 1, "q_lo": q, "q_hi": q, "m_lo": 16, "m_hi": 16, "learned": False}
    if kind == "batch":
        q = rng.randint(8, 64)
        return {"kind": kind, "count": _log_int(rng, 16, 4096), "q_lo": 4, "q_hi": q, "m_lo": 4, "m_hi": 16,
                "learned": False}
    if kind == "learned":
        q = rng.randint(40, 128)
        return {"kind": "batch", "count": _log_int(rng, 16, 512), "q_lo": rng.randint(8, 32), "q_hi": q, "m_lo": 4,
                "m_hi": 16, "learned": True}
    if kind == "sample":
        return {"kind": kind, "d": rng.choice([3, 5, 7]), "rounds": rng.randint(1, 7),
                "p": 10.0 ** rng.uniform(-4.0, -2.3), "shots": _log_int(rng, 1000, 1 << 23)}
    if kind == "train":
        return {"kind": kind, "states": _log_int(rng, 4, 8192), "per_state": rng.choice([4, 8, 16, 16])}
    return {"kind": kind, "count": _log_int(rng, 16, 1024), "qubits": rng.randint(4, 20), "depth": rng.randint(4, 21)}


# ------------------------------------------------------------------- inputs --

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _pack(bits):
    """(rows, cols) bool -> (rows, ceil(cols / 64)) int64 words, bit c % 64 of word c // 64."""
    r, c = bits.shape
    w = (c + 63) // 64
    full = torch.zeros((r, w * 64), dtype=torch.bool, device=bits.device)
    full[:, :c] = bits
    out = torch.zeros((r, w), dtype=torch.int64, device=bits.device)
    v = full.view(r, w, 64)
    for b in range(64):
        out |= v[:, :, b].to(torch.int64) << b
    return out


def _unpack(words, c):
    r, w = words.shape
    shift = torch.arange(64, device=words.device)
    return ((words[:, :, None] >> shift) & 1).view(r, w * 64)[:, :c]


def _random_words(gen, rows, cols):
    """rows x cols bits, each 0 or 1 with equal probability (bits beyond cols zero)."""
    w = (cols + 63) // 64
    a = torch.randint(-2 ** 63, 2 ** 63 - 1, (rows, w), dtype=torch.int64, device=DEV, generator=gen)
    if cols % 64:
        a[:, -1] &= (1 << (cols % 64)) - 1
    return a


def _sparse_words(gen, rows, cols, p):
    return _pack(torch.rand((rows, cols), device=DEV, generator=gen) < p)


class _Diagram:
    """Host arrays of one random graph-like diagram: inputs on the first spiders, outputs on the last."""

    def __init__(self, adj, phase, q):
        n = adj.shape[0]
        self.adj, self.phase = adj, phase
        self.inputs = np.arange(q, dtype=np.int32)
        self.outputs = (n - q + np.arange(q)).astype(np.int32)


def _random_diagrams(gen, sizes):
    """Diagrams of (q, n, p) in ``sizes``: random Hadamard edges of density p, uniform phases k pi/4."""
    words, phases = [], []
    for q, n, p in sizes:
        up = torch.triu(torch.rand((n, n), device=DEV, generator=gen) < p, 1)
        words.append(_pack_rows(up | up.T).view(-1))
        phases.append(torch.randint(0, 8, (n,), dtype=torch.int8, device=DEV, generator=gen))
    words = torch.cat(words).cpu().numpy().view(np.uint64)
    phases = torch.cat(phases).cpu().numpy()
    out, a, b = [], 0, 0
    for q, n, _ in sizes:
        w = (n + 63) // 64
        out.append(_Diagram(words[a:a + n * w].reshape(n, w), phases[b:b + n], q))
        a, b = a + n * w, b + n
    return out


def _pack_rows(bits):
    """As _pack, through bytes (few launches, for many small matrices)."""
    n, c = bits.shape
    w = (c + 63) // 64
    full = torch.zeros((n, w * 64), dtype=torch.uint8, device=bits.device)
    full[:, :c] = bits
    weight = torch.tensor([1, 2, 4, 8, 16, 32, 64, 128], dtype=torch.uint8, device=bits.device)
    by = (full.view(n, w * 8, 8) * weight).sum(dim=2, dtype=torch.uint8)
    return by.view(torch.int64)


def _arenas(diagrams, bnd_is_h=None):
    """The diagrams' graphs, carved out of one allocation as a program with many of them does."""
    sizes = [(zx.Graph.bytes_for(d.adj.shape[0], len(d.inputs), len(d.outputs)) + 255) // 256 * 256
             for d in diagrams]
    pool = torch.zeros(sum(sizes), dtype=torch.uint8, device=DEV)
    graphs, off = [], 0
    for i, (d, nb) in enumerate(zip(diagrams, sizes)):
        graphs.append(zx.Graph.create(d.adj, d.phase, d.inputs, d.outputs, None if bnd_is_h is None else bnd_is_h[i],
                                      arena=pool[off:off + nb]))
        off += nb
    return pool, graphs


def _batch_sizes(case):
    """Sizes of a batch: the case's own, whatever the seed (which fills the diagrams)."""
    rng = np.random.default_rng(case["count"] * 1000 + case["q_hi"])
    q = rng.integers(case["q_lo"], case["q_hi"] + 1, case["count"])
    n = q * rng.integers(case["m_lo"], case["m_hi"] + 1, case["count"])
    p = rng.uniform(0.05, 0.3, case["count"])
    return [(int(a), int(b), float(c)) for a, b, c in zip(q, n, p)]


def _network(gen):
    """Glorot-uniform weights, zero biases: W1 | b1 | w2 | b2."""
    p = torch.zeros(zx.MLP_NPARAM, device=DEV)
    n1, h = zx.MLP_IN * zx.MLP_HID, zx.MLP_HID
    u = torch.rand(n1 + h, device=DEV, generator=gen) * 2 - 1
    p[:n1] = u[:n1] * math.sqrt(6.0 / (zx.MLP_IN + h))
    p[n1 + h:n1 + 2 * h] = u[n1:] * math.sqrt(6.0 / (h + 1))
    return p


def _surface_model(d, rounds, p, seed):
    """Error mechanisms shaped like a distance-d rotated surface-code memory experiment: neighbouring
    checks in space, boundary checks (one boundary flips the observable), checks in time, diagonals."""
    a, b = (d + 1) // 2, d - 1
    k = a * b
    obs = k * (rounds + 1)
    cols = []
    for r in range(rounds + 1):
        at = lambda x, y, s=r: s * k + x * b + y  # noqa: E731
        cols += [[at(x, y), at(x, y + 1)] for x in range(a) for y in range(b - 1)]
        cols += [[at(x, y), at(x + 1, y)] for x in range(a - 1) for y in range(b)]
        cols += [c for x in range(a) for c in ([at(x, 0), obs], [at(x, b - 1)])]
        if r < rounds:
            cols += [[r * k + c, (r + 1) * k + c] for c in range(k)]
            cols += [[at(x, y), at(x + 1, y + 1, r + 1)] for x in range(a - 1) for y in range(b - 1)]
    ptr = np.cumsum([0] + [len(c) for c in cols])
    prob = p * np.random.default_rng(seed).uniform(0.5, 1.5, len(cols))
    return ptr, np.array([i for c in cols for i in c]), prob, obs + 1


def _circuit_diagram(rng, q, depth):
    """Diagram of a random circuit: per layer a Z rotation and Hadamard on half the qubits, and CZ gates on
    random pairs (Hadamard edges between the qubits' current spiders)."""
    cur, phase, edges = list(range(q)), [0] * q, set()
    for _ in range(depth):
        for v in rng.choice(q, q // 2, replace=False):
            phase[cur[v]] = (phase[cur[v]] + int(rng.integers(8))) % 8
            edges.add((cur[v], len(phase)))
            cur[v] = len(phase)
            phase.append(0)
        for _ in range(max(1, q // 4)):
            x, y = rng.choice(q, 2, replace=False)
            edges ^= {(min(cur[x], cur[y]), max(cur[x], cur[y]))}
    for v in range(q):  # every qubit ends on a spider of its own
        edges.add((cur[v], len(phase)))
        cur[v] = len(phase)
        phase.append(0)
    n = len(phase)
    bits = np.zeros((n, (n + 63) // 64 * 64), np.uint8)
    e = np.array(sorted(edges))
    bits[e[:, 0], e[:, 1]] = bits[e[:, 1], e[:, 0]] = 1
    d = _Diagram(np.packbits(bits, axis=1, bitorder="little").view(np.uint64), np.array(phase, np.int8), q)
    d.outputs = np.array(cur, np.int32)
    return d, np.array([0] * q + [1] * q, np.uint8)


# ------------------------------------------------------------------ prepare --

def prepare(case, seed):
    kind, g = case["kind"], _gen(seed)
    s = {"kind": kind, "case": case}
    if kind == "rref":
        m, n = case["m"], case["n_cols"]
        s["A"] = _random_words(g, m, n) if case["density"] == 0.5 else _sparse_words(g, m, n, case["density"])
        s["R"] = torch.zeros_like(s["A"])
        s["rank"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        s["pivots"] = torch.zeros(m, dtype=torch.int32, device=DEV)
        s["T"] = torch.zeros((m, (m + 63) // 64), dtype=torch.int64, device=DEV) if case["transform"] else None
        s["ws"] = torch.empty(zx.gf2_workspace_bytes(m, n), dtype=torch.uint8, device=DEV)
    elif kind == "pauli":
        n, q = case["n"], case["qubits"]
        s["X"], s["Z"] = _random_words(g, n, q), _random_words(g, n, q)
        s["C"] = torch.zeros((n, (n + 63) // 64), dtype=torch.int64, device=DEV)
    elif kind == "evaluate":
        t, l, p = case["terms"], case["settings"], case["params"]
        s["U"], s["V"] = _sparse_words(g, t, p, 1 / 16), _sparse_words(g, t, p, 1 / 16)
        s["F"] = _random_words(g, l, p)
        if case["any_phase"]:
            s["ka"] = torch.randint(0, 8, (t,), dtype=torch.int8, device=DEV, generator=g)
            s["kb"] = torch.randint(0, 8, (t,), dtype=torch.int8, device=DEV, generator=g)
        else:  # the two kinds of terms that the rules leave: half-pi terms and pairs of pi terms
            s["ka"] = 4 * torch.randint(0, 2, (t,), dtype=torch.int8, device=DEV, generator=g)
            s["kb"] = 4 * torch.randint(0, 2, (t,), dtype=torch.int8, device=DEV, generator=g)
            half = torch.rand(t, device=DEV, generator=g) < 0.5
            s["kb"][half] = 2
            s["V"][half] = 0
        w = (l + 63) // 64
        s["a"], s["b"] = (torch.zeros((t, w), dtype=torch.int64, device=DEV) for _ in range(2))
        s["mant"] = torch.zeros((l, 2), device=DEV)
        s["expo"] = torch.zeros(l, dtype=torch.int32, device=DEV)
    elif kind == "single":
        q, n = case["qubits"], case["qubits"] * case["per_qubit"]
        s["graphs"] = _arenas(_random_diagrams(g, [(q, n, case["density"])]))[1]
        s["ws"] = torch.empty(zx.simplify_workspace_bytes(1), dtype=torch.uint8, device=DEV)
    elif kind == "batch":
        s["pool"], graphs = _arenas(_random_diagrams(g, _batch_sizes(case)))
        s["batch"] = zx.Batch(graphs)
        s["mlp"] = zx.MLP(_network(g)) if case["learned"] else None
    elif kind == "sample":
        s["sampler"] = zx.DetectorSampler(*_surface_model(case["d"], case["rounds"], case["p"], seed))
        s["seed"] = seed
        s["out"] = torch.zeros((case["shots"], (s["sampler"].n_f + 63) // 64), dtype=torch.int64, device=DEV)
    elif kind == "train":
        rows = case["states"] * case["per_state"]
        s["mlp"] = zx.MLP(_network(g))
        x = torch.rand((rows, zx.MLP_IN), device=DEV, generator=g)
        x[:, 1:4] = (x[:, 1:4] > 0.5).float()
        x[:, 7:14] = 0.0  # one endpoint: candidates of a local-complementation round
        x[:, 14], x[:, 15] = 0.0, 1.0
        s["x"] = x.to(torch.bfloat16).view(torch.int16)
        s["cost"] = torch.randint(0, 40, (rows,), dtype=torch.int64, device=DEV, generator=g)
        s["cost"][torch.rand(rows, device=DEV, generator=g) < 0.1] = -1
        s["seg"] = torch.arange(0, rows + 1, case["per_state"], dtype=torch.int32, device=DEV)
        s["ws"] = torch.empty(zx.load().zx_mlp_workspace_bytes(rows), dtype=torch.uint8, device=DEV)
    elif kind == "extract":
        rng = np.random.default_rng(seed)
        made = [_circuit_diagram(rng, case["qubits"], case["depth"]) for _ in range(case["count"])]
        s["pool"], s["graphs"] = _arenas([d for d, _ in made], [h for _, h in made])
        zx.simplify(s["graphs"])
        s["gates"] = np.zeros(case["count"] * GATES, np.int32)
    else:
        raise ValueError(kind)
    return s


# ---------------------------------------------------------------------- run --

def run(s):
    kind = s["kind"]
    if kind == "rref":
        zx.gf2_eliminate(s["A"], R=s["R"], n_cols=s["case"]["n_cols"], rank=s["rank"], pivots=s["pivots"],
                         ws=s["ws"], T=s["T"])
        out = {"R": s["R"], "rank": s["rank"], "pivots": s["pivots"]}
        return out if s["T"] is None else dict(out, T=s["T"])
    if kind == "pauli":
        return zx.pauli_commute(s["X"], s["Z"], s["case"]["qubits"], C_out=s["C"])
    if kind == "evaluate":
        zx.gf2_matmul(s["U"], s["F"], s["case"]["params"], C_out=s["a"])
        zx.gf2_matmul(s["V"], s["F"], s["case"]["params"], C_out=s["b"])
        zx.phase_pair_product(s["a"], s["b"], s["ka"], s["kb"], s["case"]["settings"], mant=s["mant"],
                              expo=s["expo"])
        return {"a": s["a"], "b": s["b"], "mant": s["mant"], "expo": s["expo"]}
    if kind == "single":
        graph = s["graphs"][0]
        zx.simplify(s["graphs"], ws=s["ws"])
        adj, phase, alive, info = graph.read()
        rows, pivots = graph.frontier()
        return {"adj": adj.view(np.int64), "phase": phase, "alive": alive.view(np.int64), "rows": rows.view(np.int64),
                "pivots": pivots, "scalar": [info.pow_sqrt2, info.phase8],
                "counts": [info.status, info.n_alive, info.n_edges, info.rounds, info.fill_in, info.rank, info.rowops]}
    if kind == "batch":
        if s["mlp"] is not None:
            s["batch"].run(policy=zx.ZX_POLICY_LEARNED, mlp=s["mlp"])
        else:
            s["batch"].run()
        return s["pool"]  # every diagram's result, trace and frontier
    if kind == "sample":
        return s["sampler"].sample(s["seed"], 0, s["case"]["shots"], out=s["out"])
    if kind == "train":
        mlp = s["mlp"]
        score = mlp.forward(s["x"])
        dscore, loss = mlp.loss(score, s["cost"], s["seg"])
        grad = mlp.backward(s["x"], dscore, ws=s["ws"])
        mlp.adam(lr=1e-3)
        return {"score": score, "loss": loss, "dscore": dscore, "grad": grad, "param": mlp.param, "m": mlp.m,
                "v": mlp.v}
    exists, layers = zx.gflow(s["graphs"])
    circuits = zx.extract(s["graphs"], raw=True)
    gates = np.concatenate([c[1] for c in circuits]).view(np.int32)
    s["gates"][len(gates):] = 0  # a place of fixed size for all circuits, one after the other
    s["gates"][:len(gates)] = gates
    return {"exists": exists, "layers": np.concatenate(layers), "status": np.array([c[0] for c in circuits]),
            "length": np.array([len(c[1]) for c in circuits]), "gates": s["gates"],
            "perm": np.concatenate([c[2] for c in circuits])}


# --------------------------------------------------------------------- work --

def _arena_traffic(n, q):
    w = (n + 63) // 64
    return 2 * n * w * 8 + 2 * n + 8 * w + q * w * 8 + 16 * n  # source in, result, trace and frontier out


def work(case):
    """Inputs read once, outputs written once; a bit product counts as a multiplication and an addition."""
    kind = case["kind"]
    if kind == "rref":
        m, n = case["m"], case["n_cols"]
        w, r = (n + 63) // 64, min(m, n)
        wt = (m + 63) // 64 if case["transform"] else 0
        return {"bytes": 8 * m * (2 * w + wt) + 4 * m, "flops": 2.0 * m * r * (n - r / 2 + (m / 2 if wt else 0))}
    if kind == "pauli":
        n, q = case["n"], case["qubits"]
        return {"bytes": 16 * n * ((q + 63) // 64) + 8 * n * ((n + 63) // 64), "flops": 2.0 * n * n * q}  # symmetric
    if kind == "evaluate":
        t, l, p = case["terms"], case["settings"], case["params"]
        pw, lw = (p + 63) // 64, (l + 63) // 64
        return {"bytes": 8 * (2 * t * pw + l * pw + 2 * t * lw) + 12 * l, "flops": 4.0 * t * l * p}
    if kind == "single":
        return {"bytes": _arena_traffic(case["qubits"] * case["per_qubit"], case["qubits"]), "flops": 0}
    if kind == "batch":
        q = (case["q_lo"] + case["q_hi"]) / 2
        n = int(q * (case["m_lo"] + case["m_hi"]) / 2)
        return {"bytes": case["count"] * _arena_traffic(n, int(q)), "flops": 0}
    if kind == "sample":
        k = (case["d"] + 1) // 2 * (case["d"] - 1)
        return {"bytes": case["shots"] * 8 * ((k * (case["rounds"] + 1) + 64) // 64), "flops": 0}
    if kind == "train":
        rows = case["states"] * case["per_state"]
        return {"bytes": rows * (2 * zx.MLP_IN + 8 + 4) + 28 * zx.MLP_NPARAM,
                "flops": rows * 6.0 * zx.MLP_IN * zx.MLP_HID}
    n = case["qubits"] * (2 + case["depth"] // 2)
    return {"bytes": case["count"] * (n * ((n + 63) // 64) * 8 + 8 * n), "flops": 0}


# -------------------------------------------------------------------- exact --

def exact(case, seed):
    """Outputs in 64 bits where they are computed numbers (bits and counts are compared as they are)."""
    if case["kind"] == "evaluate":
        return _exact_evaluate(prepare(case, seed))
    if case["kind"] == "train":
        return _exact_train(prepare(case, seed))
    return None


def _exact_evaluate(s):
    if s["case"]["any_phase"]:
        return None  # a value near a power of two may fall on either side of it: mantissa and exponent together
    l, p, t = s["case"]["settings"], s["case"]["params"], s["case"]["terms"]
    f = _unpack(s["F"], p).float().T.contiguous()
    par = [torch.remainder(_unpack(s[k], p).float() @ f, 2).to(torch.float64) for k in ("U", "V")]
    r = math.sqrt(0.5)
    root = torch.complex(torch.tensor([1, r, 0, -r, -1, -r, 0, r], dtype=torch.float64),
                         torch.tensor([0, r, 1, r, 0, -r, -1, -r], dtype=torch.float64)).to(DEV)
    z = torch.ones(l, dtype=torch.complex128, device=DEV)
    for k in range(t):
        ca = (4 * par[0][k].long() + int(s["ka"][k])) % 8
        cb = (4 * par[1][k].long() + int(s["kb"][k])) % 8
        z = z * (1 + root[ca] + root[cb] - root[(ca + cb) % 8])
        if k % 16 == 15:
            big = torch.maximum(z.real.abs(), z.imag.abs())
            z = z * torch.exp2(-torch.frexp(big)[1].double())
    big = torch.maximum(z.real.abs(), z.imag.abs())
    z = z * torch.exp2(-torch.frexp(big)[1].double())
    return {"a": None, "b": None, "mant": torch.view_as_real(z), "expo": None}


def _exact_train(s):
    x = s["x"].view(torch.bfloat16).double()
    param = s["mlp"].param.double()
    n1, h = zx.MLP_IN * zx.MLP_HID, zx.MLP_HID
    w1, b1, w2, b2 = param[:n1].view(zx.MLP_IN, h), param[n1:n1 + h], param[n1 + h:n1 + 2 * h], param[-1]
    w1r, w2r = (w.to(torch.float32).to(torch.bfloat16).double() for w in (w1, w2))
    pre = x @ w1r + b1
    act = pre.clamp(min=0)
    score = act @ w2r + b2
    per = s["case"]["per_state"]
    sc, cost = score.view(-1, per), s["cost"].view(-1, per)
    here = cost >= 0
    least = torch.where(here, cost, torch.full_like(cost, 1 << 40)).min(dim=1, keepdim=True).values
    target = (here & (cost == least)).double()
    target = target / target.sum(dim=1, keepdim=True).clamp(min=1)
    masked = torch.where(here, sc, torch.full_like(sc, -float("inf")))
    some = here.any(dim=1)
    lse = torch.where(some, torch.logsumexp(masked, dim=1), torch.zeros_like(masked[:, 0]))
    loss = torch.where(some, lse - (target * sc).sum(dim=1), torch.zeros_like(lse))
    soft = torch.where(here, torch.exp(masked - lse[:, None]), torch.zeros_like(masked))
    ds = ((soft - target) / len(sc)).reshape(-1)
    dpre = torch.where(pre > 0, ds[:, None] * w2r, torch.zeros_like(pre))
    grad = torch.cat([(x.T @ dpre).reshape(-1), dpre.sum(0), act.T @ ds, ds.sum().reshape(1)])
    m, v = 0.1 * grad, 0.001 * grad * grad
    new = param - 1e-3 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
    return {"score": score, "loss": loss, "dscore": ds, "grad": grad, "param": new, "m": m, "v": v}
