"""What a program asks of the simulator, as cases that can be timed.

Every case goes through the public entry points of the package: Fourier
transforms of a resident ket, the overlap of a transformed ket with another
one, circuits (planned once, run many times), gates and dense blocks applied
one by one, batches of small circuits, an approximate run of a factorized
ket, and the training of the separability network. Dense kets and batches
hand back their own device buffer: the library takes its device memory from
allocator hooks (qs_set_allocator), and the hooks set here give it torch
tensors, so that a result can be used on the GPU without a copy.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

import paper_2304_14969_amd as qs

TWO_PI = 2.0 * math.pi

# ------------------------------------------------------------------ cases


def listed():
    return [
        # Fourier transforms, a controlled phase between the transform and its
        # inverse (arithmetic in the Fourier basis): a small register, where
        # latency counts; a register inside a wider double-precision ket; the
        # 1 GiB ket of the benchmark.
        {"name": "qft_10_c64", "kind": "qft", "n": 10, "start": 0, "len": 10, "dtype": "c64"},
        {"name": "qft_19_c128_part", "kind": "qft", "n": 19, "start": 1, "len": 17, "dtype": "c128"},
        {"name": "qft_27_c64", "kind": "qft", "n": 27, "start": 0, "len": 27, "dtype": "c64"},
        # A transform of the qubits from `start` on, whose result is compared
        # with another ket: the fidelity of two states, in qubit order.
        {"name": "overlap_23_c64", "kind": "overlap", "n": 23, "start": 0, "dtype": "c64"},
        # Gates given one at a time (an interactive program), then all
        # amplitudes read.
        {"name": "gates_18_c64", "kind": "gates", "n": 18, "count": 64, "dtype": "c64"},
        # Dense blocks of two to six qubits (a program that fuses by itself).
        {"name": "blocks_24_c64", "kind": "blocks", "n": 24, "count": 5, "dtype": "c64"},
        # Random circuits from |0...0>: a small one, one in double precision,
        # a 2 GiB ket.
        {"name": "circuit_11_c64", "kind": "circuit", "n": 11, "layers": 8, "dtype": "c64"},
        {"name": "circuit_20_c128", "kind": "circuit", "n": 20, "layers": 8, "dtype": "c128"},
        {"name": "circuit_28_c64", "kind": "circuit", "n": 28, "layers": 10, "dtype": "c64"},
        # Many small circuits together (a parameter sweep).
        {"name": "batch_256_c64", "kind": "batch", "count": 256, "low": 12, "high": 20, "layers": 8,
         "dtype": "c64"},
        # The paper's approximate mode: 54 qubits, 7 layers.
        {"name": "approx_54_7", "kind": "approx", "rows": 6, "cols": 9, "layers": 7, "p": 0.6},
        # The separability network: trained on recorded attempts, its gradient
        # over all of them, their scores.
        {"name": "train_20000", "kind": "train", "rows": 20000, "batch": 256, "steps": 40},
    ]


def draw(rng):
    kind = rng.choice(["qft", "qft", "overlap", "gates", "blocks", "circuit", "circuit", "batch",
                       "approx", "train"])
    dtype = rng.choice(["c64", "c64", "c128"])
    wide = dtype == "c128"
    if kind == "qft":
        n = rng.randint(8, 25 if wide else 27)
        start = 0 if rng.random() < 0.5 else rng.randint(0, n // 3)
        length = n - start if rng.random() < 0.5 else rng.randint(max(2, (n - start) // 2), n - start)
        return {"kind": kind, "n": n, "start": start, "len": length, "dtype": dtype}
    if kind == "overlap":
        n = rng.randint(9, 24 if wide else 26)
        return {"kind": kind, "n": n, "start": rng.randint(0, n // 3), "dtype": dtype}
    if kind == "gates":
        return {"kind": kind, "n": rng.randint(6, 20), "count": rng.randint(16, 96), "dtype": dtype}
    if kind == "blocks":
        return {"kind": kind, "n": rng.randint(9, 23 if wide else 25), "count": rng.randint(3, 9),
                "dtype": dtype}
    if kind == "circuit":
        return {"kind": kind, "n": rng.randint(6, 24 if wide else 27), "layers": rng.randint(2, 10),
                "dtype": dtype}
    if kind == "batch":
        low = rng.randint(4, 14)
        high = min(20, low + rng.randint(0, 8))
        most = min(512, 2 ** (26 - high - (1 if wide else 0)))
        count = int(round(math.exp(rng.uniform(math.log(8), math.log(max(9, most))))))
        return {"kind": kind, "count": count, "low": low, "high": high, "layers": rng.randint(2, 8),
                "dtype": dtype}
    if kind == "approx":
        rows, cols = rng.choice([(4, 5), (5, 5), (5, 7), (6, 6), (6, 9), (7, 7)])
        return {"kind": kind, "rows": rows, "cols": cols, "layers": rng.randint(3, 8),
                "p": round(rng.uniform(0.55, 0.8), 3)}
    batch = rng.randint(64, 512)
    rows = int(round(math.exp(rng.uniform(math.log(1.5 * batch), math.log(30000)))))
    return {"kind": kind, "rows": rows, "batch": batch, "steps": rng.randint(10, 50)}


# ------------------------------------------------------------------ inputs

_buffers: dict = {}  # address -> the torch tensor behind it
_asked: list = []    # the tensors given out since _ready() was last called
_hooks: list = []


def _ready():
    """The library with its device memory taken from torch tensors."""
    lib = qs.load(use_torch_allocator=False)
    if not _hooks:
        def alloc(nbytes, _user):
            try:
                t = torch.empty(int(nbytes), dtype=torch.uint8, device="cuda")
            except RuntimeError:
                return None
            _buffers[t.data_ptr()] = t
            _asked.append(t)
            return t.data_ptr()

        def free(ptr, _user):
            _buffers.pop(ptr, None)

        proto = lib.qs_set_allocator.argtypes
        _hooks.extend([proto[0](alloc), proto[1](free)])
        if lib.qs_set_allocator(_hooks[0], _hooks[1], ctypes.c_void_p()) != qs.OK:
            raise RuntimeError(lib.qs_last_error().decode())
    _asked.clear()
    return lib


def _types(case):
    return (qs.C64, torch.complex64) if case["dtype"] == "c64" else (qs.C128, torch.complex128)


def _state(n, dtype, torch_type):
    """A dense state and its amplitudes' buffer (qubit q = index bit q while
    no relabelling is pending)."""
    _ready()
    st = qs.State(n, dtype)
    size = 2 ** n * (8 if torch_type == torch.complex64 else 16)
    buf = next(t for t in _asked if t.numel() == size).view(torch_type)
    _asked.clear()
    return st, buf


def _gaussian(n, seed):
    """i.i.d. complex Gaussian amplitudes of unit norm, complex128, on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.view_as_complex(torch.randn(2 ** n, 2, dtype=torch.float64, device="cuda", generator=g))
    return a / torch.linalg.vector_norm(a)


def _u3(theta, phi, lam):
    c, s = math.cos(theta / 2), math.sin(theta / 2)
    return np.array([[c, -np.exp(1j * lam) * s],
                     [np.exp(1j * phi) * s, np.exp(1j * (phi + lam)) * c]])


def _circuit_gates(n, layers, g):
    """Per layer a U3 on every qubit, then CZ or iSWAP on a random matching."""
    gates = []
    for _ in range(layers):
        ang = g.uniform(0.0, TWO_PI, (n, 3))
        perm = g.permutation(n)
        coin = g.random(n // 2) < 0.5
        gates += [("u3", q, *(float(x) for x in ang[q])) for q in range(n)]
        gates += [("cz" if coin[i] else "iswap", int(perm[2 * i]), int(perm[2 * i + 1]))
                  for i in range(n // 2)]
    return gates


def _grid_gates(rows, cols, layers, g):
    """Per layer a U3 on every qubit, then a random coupler on every edge of
    the layer's pattern (A, B: horizontal, C, D: vertical edges)."""
    kinds = ("cx", "cy", "cz", "ax", "ay", "az")
    gates = []
    for layer in range(layers):
        ang = g.uniform(0.0, TWO_PI, (rows * cols, 3))
        gates += [("u3", q, *(float(x) for x in ang[q])) for q in range(rows * cols)]
        pat = "ABCDCDAB"[layer % 8]
        odd = 1 if pat in "BD" else 0
        if pat in "AB":
            edges = [(r * cols + c, r * cols + c + 1) for r in range(rows) for c in range(odd, cols - 1, 2)]
        else:
            edges = [(r * cols + c, (r + 1) * cols + c) for r in range(odd, rows - 1, 2) for c in range(cols)]
        for a, b in edges:
            kind = kinds[int(g.integers(0, len(kinds)))]
            gates.append((kind, b, a) if g.random() < 0.5 else (kind, a, b))
    return gates


def _mixed_gates(n, count, g):
    """Single gates of every kind; SWAPs among them, so that the amplitudes
    are read through a relabelling."""
    gates = []
    for _ in range(count):
        k = ("h", "u3", "u3", "cp", "cz", "cx", "iswap", "swap", "ctrl")[int(g.integers(0, 9))]
        q = [int(x) for x in g.choice(n, 3, replace=False)]
        ang = [float(x) for x in g.uniform(0.0, TWO_PI, 3)]
        if k == "h":
            gates.append(("h", q[0]))
        elif k == "u3":
            gates.append(("u3", q[0], *ang))
        elif k == "cp":
            gates.append(("cp", q[0], q[1], ang[0]))
        elif k == "ctrl":
            gates.append(("ctrl", (q[0], q[1]), int(g.integers(0, 4)), q[2], *ang))
        else:
            gates.append((k, q[0], q[1]))
    return gates


def _blocks(n, count, g):
    """Random unitaries on 2, 3, 4, 5, 6, 2, ... random qubits."""
    out = []
    for i in range(count):
        k = 2 + i % 5
        z = g.standard_normal((2 ** k, 2 ** k)) + 1j * g.standard_normal((2 ** k, 2 ** k))
        u, r = np.linalg.qr(z)
        d = np.diagonal(r)
        out.append(("mat", [int(x) for x in g.choice(n, k, replace=False)], u * (d / np.abs(d))))
    return out


def _phase_qubits(case):
    return case["start"], case["start"] + case["len"] - 1, 1.0


def _rows(case, g):
    """Attempts as the approximate mode records them: 21 features of unit
    size, 11 unused ones, about a quarter of the rows rounded."""
    X = np.zeros((case["rows"], qs.MLP_INPUTS), dtype=np.float32)
    X[:, :21] = g.uniform(0.0, 1.0, (case["rows"], 21))
    w = g.standard_normal(21)
    z = X[:, :21] @ w
    y = (z + 0.3 * g.standard_normal(case["rows"]) > np.quantile(z, 0.75)).astype(np.float32)
    return X, y


def _widths(case):
    g = np.random.default_rng(case["count"])
    return [int(v) for v in g.integers(case["low"], case["high"] + 1, case["count"])]


def prepare(case, seed):
    kind = case["kind"]
    g = np.random.default_rng(seed)
    s = {"case": case}
    if kind in ("qft", "overlap"):
        dtype, tt = _types(case)
        s["st"], s["buf"] = _state(case["n"], dtype, tt)
        s["st"].set_amplitudes(_gaussian(case["n"], seed).to(tt).cpu().numpy())
        if kind == "overlap":
            s["ref"], _ = _state(case["n"], dtype, tt)
            s["ref"].set_amplitudes(_gaussian(case["n"], seed + 1_000_003).to(tt).cpu().numpy())
    elif kind in ("gates", "blocks"):
        dtype, tt = _types(case)
        s["st"], s["buf"] = _state(case["n"], dtype, tt)
        make = _mixed_gates if kind == "gates" else _blocks
        s["gates"] = make(case["n"], case["count"], g)
        s["x"] = int(g.integers(0, 2 ** case["n"]))
        if kind == "blocks":
            s["st"].set_amplitudes(_gaussian(case["n"], seed).to(tt).cpu().numpy())
    elif kind == "circuit":
        dtype, tt = _types(case)
        s["st"], s["buf"] = _state(case["n"], dtype, tt)
        s["circ"] = qs.Circuit(case["n"]).add_gates(_circuit_gates(case["n"], case["layers"], g))
    elif kind == "batch":
        dtype, tt = _types(case)
        widths = _widths(case)
        s["circs"] = [qs.Circuit(w).add_gates(_circuit_gates(w, case["layers"], g)) for w in widths]
        _ready()
        s["batch"] = qs.Batch(widths, dtype)
        size = s["batch"].info()["total_amps"] * (8 if tt == torch.complex64 else 16)
        s["buf"] = next(t for t in _asked if t.numel() == size).view(tt)
        _asked.clear()
    elif kind == "approx":
        _ready()
        n = case["rows"] * case["cols"]
        s["st"] = qs.State(n, qs.C64, factorized=True, max_amps=2 ** 26)
        s["st"].set_policy(qs.SEP_AFTER_2Q, case["p"])
        s["circ"] = qs.Circuit(n).add_gates(_grid_gates(case["rows"], case["cols"], case["layers"], g))
        s["idx"] = g.integers(0, 2 ** n, 1024, dtype=np.uint64)
    else:
        _ready()
        s["X"], s["y"] = _rows(case, g)
        s["w"] = qs.mlp_init(seed)
        s["net"] = qs.MLP()
    return s


# ------------------------------------------------------------------ one pass


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "qft":
        st = s["st"]
        a, b, th = _phase_qubits(case)
        st.qft(case["start"], case["len"])
        st.apply_cphase(a, b, th)
        st.qft(case["start"], case["len"], inverse=True)
        return s["buf"]
    if kind == "overlap":
        s["st"].qft(case["start"])
        ov = s["st"].inner(s["ref"])
        # float32 kets give an overlap of float32 accuracy
        return [np.complex64(ov) if case["dtype"] == "c64" else np.complex128(ov), s["buf"]]
    if kind == "gates":
        s["st"].set_basis(s["x"])
        qs.run_gates(s["st"], s["gates"])
        return s["st"].amplitudes(np.complex64 if case["dtype"] == "c64" else np.complex128)
    if kind == "blocks":
        for _, qubits, m in s["gates"]:
            s["st"].apply_fused(qubits, m)
        return s["buf"]
    if kind == "circuit":
        s["st"].set_basis(0)
        s["st"].run(s["circ"])
        return s["buf"]
    if kind == "batch":
        s["batch"].reset()
        s["batch"].run(s["circs"])
        return s["buf"]
    if kind == "approx":
        st = s["st"]
        st.set_basis(0)
        done = True
        try:
            st.run(s["circ"])
        except qs.CapacityError:
            done = False
        sizes = np.zeros(st.n, dtype=np.int64)  # of the subsystem each qubit is in
        for sub in st.subsystems():
            sizes[sub] = len(sub)
        return {"done": done, "F": st.fidelity_estimate(), "sizes": sizes,
                "amplitudes": st.gather(s["idx"]).astype(np.complex64)}
    net = s["net"]
    net.set_params(s["w"])
    loss = net.train(s["X"], s["y"], steps=case["steps"], batch=case["batch"])
    params = net.get_params()
    grad, _ = net.grad(s["X"], s["y"])
    return {"params": params, "loss": loss, "grad": grad, "scores": net.forward(s["X"])}


# ------------------------------------------------------------------ what a pass cannot do without


def work(case):
    kind = case["kind"]
    if kind == "approx":
        n = case["rows"] * case["cols"]
        # every gate once on the kets of its own qubits
        return {"bytes": 2 * 8.0 * 1024, "flops": case["layers"] * n * (28.0 + 64.0)}
    if kind == "train":
        macs = 32 * 64 + 64 * 64 + 64
        rows = case["steps"] * case["batch"]
        # forward, and two products of the same size backward; then forward of
        # all rows for the loss, the gradient and the scores
        return {"bytes": 4.0 * case["rows"] * 34, "flops": 2.0 * macs * (3 * rows + 5 * case["rows"])}
    amp = 8.0 if case["dtype"] == "c64" else 16.0
    if kind == "batch":
        widths = _widths(case)
        return {"bytes": amp * sum(2 ** w for w in widths),
                "flops": sum(14.0 * w * case["layers"] * 2 ** w for w in widths)}
    N = 2.0 ** case["n"]
    if kind == "qft":
        return {"bytes": 2 * amp * N, "flops": 10.0 * N * case["len"]}
    if kind == "overlap":
        return {"bytes": 3 * amp * N, "flops": 5.0 * N * (case["n"] - case["start"]) + 8 * N}
    if kind == "gates":
        return {"bytes": amp * N, "flops": 10.0 * N * case["count"]}
    if kind == "blocks":
        return {"bytes": 2 * amp * N,
                "flops": sum(8.0 * 2 ** (2 + i % 5) * N for i in range(case["count"]))}
    return {"bytes": amp * N, "flops": 14.0 * N * case["n"] * case["layers"]}


# ------------------------------------------------------------------ 64-bit results


def _bits(a, n, qubits):
    """a viewed with one axis per listed qubit (ascending) and the rest
    between them; returns the view and the axis of each listed qubit."""
    order = sorted(qubits, reverse=True)
    shape, top, axis = [], n, {}
    for q in order:
        shape += [2 ** (top - q - 1), 2]
        axis[q] = len(shape) - 1
        top = q
    return a.view(shape + [2 ** top]), axis


def _apply(a, n, qubits, m):
    """The matrix m on `qubits` (row bit j = qubits[j]), in place."""
    k = len(qubits)
    v, axis = _bits(a, n, qubits)

    def at(c):
        ix = [slice(None)] * v.dim()
        for j, q in enumerate(qubits):
            ix[axis[q]] = (c >> j) & 1
        return tuple(ix)

    m = np.asarray(m)
    rows = [r for r in range(2 ** k) if m[r, r] != 1 or np.count_nonzero(m[r]) != 1]
    old = {c: v[at(c)].clone() for r in rows for c in range(2 ** k) if m[r, c] != 0}
    for r in rows:
        acc = None
        for c in range(2 ** k):
            if m[r, c] != 0:
                t = old[c] * complex(m[r, c])
                acc = t if acc is None else acc.add_(t)
        v[at(r)] = 0 if acc is None else acc


def _apply_gate(a, n, g):
    k = g[0]
    if k == "mat":
        _apply(a, n, g[1], g[2])
    elif k == "h":
        _apply(a, n, [g[1]], np.array([[1, 1], [1, -1]]) / math.sqrt(2.0))
    elif k == "u3":
        _apply(a, n, [g[1]], _u3(*g[2:5]))
    elif k in ("cp", "cz"):
        _apply(a, n, [g[1], g[2]], np.diag([1, 1, 1, -1 if k == "cz" else np.exp(1j * g[3])]))
    elif k == "iswap":
        _apply(a, n, [g[1], g[2]], np.array([[1, 0, 0, 0], [0, 0, 1j, 0], [0, 1j, 0, 0], [0, 0, 0, 1]]))
    elif k == "swap":
        _apply(a, n, [g[1], g[2]], np.eye(4)[[0, 2, 1, 3]])
    elif k == "cx":  # qubits (control, target): row bit 0 the control
        _apply(a, n, [g[1], g[2]], np.eye(4)[[0, 3, 2, 1]])
    else:  # ctrl: U3 on the target where the controls take their values
        nc = len(g[1])
        m = np.eye(2 ** (nc + 1), dtype=complex)
        at = [g[2], g[2] + 2 ** nc]
        m[np.ix_(at, at)] = _u3(*g[4:7])
        _apply(a, n, list(g[1]) + [g[3]], m)


def _transform(a, n, start, length, inverse=False):
    v = a.view(2 ** (n - start - length), 2 ** length, 2 ** start)
    # omega = exp(+2 pi i / N): numpy's inverse transform, scaled to be unitary
    f = torch.fft.fft if inverse else torch.fft.ifft
    return f(v, dim=1, norm="ortho").reshape(-1)


def _mlp64(case, g, seed):
    X, y = (torch.from_numpy(v).double() for v in _rows(case, g))
    w = torch.from_numpy(qs_mlp_init(seed)).double()

    def parts(p):
        i, out = 0, []
        for shape in ((32, 64), (64,), (64, 64), (64,), (64, 1), (1,)):
            size = math.prod(shape)
            out.append(p[i:i + size].view(shape))
            i += size
        return out

    def logits(p, x):
        w1, b1, w2, b2, w3, b3 = parts(p)
        return (torch.tanh(torch.tanh(x @ w1 + b1) @ w2 + b2) @ w3 + b3)[:, 0]

    def loss_grad(p, x, t):
        p = p.detach().requires_grad_(True)
        loss = torch.nn.functional.binary_cross_entropy_with_logits(logits(p, x), t)
        (gr,) = torch.autograd.grad(loss, p)
        return loss.detach(), gr

    m, v, at = torch.zeros_like(w), torch.zeros_like(w), 0
    B, lr, b1, b2, eps = case["batch"], 1e-3, 0.9, 0.999, 1e-8
    for step in range(1, case["steps"] + 1):
        if at + B > case["rows"]:
            at = 0
        _, gr = loss_grad(w, X[at:at + B], y[at:at + B])
        at += B
        m = b1 * m + (1 - b1) * gr
        v = b2 * v + (1 - b2) * gr * gr
        w = w - lr * (m / (1 - b1 ** step)) / (torch.sqrt(v / (1 - b2 ** step)) + eps)
    loss, gr = loss_grad(w, X, y)
    with torch.no_grad():
        scores = torch.sigmoid(logits(w, X))
    return {"params": w, "loss": loss, "grad": gr, "scores": scores}


def qs_mlp_init(seed):
    """Layer by layer uniform in +-1/sqrt(fan in), from PCG64 (as the binding
    draws its first parameters)."""
    g = np.random.default_rng(seed)
    parts = []
    for fan, size in ((32, 32 * 64), (32, 64), (64, 64 * 64), (64, 64), (64, 64), (64, 1)):
        parts.append(g.uniform(-1.0 / math.sqrt(fan), 1.0 / math.sqrt(fan), size))
    return np.concatenate(parts).astype(np.float32)


def exact(case, seed):
    kind = case["kind"]
    g = np.random.default_rng(seed)
    if kind == "approx":
        return None  # rounding decisions have no closed form; 54 qubits do not fit a dense ket
    if kind == "train":
        return _mlp64(case, g, seed)
    if kind == "batch":
        widths = _widths(case)
        kets, total = [], 0
        for w in widths:
            a = torch.zeros(2 ** w, dtype=torch.complex128, device="cuda")
            a[0] = 1
            for gate in _circuit_gates(w, case["layers"], g):
                _apply_gate(a, w, gate)
            kets.append(a)
            if 2 ** w % 64:  # kets start on multiples of 64 amplitudes
                kets.append(torch.zeros(64 - 2 ** w % 64, dtype=torch.complex128, device="cuda"))
        return torch.cat(kets)
    n = case["n"]
    single = case["dtype"] == "c64"

    def given(sd):
        a = _gaussian(n, sd)
        return a.to(torch.complex64).to(torch.complex128) if single else a

    if kind == "qft":
        a = _transform(given(seed), n, case["start"], case["len"])
        p, q, th = _phase_qubits(case)
        _apply(a, n, [p, q], np.diag([1, 1, 1, np.exp(1j * th)]))
        return _transform(a, n, case["start"], case["len"], inverse=True)
    if kind == "overlap":
        a = _transform(given(seed), n, case["start"], n - case["start"])
        ov = torch.sum(a.conj() * given(seed + 1_000_003))
        return [np.complex128(ov.item()), a]
    if kind == "circuit":
        a = torch.zeros(2 ** n, dtype=torch.complex128, device="cuda")
        a[0] = 1
        for gate in _circuit_gates(n, case["layers"], g):
            _apply_gate(a, n, gate)
        return a
    make = _mixed_gates if kind == "gates" else _blocks
    gates = make(n, case["count"], g)
    if kind == "gates":
        a = torch.zeros(2 ** n, dtype=torch.complex128, device="cuda")
        a[int(g.integers(0, 2 ** n))] = 1
    else:
        a = given(seed)
    for gate in gates:
        _apply_gate(a, n, gate)
    return a
