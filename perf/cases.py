"""Performance cases of the amplitude engine.

listed() holds the standing cases and draw() more of the same ranges: whole
contraction calls (a plan's amplitudes, from a 4x4 circuit whose tensors all
fit a cache to 32 slices of a 6x6 circuit) and the single steps that a program
can call by itself (pairwise contractions, permutations, batch statistics).
Sizes are those of the tests and of bench.py, or lie between them.

Case kinds and their fields:
  call     one Plan.contract (entry "contract") or Plan.contract_noalloc
           ("noalloc", the entry of serving loops): grid rows x cols, depth,
           circuit and planner seeds, open qubits, sliced wires, the number of
           slice ids given (0: every slice), bitstrings per call, precision;
  pair     one pair_contract of `batch` problems: 2^m rows, 2^n columns, 2^k
           summed terms.  layout "random": every operand's index order drawn
           from `order` (a permutation has to be folded in); "plan": the
           planner's layout, summed indices lowest in A and B in the same
           order, the free indices of both merged in C.  shared_b: one B for
           the whole batch (an operand that does not depend on the slice);
  permute  one permutation of a rank-r complex64 tensor;
  xeb      linear cross-entropy statistics of 2^r amplitudes.
"""
import functools
import math
import random

import numpy as np
import torch

import paper_2110_14502_amd as R


# --------------------------------------------------------------------- cases
def listed():
    return [
        # The smallest call: the 16-amplitude batch of a 4x4 (1+8+1) circuit.
        # Launches and host work are all there is.
        dict(name="call_4x4_f32", kind="call", entry="contract", rows=4, cols=4, depth=8,
             circuit=1, plan_seed=1, trials=256, open=4, sliced=-1, ids=0, batch=1, prec="f32"),
        # A serving loop's call: single amplitudes of 24 bitstrings of a 5x5
        # circuit, merged into one launch per step, without allocations.
        dict(name="serve_5x5_f32", kind="call", entry="noalloc", rows=5, cols=5, depth=10,
             circuit=7, plan_seed=1, trials=64, open=0, sliced=-1, ids=0, batch=24, prec="f32"),
        # An ordinary sliced call in reduced precision: 16 slices, 16 amplitudes.
        dict(name="call_5x5_f16", kind="call", entry="contract", rows=5, cols=5, depth=12,
             circuit=3, plan_seed=5, trials=64, open=4, sliced=4, ids=0, batch=1, prec="f16"),
        # The headline circuit, 32 of its 256 slices per call (a share of the
        # slices, as a program that checkpoints between calls runs it).
        dict(name="call_6x6_f32", kind="call", entry="contract", rows=6, cols=6, depth=14,
             circuit=2, plan_seed=42, trials=1024, open=6, sliced=8, ids=32, batch=1, prec="f32"),
        dict(name="call_6x6_f16", kind="call", entry="contract", rows=6, cols=6, depth=14,
             circuit=2, plan_seed=42, trials=1024, open=6, sliced=8, ids=32, batch=1, prec="f16"),
        # A dense step with a long sum and random index orders (the synthetic
        # rank-24..32 steps), in full and in reduced precision.
        dict(name="dense_f32", kind="pair", m=14, n=12, k=12, batch=1, layout="random", order=11,
             shared_b=False, prec="f32"),
        dict(name="dense_bf16", kind="pair", m=14, n=13, k=13, batch=1, layout="random", order=12,
             shared_b=False, prec="bf16"),
        # A dense step with a short sum, one problem per slice, the small
        # operand shared by all slices.
        dict(name="short_f32", kind="pair", m=14, n=7, k=6, batch=37, layout="plan", order=13,
             shared_b=True, prec="f32"),
        # A stem step: a large tensor absorbs a small one, memory bound.
        dict(name="stem_f32", kind="pair", m=17, n=4, k=4, batch=32, layout="plan", order=14,
             shared_b=False, prec="f32"),
        # The last step of a call: a few outputs, sums of 2^18 terms.
        dict(name="tail_f32", kind="pair", m=3, n=3, k=18, batch=32, layout="plan", order=15,
             shared_b=False, prec="f32"),
        # A separate permutation of a rank-26 tensor.
        dict(name="permute_26", kind="permute", rank=26, order=16),
        # The score of a 2^21-amplitude correlated batch.
        dict(name="xeb_21", kind="xeb", rank=21, samples=4096),
    ]


def draw(rng):
    kind = rng.choice(["call", "call", "call6", "dense", "dense", "short", "stem", "tail", "permute",
                       "xeb"])
    if kind == "call":
        rows, cols = rng.choice([(3, 4), (4, 4), (4, 5), (5, 5)])
        n = rows * cols
        return dict(kind="call", entry=rng.choice(["contract", "noalloc"]), rows=rows, cols=cols,
                    depth=rng.randint(6, 11), circuit=rng.randint(1, 99), plan_seed=rng.randint(1, 99),
                    trials=64, open=rng.randint(0, min(6, n)), sliced=rng.choice([-1, 2, 3]), ids=0,
                    batch=int(round(2 ** rng.uniform(0, 5))), prec=rng.choice(["f32", "f32", "f16", "bf16"]))
    if kind == "call6":
        return dict(kind="call", entry="contract", rows=6, cols=6, depth=14, circuit=2, plan_seed=42,
                    trials=1024, open=6, sliced=8, ids=rng.randint(1, 32), batch=1,
                    prec=rng.choice(["f32", "f16"]))
    order, prec = rng.randint(1, 10 ** 6), rng.choice(["f32", "f32", "f16", "bf16"])
    if kind == "dense":
        while True:
            m, n, k = rng.randint(8, 15), rng.randint(6, 14), rng.randint(8, 14)
            if 28 <= m + n + k <= (38 if prec == "f32" else 39) and max(m + n, m + k, n + k) <= 27:
                return dict(kind="pair", m=m, n=n, k=k, batch=1, layout="random", order=order,
                            shared_b=False, prec=prec)
    if kind in ("short", "stem"):
        while True:
            if kind == "short":
                m, n, k = rng.randint(9, 16), rng.randint(6, 9), rng.randint(4, 7)
            else:
                m, n, k = rng.randint(12, 19), rng.randint(1, 5), rng.randint(1, 6)
            batch = int(round(2 ** rng.uniform(0, 6)))
            if 18 <= math.log2(batch) + max(m + n, m + k) <= 26.5:
                return dict(kind="pair", m=m, n=n, k=k, batch=batch, layout="plan", order=order,
                            shared_b=rng.random() < 0.4, prec=prec if kind == "short" else "f32")
    if kind == "tail":
        return dict(kind="pair", m=rng.randint(0, 4), n=rng.randint(0, 3), k=rng.randint(12, 18),
                    batch=int(round(2 ** rng.uniform(0, 5))), layout="plan", order=order,
                    shared_b=False, prec="f32")
    if kind == "permute":
        return dict(kind="permute", rank=rng.randint(14, 27), order=order)
    return dict(kind="xeb", rank=rng.randint(6, 22), samples=int(round(2 ** rng.uniform(0, 14))))


# ---------------------------------------------------------------- circuits
class _Gate:
    """One gate as Circuit takes it."""

    def __init__(self, kind, q0, q1=-1, theta=0.0, phi=0.0):
        self.kind, self.q0, self.q1, self.theta, self.phi, self.u = kind, q0, q1, theta, phi, None


def _grid_circuit(rows, cols, depth, seed):
    """Seeded (1+depth+1) grid circuit: H on every qubit; per cycle a random
    layer of sqrt(X), sqrt(Y), sqrt(W) without repeats on a qubit, then
    fSim(pi/2, pi/6) on the couplers of class "ABCDCDAB"[cycle % 8]; a last
    random layer."""
    n = rows * cols
    rng = np.random.default_rng(seed)
    gates = [_Gate(R.GATE_H, q) for q in range(n)]
    prev = [-1] * n

    def layer():
        for q in range(n):
            g = int(rng.integers(3)) if prev[q] < 0 else (prev[q] + 1 + int(rng.integers(2))) % 3
            prev[q] = g
            gates.append(_Gate((R.GATE_SQRT_X, R.GATE_SQRT_Y, R.GATE_SQRT_W)[g], q))

    for cycle in range(depth):
        layer()
        cls = "ABCDCDAB"[cycle % 8]
        for r in range(rows):
            for c in range(cols):
                q = r * cols + c
                if cls in "AB":
                    if c + 1 < cols and c % 2 == "AB".index(cls):
                        gates.append(_Gate(R.GATE_FSIM, q, q + 1, math.pi / 2, math.pi / 6))
                elif r + 1 < rows and r % 2 == "CD".index(cls):
                    gates.append(_Gate(R.GATE_FSIM, q, q + cols, math.pi / 2, math.pi / 6))
    layer()
    return n, gates


def _plan(case):
    n, gates = _grid_circuit(case["rows"], case["cols"], case["depth"], case["circuit"])
    net = R.Network(R.Circuit(n, gates), list(range(n - case["open"], n)))
    return R.Plan(net, n_sliced=case["sliced"], seed=case["plan_seed"], path_trials=case["trials"])


@functools.lru_cache(maxsize=64)
def _plan_info(key):
    return _plan(dict(key)).info()


def _call_bits(case, seed):
    n = case["rows"] * case["cols"]
    return np.random.default_rng(seed).integers(0, 2, size=(case["batch"], n - case["open"]), dtype=np.uint8)


def _matrix(g):
    s = 1.0 / math.sqrt(2.0)
    x = torch.tensor([[0, 1], [1, 0]], dtype=torch.complex128)
    y = torch.tensor([[0, -1j], [1j, 0]], dtype=torch.complex128)
    one = torch.eye(2, dtype=torch.complex128)
    if g.kind == R.GATE_H:
        return torch.tensor([[s, s], [s, -s]], dtype=torch.complex128)
    if g.kind == R.GATE_FSIM:
        m = torch.zeros(4, 4, dtype=torch.complex128)
        m[0, 0] = 1.0
        m[1, 1] = m[2, 2] = math.cos(g.theta)
        m[1, 2] = m[2, 1] = -1j * math.sin(g.theta)
        m[3, 3] = complex(math.cos(g.phi), -math.sin(g.phi))
        return m
    # exp(-i pi/4 G) = (1 - i G) / sqrt(2): its square is -i G.
    gen = {R.GATE_SQRT_X: x, R.GATE_SQRT_Y: y, R.GATE_SQRT_W: (x + y) * s}[g.kind]
    return (one - 1j * gen) * s


def _state_vector(n, gates, device):
    psi = torch.zeros(1 << n, dtype=torch.complex128, device=device)
    psi[0] = 1.0
    for g in gates:
        m = _matrix(g).to(device)
        if g.q1 < 0:
            v = psi.view(1 << g.q0, 2, -1)
            a, b = v[:, 0], v[:, 1]
            psi = torch.stack([m[0, 0] * a + m[0, 1] * b, m[1, 0] * a + m[1, 1] * b], 1).reshape(-1)
            continue
        # q0 < q1; every two-qubit gate here is an fSim: |00> keeps its value.
        v = psi.view(1 << g.q0, 2, 1 << (g.q1 - g.q0 - 1), 2, -1)
        v01, v10 = v[:, 0, :, 1].clone(), v[:, 1, :, 0].clone()
        v[:, 0, :, 1] = m[1, 1] * v01 + m[1, 2] * v10
        v[:, 1, :, 0] = m[2, 1] * v01 + m[2, 2] * v10
        v[:, 1, :, 1] *= m[3, 3]
    return psi


# ------------------------------------------------------------------- steps
def _pair_labels(case):
    m, n, k = case["m"], case["n"], case["k"]
    M, N, K = list(range(m)), list(range(m, m + n)), list(range(m + n, m + n + k))
    rng = random.Random(case["order"])
    c = M + N
    rng.shuffle(c)
    if case["layout"] == "random":
        a, b = M + K, N + K
        rng.shuffle(a)
        rng.shuffle(b)
    else:
        # Free indices of both operands keep their order in C; the summed
        # ones are the lowest address bits of both, in the same order.
        rng.shuffle(K)
        a = [x for x in c if x < m] + K
        b = [x for x in c if x >= m] + K
    return a, b, c


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _normal(seed, part, n):
    """n complex normal values of unit variance (complex64, on the device)."""
    g = torch.Generator(device=_device()).manual_seed(seed * 16 + part)
    return torch.randn(n, dtype=torch.complex64, device=_device(), generator=g)


def _pair_inputs(case, seed):
    nb = case["batch"]
    A = _normal(seed, 0, nb << (case["m"] + case["k"]))
    B = _normal(seed, 1, (1 if case["shared_b"] else nb) << (case["n"] + case["k"]))
    return A, B


def _permute_labels(case):
    a = list(range(case["rank"]))
    b = list(a)
    random.Random(case["order"]).shuffle(b)
    return a, b


def _xeb_inputs(case, seed):
    """Porter-Thomas amplitudes of a 36-qubit circuit as (re, im) doubles, and
    sampled entries."""
    n = 1 << case["rank"]
    g = torch.Generator(device=_device()).manual_seed(seed * 16 + 2)
    amps = torch.randn(2 * n, dtype=torch.float64, device=_device(), generator=g) * (0.5 * 2.0 ** -36) ** 0.5
    idx = torch.randint(0, n, (case["samples"],), device=_device(), generator=g)
    return amps, idx


def _reorder(x, have, want):
    """The flat tensor x with index order `have` in index order `want` (most
    significant address bit first)."""
    r = len(have)
    at = torch.arange(1 << r, device=x.device)
    src = torch.zeros_like(at)
    for i, label in enumerate(reversed(want)):
        src |= ((at >> i) & 1) << (r - 1 - have.index(label))
    return x[src]


# --------------------------------------------------------------- interface
def prepare(case, seed):
    if case["kind"] == "call":
        plan = _plan(case).bind()
        ids = np.arange(case["ids"], dtype=np.uint64) if case["ids"] else None
        return dict(kind="call", plan=plan, bits=_call_bits(case, seed), ids=ids, prec=case["prec"],
                    noalloc=case["entry"] == "noalloc")
    if case["kind"] == "pair":
        a, b, c = _pair_labels(case)
        A, B = _pair_inputs(case, seed)
        nb, prec = case["batch"], R.PRECISIONS[case["prec"]]
        stride = dict(batch=nb, stride_a=1 << len(a), stride_b=0 if case["shared_b"] else 1 << len(b))
        need = R.pair_workspace_bytes(a, b, c, prec=prec, **stride)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
        out = torch.empty(nb << len(c), dtype=torch.complex64, device="cuda")
        return dict(kind="pair", A=A, B=B, labels=(a, b, c),
                    args=dict(C_out=out, workspace=ws, prec=prec, stride_c=1 << len(c), **stride))
    if case["kind"] == "permute":
        X = _normal(seed, 3, 1 << case["rank"])
        return dict(kind="permute", X=X, labels=_permute_labels(case), out=torch.empty_like(X))
    amps, idx = _xeb_inputs(case, seed)
    return dict(kind="xeb", amps=amps, samples=idx)


def run(state):
    if state["kind"] == "call":
        contract = state["plan"].contract_noalloc if state["noalloc"] else state["plan"].contract
        return contract(state["bits"], slice_ids=state["ids"], prec=state["prec"])
    if state["kind"] == "pair":
        return R.pair_contract(state["A"], state["B"], *state["labels"], **state["args"])
    if state["kind"] == "permute":
        return R.permute(state["X"], *state["labels"], out=state["out"])
    return R.batch_xeb(state["amps"], 36, samples=state["samples"])


def work(case):
    if case["kind"] == "call":
        i = _plan_info(tuple(sorted(case.items())))
        n_ids = case["ids"] or i["n_slices"]
        flops = (i["flops_per_slice"] * n_ids + i["flops_per_bitstring"]) * case["batch"]
        # Leaves (at most 16 complex64 values each), bitstrings, slice ids; the
        # amplitudes in complex128.
        data = 128 * i["n_leaves"] + case["batch"] * i["n_closed"] + 8 * n_ids
        return {"bytes": data + 16.0 * case["batch"] * 2 ** case["open"], "flops": flops}
    if case["kind"] == "pair":
        m, n, k, nb = case["m"], case["n"], case["k"], case["batch"]
        elems = nb * 2.0 ** (m + k) + (1 if case["shared_b"] else nb) * 2.0 ** (n + k) + nb * 2.0 ** (m + n)
        return {"bytes": 8.0 * elems, "flops": 8.0 * nb * 2.0 ** (m + n + k)}
    if case["kind"] == "permute":
        return {"bytes": 16.0 * 2 ** case["rank"], "flops": 0.0}
    return {"bytes": 16.0 * 2 ** case["rank"] + 24.0 * case["samples"] + 40.0,
            "flops": 6.0 * 2 ** case["rank"] + 4.0 * case["samples"]}


def exact(case, seed):
    if case["kind"] == "call":
        n, gates = _grid_circuit(case["rows"], case["cols"], case["depth"], case["circuit"])
        if n > 25 or case["ids"]:  # no state vector; a part of the slices has none either
            return None
        psi = _state_vector(n, gates, _device())
        no = case["open"]
        bits = _call_bits(case, seed)
        # Closed qubits come first; open qubit i (the i-th of the last `no`) is
        # bit i of the entry index, so the last axis of a row is bit reversed.
        rev = [sum(((e >> i) & 1) << (no - 1 - i) for i in range(no)) for e in range(1 << no)]
        rows = [int("".join(map(str, b)) or "0", 2) for b in bits.tolist()]
        amps = psi.view(-1, 1 << no)[torch.tensor(rows, device=psi.device)]
        return torch.view_as_real(amps[:, torch.tensor(rev, device=psi.device)].contiguous())
    if case["kind"] == "pair":
        a, b, c = _pair_labels(case)
        A, B = _pair_inputs(case, seed)
        m, n, k, nb = case["m"], case["n"], case["k"], case["batch"]
        M, N, K = list(range(m)), list(range(m, m + n)), list(range(m + n, m + n + k))
        out = torch.empty(nb << (m + n), dtype=torch.complex128, device=A.device)

        def ordered(x, have, want, rows):
            return _reorder(x.to(torch.complex128), have, want).view(rows, -1)

        for j in range(nb):
            jb = 0 if case["shared_b"] else j
            x = ordered(A[j << (m + k):(j + 1) << (m + k)], a, M + K, 1 << m)
            y = ordered(B[jb << (n + k):(jb + 1) << (n + k)], b, K + N, 1 << k)
            out[j << (m + n):(j + 1) << (m + n)] = _reorder((x @ y).view(-1), M + N, c)
        return out
    if case["kind"] == "permute":
        X = _normal(seed, 3, 1 << case["rank"])
        a, b = _permute_labels(case)
        return _reorder(X.to(torch.complex128), a, b)
    amps, idx = _xeb_inputs(case, seed)
    p = amps.view(-1, 2).square().sum(1)
    s, s2, dim = p.sum(), p.square().sum(), 2.0 ** 36
    return {"sum_p": float(s), "sum_p2": float(s2), "xeb_all": float(dim * p.mean() - 1),
            "xeb_ideal_sampling": float(dim * s2 / s - 1), "xeb_samples": float(dim * p[idx].mean() - 1)}
