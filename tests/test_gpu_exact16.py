"""Whole calls whose every value is exact in 16 bits: circuits of unnormalised Clifford
gates, whose tensors hold 0 and power-of-two multiples of 1, i and 1 +- i, so that every
sum is exact and a call in FP16 or BF16 gives the bits of the FP32 call.  That
reaches what a tolerance would hide: the streaming dot products on 16-bit stored
operands (the last step, sums of 2^14 terms) and, with a non-finite gate, the
flags of the fused subtrees."""
import numpy as np
import pytest
import torch

import paper_2110_14502_amd as R

pytestmark = pytest.mark.gpu


class _Gate:
    def __init__(self, kind, q0, q1, u):
        self.kind, self.q0, self.q1, self.theta, self.phi, self.u = kind, q0, q1, 0.0, 0.0, u


ONE = [np.array([[1, 1], [1, -1]], complex), np.array([[1, -1j], [-1j, 1]]), np.array([[1, -1], [1, 1]], complex)]
TWO = np.zeros((4, 4), complex)  # iSWAP and a phase
TWO[0, 0], TWO[1, 2], TWO[2, 1], TWO[3, 3] = 1, -1j, -1j, -1


def _circuit(rows, cols, depth, seed, first=ONE[0]):
    """A grid circuit of the usual layers and couplers with these gates."""
    rng = np.random.default_rng(seed)
    n = rows * cols
    gates = [_Gate(R.GATE_U1, q, -1, first if q == 0 else ONE[0]) for q in range(n)]
    prev = [-1] * n

    def layer():
        for q in range(n):
            prev[q] = int(rng.integers(3)) if prev[q] < 0 else (prev[q] + 1 + int(rng.integers(2))) % 3
            gates.append(_Gate(R.GATE_U1, q, -1, ONE[prev[q]]))

    for cycle in range(depth):
        layer()
        c = "ABCDCDAB"[cycle % 8]
        for r in range(rows):
            for x in range(cols):
                q = r * cols + x
                if c in "AB" and x + 1 < cols and x % 2 == "AB".index(c):
                    gates.append(_Gate(R.GATE_U2, q, q + 1, TWO))
                elif c in "CD" and r + 1 < rows and r % 2 == "CD".index(c):
                    gates.append(_Gate(R.GATE_U2, q, q + cols, TWO))
    layer()
    return R.Circuit(n, gates)


@pytest.mark.parametrize("batch", [64, 1])  # 2^10 terms per split: direct copies; fewer: through registers
def test_dot_products_on_16_bit_operands(batch):
    print("[case]", batch, flush=True)
    P = R.Plan(R.Network(_circuit(5, 5, 14, 1), list(range(20, 25))), n_sliced=2, seed=2, path_trials=32, lp_min_log2=9,
               bf16_min_log2=9).bind()
    bits = np.random.default_rng(0).integers(0, 2, size=(64, 20), dtype=np.uint8)
    if batch == 1:  # a bitstring with amplitudes that are not zero
        at = int(P.contract(bits).ne(0).any(-1).any(-1).nonzero()[0])
        bits = bits[at:at + 1]
    P.set_timing(4)
    ref, got = P.contract(bits, per_slice=True)[1].clone(), {}
    for prec, store in ((R.F16, R.ST_F16), (R.BF16, R.ST_BF16)):
        got[store] = P.contract(bits, prec=prec, per_slice=True)[1].clone()
        assert P.last_report["fp32_reruns"] == 0
        last = P.launch_timings()[-1]
        assert (last["kernel"], last["m"], last["n"], last["k"]) == (R.KERN_SIMT, 3, 2, 14), last
        assert last["copies"] == 4 * batch and (last["store_a"], last["store_b"]) == (store, store), last
    P.set_timing(-1)
    # (most amplitudes of such a circuit cancel: any error in a term shows there, too)
    assert ref.ne(0).sum().item() >= (64 if batch > 1 else 1)
    for store, x in got.items():
        assert torch.equal(x, ref), store


@pytest.mark.parametrize("prec", [R.F32, R.F16, R.BF16])
def test_non_finite_gates_are_reported(prec):
    """Every step inside fused subtrees: their flags lead to the FP32 re-run and, as
    it is not finite either, to the error."""
    print("[case]", prec, flush=True)
    bits = np.zeros((3, 7), np.uint8)
    for bad, first in ((False, ONE[0]), (True, np.array([[float("inf"), 1], [1, -1]], complex))):
        P = R.Plan(R.Network(_circuit(3, 3, 6, 2, first), [7, 8]), n_sliced=2, seed=1, path_trials=32).bind()
        if not bad:
            assert torch.isfinite(P.contract(bits, prec=prec)).all()
            continue
        with pytest.raises(R.RqcError) as e:
            P.contract(bits, prec=prec)
        assert e.value.code == R.ENUMERIC
