"""Forward 2x2 products on the matrix cores: operands shared by groups of four matrix slots
(full, partly filled and interleaved groups of weight-only and per-sample
matrices, and operations between them that use other slots) and sign flips
taken along by the next product (before controlled products, swaps, diagonals,
exchanges and the final store). Against the oracle.

Tolerances are the parity tests' (the products are the same ones).
"""
import numpy as np
import pytest

from paper_2404_09213_amd import inputs as I

from .helpers import AMP_TOL, EXP_TOL, gpu_run, oracle_run


def circuit(n, rng, n_input):
    c = I.Circuit(n, name=f"matrix_ops{n}")
    c.n_inputs = n_input
    for q in range(n):
        c.fixed("H", q)
    for r in range(4):
        for q in range(n):  # 1 to 3 rotations: generic, real and RX-like products
            for k in rng.choice(["RX", "RY", "RZ"], size=int(rng.integers(1, 4))):
                if n_input and rng.random() < 0.4:
                    c.input(str(k), q, int(rng.integers(n_input)))
                else:
                    c.weight(str(k), q)
        for _ in range(n):  # signs inside and outside the registers
            a, b = (int(v) for v in rng.choice(n, size=2, replace=False))
            c.fixed("CZ", a, b)
        if n > 2:
            a, b, t = (int(v) for v in rng.choice(n, size=3, replace=False))
            c.fixed("CCZ", a, b, t)
        a, b = (int(v) for v in rng.choice(n, size=2, replace=False))
        k = ["CRX", "CRY", "CNOT", "CRZ"][r]
        (c.fixed if k == "CNOT" else c.weight)(k, a, b)
    for q in range(n - 1):  # ends on signs: nothing takes them along
        c.fixed("CZ", q, q + 1)
    return c


CASES = [(2, {}), (4, {}), (5, {}), (9, {"tile_qubits": 6, "low_qubits": 2}), (10, {}), (12, {}), (13, {}),
         (10, {"mfma": 0})]


@pytest.mark.gpu
@pytest.mark.parametrize("n_input", [0, 2], ids=["shared", "per_sample"])
@pytest.mark.parametrize("n,opts", CASES, ids=["-".join([str(n)] + [f"{k}{v}" for k, v in o.items()]) for n, o in CASES])
def test_forward_products_and_signs(orc, n, opts, n_input):
    rng = np.random.default_rng(40 + n)
    print(f"[matrix ops] n={n} {opts} n_input={n_input}", flush=True)
    c = circuit(n, rng, n_input)
    B = 3
    w, x = I.draw_angles(c, B, 5 + n)
    g = I.draw_grad_out(c, B, n)
    ref = oracle_run(orc, c, w, x, B, g)
    got = gpu_run(c, w, x, B, g, **opts)
    assert np.abs(got["state"].cpu().numpy() - ref["state"]).max() <= AMP_TOL
    assert np.abs(got["E"].cpu().numpy() - ref["E"]).max() <= EXP_TOL
