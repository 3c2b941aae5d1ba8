"""Rotation cores of the generated backward kernels (shears with waiting phases) against
the oracle and the table-driven kernels, where they can go wrong: angles at
which a matrix entry vanishes or changes sign, every kind of gate run (lead and
trailing diagonals, one or several rotations, fixed gates), runs separated by
controlled gates of every kind, tiles smaller than, equal to and larger than
the state, and matrices shared by the batch or per sample.

Tolerances are the parity tests': 1e-5 on amplitudes and expectations, 1e-4
normwise on gradients. A core adds three float32 roundings per amplitude where
a 2x2 product adds four, so they carry over.
"""
import math

import numpy as np
import pytest

from paper_2404_09213_amd import inputs as I

from .helpers import AMP_TOL, EXP_TOL, grad_close, gpu_run, oracle_run

# zeros and sign changes of cos(theta / 2) and sin(theta / 2), both ends of the
# folded range (theta = pi folds phi to pi/2), tiny and large angles
ANGLES = [0.0, math.pi, -math.pi, 2 * math.pi, -2 * math.pi, 3 * math.pi, 4 * math.pi, math.pi / 2, -math.pi / 2,
          1e-6, -1e-6, math.pi - 1e-6, math.pi + 1e-6, 1e-20, 100.25, 0.7]

RUNS = [("RY",), ("RX",), ("RZ",), ("RX", "RY"), ("RY", "RX"), ("RX", "RY", "RZ"), ("RY", "RZ"), ("RZ", "RY"),
        ("RZ", "RX", "RZ"), ("H", "RY"), ("RX", "H", "RZ"), ("H", "RZ", "H"), ("X", "RY", "Y"), ("Z", "RX", "Z"),
        ("RZ", "RZ"), ("RY", "RY", "RY", "RX", "RZ", "RY"), ("Y",), ("H", "Z"), ("RZ", "H", "RX", "Y", "RZ")]


def runs_circuit(n, rng, per_sample, rounds=3):
    """Every qubit gets a random run, then a few controlled gates, `rounds` times."""
    c = I.Circuit(n, name=f"runs{n}")
    for r in range(rounds):
        for q in range(n):
            for k in RUNS[int(rng.integers(len(RUNS)))]:
                if k not in I.PARAMETRIC:
                    c.fixed(k, q)
                elif per_sample and rng.random() < 0.5:
                    c.input(k, q, int(rng.integers(n)))
                else:
                    c.weight(k, q)
        for k in rng.choice(["CNOT", "CZ", "CRX", "CRY", "CRZ", "CCX", "CCZ", "CCRX"], size=n):
            a, b, t = (int(v) for v in rng.choice(n, size=3, replace=False))
            three = k in I.THREE_QUBIT
            add = c.weight if k in I.PARAMETRIC else c.fixed
            add(str(k), a, b, t if three else -1)
    c.n_inputs = n if per_sample else 0
    return c


CASES = [(4, {}), (5, {}), (6, {"tile_qubits": 4, "low_qubits": 1}), (9, {"tile_qubits": 6, "low_qubits": 2}),
         (12, {}), (13, {}), (9, {"bwd_gate_by_gate": 1}), (9, {"mfma": 7}), (8, {"fuse_width": 4, "splitter": 1})]


@pytest.mark.gpu
@pytest.mark.parametrize("per_sample", [False, True], ids=["shared", "per_sample"])
@pytest.mark.parametrize("n,opts", CASES, ids=["-".join([str(n)] + [f"{k}{v}" for k, v in o.items()]) for n, o in CASES])
def test_cores_match_oracle_and_tables(orc, n, opts, per_sample):
    rng = np.random.default_rng(700 + n + per_sample)
    print(f"[cores] n={n} {opts} per_sample={per_sample}", flush=True)
    c = runs_circuit(n, rng, per_sample)
    B = 3
    w = rng.choice(ANGLES, size=c.n_weights).astype(np.float32)
    x = rng.choice(ANGLES, size=(B, c.n_inputs)).astype(np.float32)
    g = I.draw_grad_out(c, B, n)
    ref = oracle_run(orc, c, w, x, B, g)
    tables = {k: v for k, v in opts.items() if k in ("tile_qubits", "low_qubits")}
    for o in (opts, {**tables, "codegen": 0}):
        got = gpu_run(c, w, x, B, g, **o)
        assert np.abs(got["state"].cpu().numpy() - ref["state"]).max() <= AMP_TOL
        assert np.abs(got["E"].cpu().numpy() - ref["E"]).max() <= EXP_TOL
        ok, rel = grad_close(got["gw"].cpu().numpy(), ref["gw"])
        assert ok, f"weight gradients off by {rel:.2e} ({o})"
        if per_sample:
            ok, rel = grad_close(got["gx"].cpu().numpy(), ref["gx"])
            assert ok, f"input gradients off by {rel:.2e} ({o})"


@pytest.mark.gpu
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_cores_pass_on_nan_and_infinity(bad):
    """One bad angle of one sample spoils that sample and leaves the others alone."""
    c = I.Circuit(5, name="bad")
    for q in range(5):
        c.input("RX", q, q)
        c.weight("RY", q)
    for q in range(4):
        c.fixed("CZ", q, q + 1)
    for q in range(5):
        c.weight("RX", q)
        c.input("RY", q, q)
        c.weight("RZ", q)
    w, x = I.draw_angles(c, 3, 77)
    x[1, 2] = bad
    got = gpu_run_plain(c, w, x)
    st = got.cpu().numpy()
    assert np.isnan(st[1]).all()
    x[1, 2] = 0.0
    fine = gpu_run_plain(c, w, x).cpu().numpy()
    assert np.array_equal(st[[0, 2]], fine[[0, 2]])


def gpu_run_plain(c, w, x):
    import torch

    from paper_2404_09213_amd import binding
    plan = binding.Plan(c.n_qubits, c.gates, c.n_weights, c.n_inputs)
    dev = torch.device("cuda:0")
    return plan.forward(torch.from_numpy(w).to(dev), torch.from_numpy(x).to(dev), x.shape[0])


@pytest.mark.gpu
@pytest.mark.parametrize("gbg", [0, 1])
@pytest.mark.parametrize("n", [4, 5, 12])
def test_several_z_components_at_one_point(orc, n, gbg):
    """Diagonal gates on all register qubits, and twice on one of them with only
    diagonal gates between: their components share one set of products."""
    c = I.Circuit(n, name=f"zz{n}")
    for q in range(n):
        c.weight("RY", q)
    for r in range(3):
        for q in range(n):
            for _ in range(1 + (q + r) % 3):
                c.weight("RZ", q)
        for q in range(n - 1):
            c.fixed("CZ", q, q + 1)
    for q in range(n):
        c.weight("RX", q)
    print(f"[z] n={n} gbg={gbg}", flush=True)
    w, x = I.draw_angles(c, 2, 30 + n)
    g = I.draw_grad_out(c, 2, 30 + n)
    got = gpu_run(c, w, x, 2, g, bwd_gate_by_gate=gbg)
    ok, rel = grad_close(got["gw"].cpu().numpy(), oracle_run(orc, c, w, x, 2, g)["gw"])
    assert ok, rel
