"""Backward passes of the generated kernels take their gate runs as rotation cores or as 2x2
products, by instructions. On the CPU: which circuits get which. On the GPU: circuits that get cores,
with every kind of controlled gate between the runs and angles at which a core's entries
vanish, against the oracle (random circuits, which get products, are in the other tests)."""
import numpy as np
import pytest

from paper_2404_09213_amd import binding, inputs as I

from .helpers import AMP_TOL, EXP_TOL, grad_close, gpu_run, oracle_run
from .test_gpu_cores import ANGLES, CASES

RUNS = [("RX", "RY", "RZ"), ("RZ", "RY", "RX", "RZ"), ("RZ", "RX", "RZ", "RY", "RZ"), ("RY", "Z", "RX", "RZ", "RY"),
        ("RX", "H", "RZ", "RY", "RZ")]


def rotations(n, rng, per_sample, rounds=3):
    c = I.Circuit(n, name=f"rotations{n}")
    for _ in range(rounds):
        for q in range(n):
            for k in RUNS[int(rng.integers(len(RUNS)))]:
                if k not in I.PARAMETRIC:
                    c.fixed(k, q)
                elif per_sample and rng.random() < 0.5:
                    c.input(k, q, int(rng.integers(n)))
                else:
                    c.weight(k, q)
        for k in rng.choice(["CNOT", "CZ", "CRX", "CRY", "CRZ", "CCX", "CCZ", "CCRX"], size=n // 3 + 1):
            a, b, t = (int(v) for v in rng.choice(n, size=3, replace=False))
            (c.weight if k in I.PARAMETRIC else c.fixed)(str(k), a, b, t if k in I.THREE_QUBIT else -1)
    c.n_inputs = n if per_sample else 0
    return c


def _plan(c, **opts):
    return binding.Plan(c.n_qubits, c.gates, c.n_weights, c.n_inputs, **opts)


def _cores(plan):
    return binding.qsv_plan_codegen_source(plan.handle).count("a_ = M_[0], b_ = M_[1]")


@pytest.mark.parametrize("n,gates,seed", [(16, 120, 16), (12, 120, 12), (6, 120, 6), (9, 120, 7)])
def test_random_circuits_keep_their_stages(n, gates, seed):
    """Taken apart, the runs of these circuits need a stage more, and more instructions."""
    c = I.random_mixed(n, gates, np.random.default_rng(seed), n_inputs=n, p_input=0.3, kinds=I.ALL_KINDS)
    assert _plan(c).info()["n_bwd_stages"] <= _plan(c, codegen=0).info()["n_bwd_stages"]


@pytest.mark.parametrize("n", [4, 9, 12, 13, 20])
def test_runs_of_rotations_are_cores(n):
    assert _cores(_plan(I.rx_ry_rz_cz_ladder(n, 3))) > 0


IDS = ["-".join([str(n)] + [f"{k}{v}" for k, v in o.items()]) for n, o in CASES]


@pytest.mark.gpu
@pytest.mark.parametrize("per_sample", [False, True], ids=["shared", "per_sample"])
@pytest.mark.parametrize("n,opts", CASES, ids=IDS)
def test_cores_between_controlled_gates(orc, n, opts, per_sample):
    def circuit(seed):
        return rotations(n, np.random.default_rng(seed), per_sample)

    # the first seed whose plan has cores (gate by gate there are none: vectors only)
    seed = 40 if opts.get("bwd_gate_by_gate") else next(s for s in range(40, 60) if _cores(_plan(circuit(s), **opts)))
    print(f"[rotations] n={n} {opts} per_sample={per_sample} seed={seed}", flush=True)
    c, rng, B = circuit(seed), np.random.default_rng(seed), 3
    w = rng.choice(ANGLES, size=c.n_weights).astype(np.float32)
    x = rng.choice(ANGLES, size=(B, c.n_inputs)).astype(np.float32)
    g = I.draw_grad_out(c, B, n)
    ref = oracle_run(orc, c, w, x, B, g)
    got = gpu_run(c, w, x, B, g, **opts)
    assert np.abs(got["state"].cpu().numpy() - ref["state"]).max() <= AMP_TOL
    assert np.abs(got["E"].cpu().numpy() - ref["E"]).max() <= EXP_TOL
    for k in ("gw", "gx"):
        if k == "gx" and not per_sample:
            continue
        ok, rel = grad_close(got[k].cpu().numpy(), ref[k])
        assert ok, f"{k} off by {rel:.2e}"
