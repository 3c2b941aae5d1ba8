"""Angles that are not finite, through both directions: one bad input spoils every result of
its own sample and the weight gradients (sums over the batch), and leaves the
other samples' results bit for bit as they were. The circuits have runs of several
rotations after controlled gates, with weights and inputs in one run, so that the
generated backward has shears and phase vectors per sample and shared row sums."""
import numpy as np
import pytest

from paper_2404_09213_amd import binding, inputs as I


def circuit(n):
    c = I.Circuit(n, name="bad")
    for q in range(n):
        c.input("RX", q, q)
        c.weight("RY", q)
        c.input("RZ", q, q)
    for r in range(2):
        for q in range(n - 1):
            c.fixed("CNOT" if r else "CZ", q, q + 1)
        for q in range(n):
            c.weight("RZ", q)
            c.weight("RX", q)
            c.input("RY", q, (q + r) % n)
            c.weight("RZ", q)
    return c


CASES = [(4, {}), (5, {}), (12, {}), (13, {}), (6, {"tile_qubits": 4, "low_qubits": 1}), (5, {"codegen": 0}),
         (13, {"codegen": 0}), (5, {"method": "per_gate"}), (11, {"method": "per_gate", "amp_dtype": "c128"})]


@pytest.mark.gpu
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("n,opts", CASES, ids=["-".join([str(n)] + [f"{k}{v}" for k, v in o.items()]) for n, o in CASES])
def test_a_bad_angle_stays_in_its_sample(n, opts, bad):
    import torch
    print(f"[bad angle] n={n} {opts} {bad}", flush=True)
    c = circuit(n)
    plan = binding.Plan(c.n_qubits, c.gates, c.n_weights, c.n_inputs, **opts)
    if not opts:  # the generated backward has shears and phase vectors
        src = binding.qsv_plan_codegen_source(plan.handle)
        assert "a_ = M_[0], b_ = M_[1]" in src and "r_ = M_[" in src
    B = 4
    w, x = (torch.from_numpy(t).cuda() for t in I.draw_angles(c, B, 60 + n))
    g = torch.from_numpy(I.draw_grad_out(c, B, 60 + n)).cuda()

    def run(x):
        state, E = plan.forward_expval(w, x, B)
        gw, gx = plan.backward(w, x, state, g)
        return [t.clone() for t in (state, E, gw, gx)]

    fine = run(x)
    x2 = x.clone()
    x2[1, 2] = bad
    state, E, gw, gx = run(x2)
    for got, ref in ((state, fine[0]), (E, fine[1]), (gx, fine[3])):
        assert torch.isnan(got[1]).all()
        for b in (0, 2, 3):
            assert torch.equal(got[b], ref[b]) and not torch.isnan(ref[b]).any()
    assert torch.isnan(gw).all()
