"""Steps on many samples: sums of gradient partials at every launch shape, and what such
steps spend outside their passes."""
import numpy as np
import pytest

from paper_2404_09213_amd import binding, inputs as I


def reuploading(n, layers):
    c = I.Circuit(n, name=f"reuploading{n}")
    for _ in range(layers):
        for q in range(n):
            c.input("RX", q, q)
            c.weight("RY", q)
            c.input("RZ", q, (q + 1) % n)
        for q in range(n - 1):
            c.fixed("CZ", q, q + 1)
    c.n_inputs += 1  # a column that no gate reads
    return c


def _plan(c, **opts):
    return binding.Plan(c.n_qubits, c.gates, c.n_weights, c.n_inputs, **opts)


def _data(c, batch, seed):
    import torch
    w, x = I.draw_angles(c, batch, seed)
    return [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in (w, x, I.draw_grad_out(c, batch, seed))]


# chunks per sample from 1 to 4096: input gradients by thread, by wave and by block;
# batches below and above the weights' change from waves to blocks
SUMS = [(3, 1, {}), (5, 257, {}), (12, 513, {}), (13, 2, {}), (15, 5, {}), (15, 70, {}), (16, 3, {}), (16, 33, {}),
        (12, 3, {"tile_qubits": 4, "low_qubits": 0}), (14, 2, {"tile_qubits": 4, "low_qubits": 0}),
        (16, 1, {"tile_qubits": 4, "low_qubits": 0}), (10, 9, {"method": "per_gate"}), (13, 1, {"method": "per_gate"}),
        (13, 200, {"method": "per_gate"}), (17, 2, {"codegen": 0})]


@pytest.mark.gpu
@pytest.mark.parametrize("n,batch,opts", SUMS, ids=["-".join(map(str, (n, b, *o.values()))) for n, b, o in SUMS])
def test_gradient_sums(n, batch, opts):
    """A sample's input gradients are its own partials' sums, and weight gradients the sums over
    the samples: against the same samples one by one. Partials are the same numbers where the
    chunks are (the plain method splits small batches further: float32 sums of other parts)."""
    import torch
    print(f"[sums] n={n} batch={batch} {opts}", flush=True)
    c = reuploading(n, 2)
    plan = _plan(c, **opts)
    w, x, g = _data(c, batch, 5)
    state, _ = plan.forward_expval(w, x, batch)
    gw, gx = plan.backward(w, x, state, g)
    some = sorted({0, 1 % batch, batch // 2, batch - 1})
    # float64 sums of up to 4096 partials, each at most n in size, in another order
    tol = n * 4096 * 4096 * 2.0 ** -53 if "method" not in opts else 1e-5 * n
    for b in some:
        dw, dx = plan.backward(w, x[b:b + 1].contiguous(), state[b:b + 1], g[b:b + 1].contiguous())
        assert (gx[b] - dx[0]).abs().max().item() <= tol, b
    assert (gx[:, -1] == 0).all()
    total = torch.zeros_like(gw)
    for b in range(batch):
        total += plan.backward(w, x[b:b + 1].contiguous(), state[b:b + 1], g[b:b + 1].contiguous())[0]
    assert (total - gw).abs().max().item() <= tol * batch
    only_w = plan.backward(w, x, state, g, want_inputs=False)
    assert only_w[1] is None and torch.equal(only_w[0], gw)


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", ["k_grad_reduce", "k_coef"])
def test_passes_take_most_of_a_step(kernel):
    """8 qubits, batch 8192, every gate run per sample: one block per input gradient took 2.7 times
    as long as the backward pass, coefficients by quads of lanes 4 times as long."""
    import torch
    c = reuploading(8, 5)
    plan = _plan(c)
    w, x, g = _data(c, 8192, 9)
    best = {}
    for i in range(6):
        plan.profile(i > 0)  # the first call compiles
        state, _ = plan.forward_expval(w, x, 8192)
        plan.backward(w, x, state, g)
        torch.cuda.synchronize()
        for k, v in plan.profile_read().items():
            best[k] = min(best.get(k, 1e9), v["total_ms"])
    plan.profile(False)
    passes = sum(v for k, v in best.items() if k.startswith("qsv_"))
    print({k: round(1e3 * v, 1) for k, v in best.items()})
    assert best[kernel] < passes


def _mixed(n, gates, n_inputs, p_input):
    return I.random_mixed(n, gates, np.random.default_rng(n), n_inputs=n_inputs, p_input=p_input, kinds=I.ALL_KINDS)


# (circuit, batch, options): coefficients by quads in pieces of 16 samples, by sample in
# the whole batch, whose last 64 samples are not all there
FORMS = [("reup4", lambda: reuploading(4, 4), 4001, {}),
         ("reup8", lambda: reuploading(8, 5), 1000, {}),
         ("reup13", lambda: reuploading(13, 2), 1001, {}),
         ("mixed5", lambda: _mixed(5, 150, 5, 1.0), 3003, {}),
         ("mixed9_remap", lambda: _mixed(9, 200, 3, 0.5), 2049, {"weight_remap": 1}),
         ("ladder_tables", lambda: I.rx_ry_rz_cz_ladder(5, 2), 9000, {"codegen": 0}),
         ("mixed_tables", lambda: _mixed(6, 120, 6, 0.7), 2100, {"codegen": 0}),
         ("plain", lambda: _mixed(5, 150, 5, 0.8), 1300, {"method": "per_gate"}),
         ("plain_c128", lambda: _mixed(4, 150, 4, 0.8), 1290, {"method": "per_gate", "amp_dtype": "c128"})]


@pytest.mark.gpu
@pytest.mark.parametrize("name,make,batch,opts", FORMS, ids=[f[0] for f in FORMS])
def test_coefficients_do_not_depend_on_the_batch(name, make, batch, opts):
    """Both forms of the coefficients' kernel round alike: states, expectations and (where the
    partials' chunks are the same) input gradients agree bit for bit."""
    import torch
    print(f"[coefficients] {name}", flush=True)
    c = make()
    plan = _plan(c, **opts)
    w, x, g = _data(c, batch, 21)
    state, E = plan.forward_expval(w, x, batch)
    gw, gx = plan.backward(w, x, state, g)
    for b in list(range(0, batch, 16 * max(1, batch // 160))) + [batch - 1 - (batch - 1) % 16]:
        s = slice(b, min(b + 16, batch))
        st, e = plan.forward_expval(w, x[s].contiguous(), s.stop - b)
        assert torch.equal(st, state[s]) and torch.equal(e, E[s]), b
        dw, dx = plan.backward(w, x[s].contiguous(), st, g[s].contiguous())
        assert torch.equal(dx, gx[s]) if "method" not in opts else (dx - gx[s]).abs().max().item() <= 1e-5 * c.n_qubits, b
