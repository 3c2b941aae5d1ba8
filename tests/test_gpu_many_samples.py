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
@pytest.mark.parametrize("kernel", ["k_grad_reduce"])
def test_passes_take_most_of_a_step(kernel):
    """8 qubits, batch 8192, every gate run per sample: one block per input gradient took 2.7 times
    as long as the backward pass."""
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
