"""Large batches, whose arrays pass the caches by (non-temporal accesses from 512 MB a
launch on), against the same samples in small batches: the arithmetic of a
sample is the same, so states, expectations and input gradients agree bit for
bit; weight gradients are float64 sums over another grouping of the batch.
"""
import numpy as np
import pytest

from paper_2404_09213_amd import binding, inputs as I

N, CHUNK = 14, 512   # 2^14 amplitudes: 4 tiles a sample, 4096 samples fill 512 MB


@pytest.mark.gpu
@pytest.mark.parametrize("batch", [2047, 2048, 4095, 4096])  # each direction's rule: off and on
@pytest.mark.parametrize("low_qubits", [4, 2])
def test_large_batch_matches_small_ones(batch, low_qubits):
    import torch
    print(f"[large batch] {batch} low_qubits={low_qubits}", flush=True)
    c = I.ry_rz_cnot_ring(N, 2)
    w, x = I.draw_angles(c, batch, 3)
    g = torch.tensor(I.draw_grad_out(c, batch, 3)).cuda()
    w, x = torch.tensor(w).cuda(), torch.tensor(x).cuda()
    plan = binding.Plan(c.n_qubits, c.gates, c.n_weights, c.n_inputs, low_qubits=low_qubits)
    state, E = plan.forward_expval(w, x, batch)
    gw, gx = plan.backward(w, x, state, g)
    total = torch.zeros_like(gw)
    for b in range(0, batch, CHUNK):
        s = slice(b, min(b + CHUNK, batch))
        st, e = plan.forward_expval(w, x[s].contiguous(), s.stop - b)
        assert torch.equal(st, state[s]) and torch.equal(e, E[s]), b
        dw, dx = plan.backward(w, x[s].contiguous(), st, g[s].contiguous())
        assert torch.equal(dx, gx[s]), b
        total += dw
    # up to 4096 x 4 float64 partials a weight, each at most 14 in size
    assert np.abs((total - gw).cpu().numpy()).max() <= 4096 * 4 * 14 * 2.0 ** -52 * 16
