"""Workspace sizes do not fall when the batch grows: a workspace that was sized
for a batch serves every smaller one."""
import numpy as np
import pytest

from paper_2404_09213_amd import binding, inputs

CASES = [(W, opts) for W in (1, 2, 5, 9, 12, 13, 18, 23)
         for opts in (dict(), dict(codegen=0), dict(method="per_gate"), dict(method="per_gate", amp_dtype="c128"))]


def _check(plan):
    batches = sorted(set(range(1, 70)) | {2 ** k + d for k in range(6, 14) for d in (-1, 0, 1)})
    for op in (binding.OP_FORWARD, binding.OP_EXPVAL, binding.OP_FORWARD_EXPVAL, binding.OP_BACKWARD):
        sizes = [binding.qsv_workspace_size(plan.handle, b, op) for b in batches]
        assert sizes == sorted(sizes), op


@pytest.mark.parametrize("n_qubits,opts", CASES)
def test_sizes_grow_with_the_batch(n_qubits, opts):
    c = inputs.rx_ry_rz_cz_ladder(n_qubits, 2)
    _check(binding.Plan(c.n_qubits, c.gates, c.n_weights, c.n_inputs, **opts))


def test_sizes_grow_with_the_batch_multi():
    rng = np.random.default_rng(5)
    _check(binding.MultiPlan([inputs.random_layers(n, 1, rng) for n in (4, 8, 13, 14)]))
