"""The allocation-free call's limit counts what a forward needs (its gate matrices and
the readout partials), not the backward's matrices."""
import numpy as np
import pytest

from paper_2404_09213_amd import binding, inputs

TOO_BIG, LIMIT = -5, 16 * 1024 * 1024


def _reuploading(n, layers):
    """Every angle reads an input, so every matrix is per sample; the forward fuses a
    run of rotations into one matrix, the backward has several per run."""
    c = inputs.Circuit(n, name="reuploading")
    for _ in range(layers):
        for q in range(n):
            for k in ("RX", "RY", "RZ"):
                c.input(k, q, q)
        for q in range(n - 1):
            c.fixed("CZ", q, q + 1)
    return c


def _plan(c, **opts):
    return binding.Plan(c.n_qubits, c.gates, c.n_weights, c.n_inputs, **opts)


# per sample: n matrices of 32 bytes a layer, and n readout float64 per tile (one tile)
N, LAYERS = 4, 3
PER_SAMPLE = N * LAYERS * 32 + N * 8


@pytest.mark.parametrize("opts", [{}, {"codegen": 0}], ids=["generated", "tables"])
def test_limit_is_the_forwards_need(opts):
    p = _plan(_reuploading(N, LAYERS), **opts)
    fits = LIMIT // PER_SAMPLE - 64  # 64 samples of slack for shared matrices and rounding to 256 bytes
    assert binding.qsv_workspace_size(p.handle, fits, binding.OP_FORWARD_EXPVAL) > LIMIT
    L, fake = binding.lib(), 256
    # past the size check: without tables (and without a device) the call is refused there
    assert L.qsv_forward_expval_noalloc(p.handle, fake, fake, fits, fake, fake, None) not in (0, TOO_BIG)
    assert L.qsv_forward_expval_noalloc(p.handle, fake, fake, fits + 128, fake, fake, None) == TOO_BIG


@pytest.mark.gpu
@pytest.mark.parametrize("opts", [{}, {"codegen": 0}], ids=["generated", "tables"])
def test_a_forward_at_the_limit(opts):
    import torch
    p = _plan(_reuploading(N, LAYERS), **opts)
    batch = LIMIT // PER_SAMPLE - 64
    x = torch.from_numpy(np.random.default_rng(3).uniform(-3, 3, (batch, N)).astype(np.float32)).cuda()
    w = torch.empty(0, device="cuda")
    ref_state, ref_E = p.forward_expval(w, x, batch)
    state, E = torch.full_like(ref_state, float("nan")), torch.full_like(ref_E, float("nan"))
    p.forward_expval_noalloc(w, x, batch, state, E)
    assert torch.equal(state, ref_state) and torch.equal(E, ref_E)
