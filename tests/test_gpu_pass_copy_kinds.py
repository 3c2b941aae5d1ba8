"""qsv_pass_copy in each kind of access the passes use: buffers below the size from which a launch
passes the caches by, non-temporal buffers above (512 MB in the launch's arrays), and
without 16-byte pairs. Values are moved between the same indices; the first backward pass
writes what it reads to psi and lambda."""
import pytest

from paper_2404_09213_amd import binding, inputs

N = 14  # 4 tiles a sample: 4,096 samples of one array, 2,048 of two fill 512 MB


@pytest.mark.gpu
@pytest.mark.parametrize("low_qubits", [4, 0])
@pytest.mark.parametrize("batch", [2047, 2048, 4095, 4096])
def test_copies_of_large_launches(batch, low_qubits):
    import torch
    print(f"[pass copy] batch={batch} low_qubits={low_qubits}", flush=True)
    c = inputs.ry_rz_cnot_ring(N, 2)
    p = binding.Plan(c.n_qubits, c.gates, c.n_weights, c.n_inputs, low_qubits=low_qubits)
    info = p.info()
    state = torch.empty((batch, 1 << N), dtype=torch.complex64, device="cuda")
    state.real.copy_(torch.arange(1, 1 + (1 << N), device="cuda").float())
    state.imag.copy_(torch.arange(1, 1 + batch, device="cuda").view(-1, 1).float())
    ref = state.clone()
    for i in range(1, info["n_fwd_passes"]):
        p.pass_copy(0, i, batch, state)
        assert torch.equal(state, ref)
    ws = p.workspace(batch, binding.OP_BACKWARD, "cuda")
    mats, nbytes = binding.qsv_workspace_size(p.handle, batch, binding.OP_FORWARD), batch << (N + 3)
    lo = mats + (nbytes + 255) // 256 * 256 + 4096 + 256  # where the backward keeps lambda
    psi, lam = (ws[a:a + nbytes].view(torch.complex64).view(batch, 1 << N) for a in (mats, lo))
    assert info["n_bwd_passes"] > 2
    ws.fill_(255)
    p.pass_copy(1, 0, batch, state)
    assert torch.equal(psi, ref) and torch.equal(lam, ref)
    lam.imag.neg_()
    conj = lam.clone()
    for i in range(1, info["n_bwd_passes"]):
        p.pass_copy(1, i, batch, state)
        assert torch.equal(psi, ref) and torch.equal(lam, conj) and torch.equal(state, ref)
    state.zero_()
    p.pass_copy(0, 0, batch, ref)
    assert torch.equal(ref, state)


@pytest.mark.gpu
@pytest.mark.parametrize("tile", [12, 13, 14])
def test_copies_of_large_tiles(tile):
    """Workgroups of 256, 512 and 1,024 threads."""
    import torch
    print(f"[pass copy] tile={tile}", flush=True)
    c = inputs.ry_rz_cnot_ring(16, 2)
    p = binding.Plan(c.n_qubits, c.gates, c.n_weights, c.n_inputs, tile_qubits=tile)
    state = torch.randn((3, 1 << 16), dtype=torch.complex64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    ref = state.clone()
    assert p.info()["n_fwd_passes"] > 1
    for i in range(1, p.info()["n_fwd_passes"]):
        p.pass_copy(0, i, 3, state)
        assert torch.equal(state, ref)
    p.pass_copy(0, 0, 3, state)
    assert (state == 0).all()
