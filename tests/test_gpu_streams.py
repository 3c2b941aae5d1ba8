"""One plan used from several streams and threads at once, with batches that grow and
shrink: every stream has workspaces of its own, sized for its largest batch, and
results are bit for bit those of a plan that is used alone."""
import threading

import numpy as np
import pytest

from paper_2404_09213_amd import binding, inputs as I

BATCHES = (2, 7, 3, 33, 5, 64, 1, 130)
CASES = [("fused", lambda: I.rx_ry_rz_cz_ladder(10, 3), {}),
         ("fused_two_tiles", lambda: I.ry_rz_cnot_ring(13, 2), {}),
         ("plain", lambda: I.ry_rz_cnot_ring(9, 2), {"method": "per_gate"})]


def _plan(c, opts):
    return binding.Plan(c.n_qubits, c.gates, c.n_weights, c.n_inputs, **opts)


def _data(c, lane, batch):
    import torch
    w, x = I.draw_angles(c, batch, 31 * lane + batch)
    return [torch.from_numpy(np.ascontiguousarray(t)).cuda() for t in (w, x, I.draw_grad_out(c, batch, lane + batch))]


def _step(plan, w, x, g):
    state, E = plan.forward_expval(w, x, x.shape[0])
    return [state, E, plan.expval(state), *plan.backward(w, x, state, g)]


@pytest.mark.gpu
@pytest.mark.parametrize("threads", [False, True], ids=["one_thread", "threads"])
@pytest.mark.parametrize("name,make,opts", CASES, ids=[c[0] for c in CASES])
def test_streams_with_growing_batches(name, make, opts, threads):
    import torch
    print(f"[streams] {name} threads={threads}", flush=True)
    c, lanes = make(), 2
    data = [[_data(c, lane, b) for b in (BATCHES if lane == 0 else BATCHES[::-1])] for lane in range(lanes)]
    alone = _plan(c, opts)
    ref = [[_step(alone, *d) for d in lane] for lane in data]
    plan = _plan(c, opts)
    streams = [torch.cuda.Stream() for _ in range(lanes)]
    got = [[] for _ in range(lanes)]
    torch.cuda.synchronize()

    def one(lane, d):
        with torch.cuda.stream(streams[lane]):
            got[lane].append(_step(plan, *d))

    if threads:
        errors = []

        def work(lane):
            try:
                for d in data[lane]:
                    one(lane, d)
            except Exception as e:  # reported by the main thread
                errors.append(e)

        ts = [threading.Thread(target=work, args=(i,)) for i in range(lanes)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert not errors, errors
    else:
        for i in range(len(BATCHES)):
            for lane in range(lanes):
                one(lane, data[lane][i])
    torch.cuda.synchronize()
    for lane in range(lanes):
        for i, (a, b) in enumerate(zip(got[lane], ref[lane])):
            assert all(torch.equal(u, v) for u, v in zip(a, b)), (lane, i)
    # a workspace per stream, none shared
    at = [plan.workspace(1, binding.OP_BACKWARD, "cuda").data_ptr()]
    for s in streams:
        with torch.cuda.stream(s):
            at.append(plan.workspace(1, binding.OP_BACKWARD, "cuda").data_ptr())
    assert len(set(at)) == 1 + lanes


@pytest.mark.parametrize("device", ["cpu", "meta"])
def test_no_workspace_off_the_gpu(device):
    import torch
    with pytest.raises(ValueError):
        _plan(I.ry_rz_cnot_ring(4, 1), {}).workspace(1, binding.OP_BACKWARD, torch.device(device))
