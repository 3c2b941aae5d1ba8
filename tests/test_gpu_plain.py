"""The plain method's launches at the sizes where their shape changes: samples
below and above 256 items per launch, chunks of the backward split further for
small batches, every control and target position, both precisions."""
import numpy as np
import pytest

from paper_2404_09213_amd import inputs as I

from .helpers import AMP_TOL, EXP_TOL, grad_close, gpu_run, oracle_run


@pytest.mark.gpu
@pytest.mark.parametrize("amp", ["c64", "c128"])
@pytest.mark.parametrize("n,batch", [(3, 2), (8, 3), (9, 1), (10, 2), (11, 1), (12, 5), (14, 1)])
def test_plain_launch_shapes(orc, n, batch, amp):
    rng = np.random.default_rng(900 + n)
    print(f"[plain] n={n} B={batch} {amp}", flush=True)
    c = I.random_mixed(n, 100, rng, n_inputs=3, p_input=0.3, kinds=I.ALL_KINDS)
    w, x = I.draw_angles(c, batch, 40 + n)
    g = I.draw_grad_out(c, batch, 40 + n)
    got = gpu_run(c, w, x, batch, g, method="per_gate", amp_dtype=amp)
    ref = oracle_run(orc, c, w, x, batch, g)
    # complex128 gates are float64 throughout: rounding of some 100 gates stays below 1e-12
    a_tol, e_tol, g_tol = (AMP_TOL, EXP_TOL, 1e-4) if amp == "c64" else (1e-12, 1e-12, 1e-11)
    assert np.abs(got["state"].cpu().numpy() - ref["state"]).max() <= a_tol
    assert np.abs(got["E"].cpu().numpy() - ref["E"]).max() <= e_tol
    for k in ("gw", "gx"):
        ok, rel = grad_close(got[k].cpu().numpy(), ref[k], tol=g_tol)
        assert ok, (k, rel)
