"""Arnoldi steps with more than ten and more than sixteen basis vectors: the
operator pass planned for three blocks per CU, and the dots of a second batch."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("steps", [11, 14, 19])
def test_estimate_is_the_true_residual(steps, precision):
    """Without restarts the least-squares residual of the Arnoldi relation is
    the true one up to the roundings of the basis, 1e-16 times its condition
    (below 1 / relres): at most 1e-6 relative while relres > 1e-10.  A wrong
    dot or chunk breaks the relation."""
    print(f"many vectors {steps} {precision}", flush=True)
    rng = np.random.default_rng(steps)
    a = torch.tensor(np.exp(rng.uniform(-0.5, 0.5, (80, 96, 128)) * np.log(1e2)), device=DEV)
    f = torch.tensor(rng.standard_normal(a.shape), device=DEV)
    s = gm.GMGPoisson(a, precision=precision, restart=20, max_iter=steps, nu_pre=0, nu_post=1, cold_cycle="vcycle")
    r = s.solve(f, 0.2, 0.7, tol=0.0, raise_on_error=False)
    assert r.iterations == steps and r.final_relres > 1e-10
    assert abs(r.res_hist[-1] / r.final_relres - 1.0) < 1e-6
