"""Vector passes of the other Krylov methods, whose threads load four elements
per wait: vectors of less than one pass of the launch, of whole passes and of
more than four with a remainder."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("method", ["bicgstab", "fcg", "cgs"])
@pytest.mark.parametrize("shape", [(20, 12, 28), (64, 64, 64), (80, 96, 72)])
def test_methods_agree(shape, method):
    """Each solve stops at a relative residual of 1e-11, so two solutions
    differ by at most 2e-11 kappa(A): below 4 / pi^2 n^2 (n = 96 cells) times
    the coefficient's contrast of 10, 4e4, so 1e-6; an element left out of an
    update or a sum stops the convergence instead."""
    nx, ny, nz = shape
    print(f"krylov {method} {shape}", flush=True)
    rng = np.random.default_rng(nx)
    a = torch.tensor(np.exp(rng.uniform(-0.5, 0.5, (nz, ny, nx)) * np.log(10.0)), device=DEV)
    f = torch.tensor(rng.standard_normal((nz, ny, nx)), device=DEV)
    s = gm.GMGPoisson(a, precision="fp64")
    ref = s.solve(f, 0.2, 0.7, tol=1e-11)
    r, _ = s.krylov_solve(f, 0.2, 0.7, method=method, tol=1e-11)
    assert ref.final_relres <= 1e-11 and r.final_relres <= 1e-11
    assert ((r.phi - ref.phi).norm() / ref.phi.norm()).item() < 1e-6
