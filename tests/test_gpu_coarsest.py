"""Direct solver of the coarsest level: blocked inverse (64-wide blocks) and
matrix-vector product on the GPU against a dense float64 solve."""
import numpy as np
import pytest
import torch

from oracle.operator import apply_operator

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")
EPS = np.finfo(np.float64).eps


# single-level grids (nx, ny, nz; one dimension odd or below 4): one cell, the
# edges of one and two blocks, several blocks with a remainder
SHAPES = [(1, 1, 1), (2, 1, 1), (7, 9, 1), (64, 1, 1), (5, 13, 1), (1, 1, 127), (2, 64, 1), (3, 43, 1), (7, 7, 7),
          (2, 21, 25)]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape", SHAPES)
def test_single_level_direct_solve(shape, precision):
    """z = A^{-1} v of a single-level grid.  Forward error of a solve by the
    computed inverse: at most a small multiple of n eps cond(A) in float64;
    with the inverse, v and z rounded to float32 each row adds about
    sqrt(n) float32 roundings of terms up to |A^{-1}| |v| (bounded here by n
    of them)."""
    nx, ny, nz = shape
    n = nx * ny * nz
    print(f"direct solve {shape} {precision}", flush=True)
    rng = np.random.default_rng(n)
    a = np.exp(rng.uniform(-0.5, 0.5, (nz, ny, nx)) * np.log(1e2))
    v = rng.standard_normal(a.shape)
    h = (1.0 / nx, 1.3 / ny, 0.9 / nz)
    A = np.empty((n, n))
    for c in range(n):
        e = np.zeros(n)
        e[c] = 1.0
        A[:, c] = apply_operator(e.reshape(a.shape), a, h).ravel()
    inv = np.linalg.inv(A)
    ref = np.linalg.solve(A, v.ravel())
    s = gm.GMGPoisson(torch.tensor(a, device=DEV), h=h, precision=precision)
    assert len(s.levels) == 1
    z = s.vcycle(torch.tensor(v, device=DEV)).cpu().numpy().ravel()
    lam = np.linalg.eigvalsh(A)
    bound = 4 * n * EPS * lam[-1] / lam[0] * np.linalg.norm(ref)
    if precision == "mixed":
        bound += (n + 3) * np.finfo(np.float32).eps * np.linalg.norm(np.abs(inv) @ np.abs(v.ravel()))
    assert np.linalg.norm(z - ref) <= bound
