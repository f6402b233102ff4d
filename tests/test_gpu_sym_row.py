"""The fused symmetric sweep whose blocks span the row, against the half-sweep
kernels: rows of one and two waves, full and with a remainder, thin and deep
grids, z-chunks that end inside the grid."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")

# (nx, ny, nz), above the sizes that run as legs (2^20 cells in float32, 2^19
# in float64): 64 pairs (one wave), 128 (two), 56 and 96 (remainders), few
# rows, few planes
SHAPES = [(128, 96, 96), (256, 128, 64), (112, 112, 96), (192, 96, 80), (128, 16, 640), (256, 512, 16)]


@pytest.mark.parametrize("nu", [(2, 2), (1, 3)])
@pytest.mark.parametrize("shape", SHAPES)
def test_row_sweeps_match_half_sweeps(shape, nu):
    """The default V-cycle and full multigrid cycle against those of
    half-sweep kernels: the same arithmetic face by face, contracted
    differently: 1e-13 in float64, 1e-5 in float32 (the fused sweeps'
    tolerances)."""
    nx, ny, nz = shape
    print(f"row sweeps {shape} nu {nu}", flush=True)
    rng = np.random.default_rng(nx + ny + nz)
    a = torch.tensor(np.exp(rng.uniform(-0.5, 0.5, (nz, ny, nx)) * np.log(1e2)), device=DEV)
    v = torch.tensor(rng.standard_normal((nz, ny, nx)), device=DEV)
    used = []
    for precision, tol in (("fp64", 1e-13), ("mixed", 1e-5)):
        out = {}
        for sweep in ("half", "auto"):
            s = gm.GMGPoisson(a, precision=precision, fine_sweep=sweep, nu_pre=nu[0], nu_post=nu[1])
            s.profile(True)
            out[sweep] = (s.vcycle(v), s.fmg(v))
            names = set(s.profile_read())
            s.profile(False)
        used.append(any(n.startswith("sym_row_") for n in names))
        for z, r in zip(out["auto"], out["half"]):
            assert ((z - r).norm() / r.norm()).item() < tol
    if shape in ((128, 96, 96), (256, 128, 64)):
        assert used[0]


def test_row_sweep_in_a_solve():
    """From zero with the lazily scaled Krylov vector as right side (warm V-cycles)."""
    rng = np.random.default_rng(7)
    a = torch.tensor(np.exp(rng.uniform(-0.5, 0.5, (96, 96, 128)) * np.log(1e2)), device=DEV)
    f = torch.tensor(rng.standard_normal(a.shape), device=DEV)
    x0 = torch.tensor(rng.standard_normal(a.shape), device=DEV)
    out = []
    for sweep in ("auto", "half"):
        s = gm.GMGPoisson(a, precision="fp64", fine_sweep=sweep, max_iter=5)
        s.profile(True)
        out.append(s.solve(f, 0.2, 0.7, tol=0.0, x0=x0.clone()).phi)
        assert ("sym_row_first_fine_f64" in s.profile_read()) == (sweep == "auto")
    assert ((out[0] - out[1]).norm() / out[1].norm()).item() < 1e-11
