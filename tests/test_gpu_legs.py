"""Smoothing legs of small levels (several half-sweeps per launch, the halo
recomputed) against the oracle: boxes that tile the level exactly and with
remainders in x, y and z, full rows and x-tiles, the finest (colour-split)
level and coarse ones, one to four sweeps (one launch or a split leg), and the
largest levels that run as legs."""
import numpy as np
import pytest
import torch

from oracle.multigrid import build_hierarchy, fmg, vcycle

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")

# (nx, ny, nz); 44 x 52 x 60 over 22 x 26 x 30; 4 x 4 x 36 and 132 x 4 x 4:
# boxes larger than the level; 2 levels: no bottom kernel below the leg
SHAPES = [(64, 64, 64), (44, 52, 60), (36, 28, 20), (4, 4, 36), (132, 4, 4), (18, 22, 26), (64, 96, 80)]


def _check(shape, nu, precisions=(("fp64", np.float64, 1e-12), ("mixed", np.float32, 2e-5))):
    nx, ny, nz = shape
    print(f"legs {shape} nu {nu}", flush=True)
    rng = np.random.default_rng(nx * ny + nz)
    a = np.exp(rng.uniform(-0.5, 0.5, (nz, ny, nx)) * np.log(1e2))
    f = rng.standard_normal(a.shape)
    h = (1.0 / nx, 1.3 / ny, 0.9 / nz)
    for precision, dtype, tol in precisions:
        s = gm.GMGPoisson(torch.tensor(a, device=DEV), h=h, precision=precision, nu_pre=nu[0], nu_post=nu[1])
        hier = build_hierarchy(a, h, nu_pre=nu[0], nu_post=nu[1], dtype=dtype)
        s.profile(True)
        for fn, ref in ((s.vcycle, vcycle), (s.fmg, fmg)):
            z = fn(torch.tensor(f, device=DEV)).cpu().numpy()
            r = ref(hier, f.astype(dtype)).astype(np.float64)
            assert np.linalg.norm(z - r) <= tol * np.linalg.norm(r)
        assert any(k.startswith("leg_pre_fine") for k in s.profile_read())


@pytest.mark.parametrize("nu", [(2, 2), (1, 3)])
@pytest.mark.parametrize("shape", SHAPES)
def test_legs(shape, nu):
    """Tolerances as for the per-sweep kernels: 1e-12 in float64, 2e-5 in
    float32 (the half-sweeps' arithmetic, summed in another order)."""
    _check(shape, nu)


@pytest.mark.parametrize("nu", [(4, 1), (1, 1), (3, 5)])
def test_legs_split_into_launches(nu):
    _check((36, 28, 20), nu)


def test_largest_level_in_legs():
    """4 MiB of iterate: 2^20 cells in float32, 2^19 in float64."""
    _check((128, 128, 64), (2, 2), (("mixed", np.float32, 2e-5),))
    _check((64, 128, 64), (2, 2), (("fp64", np.float64, 1e-12),))


def test_warm_and_scaled_right_side():
    """Inside a solve the finest leg reads the Krylov vector times its scale
    and stores the right side for the post-smoothing: the float64 solve
    agrees with the per-sweep kernels' to rounding at a fixed step count."""
    rng = np.random.default_rng(3)
    a = np.exp(rng.uniform(-0.5, 0.5, (40, 48, 64)) * np.log(1e2))
    f = torch.tensor(rng.standard_normal(a.shape), device=DEV)
    x0 = torch.tensor(rng.standard_normal(a.shape), device=DEV)
    for warm in ("vcycle", "fmg"):
        out = []
        for sweep in ("auto", "half"):
            s = gm.GMGPoisson(torch.tensor(a, device=DEV), precision="fp64", fine_sweep=sweep, max_iter=5,
                              warm_cycle=warm)
            out.append(s.solve(f, 0.2, 0.7, tol=0.0, x0=x0).phi.cpu().numpy())
        assert np.linalg.norm(out[0] - out[1]) <= 1e-11 * np.linalg.norm(out[1])
