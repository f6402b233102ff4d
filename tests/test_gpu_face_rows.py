"""The fused symmetric sweep of the coarse levels in blocks of eight rows of one
wave (six rows own cells), against the half-sweep kernels."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")


# level 1 of nx / 2 x ny / 2 x nz / 2 cells: 12 rows (two blocks), 4 rows (less
# than one), 14 and 40 rows (remainders of two and four); 64 and fewer pairs
@pytest.mark.parametrize("shape", [(256, 24, 32), (128, 8, 64), (128, 28, 32), (96, 80, 16)])
def test_fused_rows_match_half_sweeps(shape):
    """The same arithmetic face by face, contracted differently: 1e-13 in
    float64, 1e-5 in float32 (the fused sweeps' tolerances)."""
    nx, ny, nz = shape
    print(f"face rows {shape}", flush=True)
    rng = np.random.default_rng(nx + ny + nz)
    a = torch.tensor(np.exp(rng.uniform(-0.5, 0.5, (nz, ny, nx)) * np.log(1e2)), device=DEV)
    v = torch.tensor(rng.standard_normal((nz, ny, nx)), device=DEV)
    for precision, tol, sfx in (("fp64", 1e-13, "f64"), ("mixed", 1e-5, "f32")):
        out = {}
        for sweep in ("half", "fused"):
            s = gm.GMGPoisson(a, precision=precision, fine_sweep=sweep)
            s.profile(True)
            out[sweep] = (s.vcycle(v), s.fmg(v))
            assert ("sym_L1_" + sfx in s.profile_read()) == (sweep == "fused")
        for z, r in zip(out["fused"], out["half"]):
            assert ((z - r).norm() / r.norm()).item() < tol


# level 1 by default fused from 2^19 cells where a row fills more than half of
# one wave (legs run up to 2^20 cells in float32, 2^19 in float64)
@pytest.mark.parametrize("shape,fused", [((176, 208, 240), (True, True)), ((128, 320, 256), (False, False)),
                                         ((144, 192, 160), (False, True)), ((272, 160, 160), (False, False))])
def test_default_level_one_sweeps(shape, fused):
    """Which sweeps the default takes, and its V-cycle against half-sweeps
    (tolerances as above)."""
    nx, ny, nz = shape
    print(f"default sweeps {shape}", flush=True)
    rng = np.random.default_rng(nx + ny + nz)
    a = torch.tensor(np.exp(rng.uniform(-0.5, 0.5, (nz, ny, nx)) * np.log(1e2)), device=DEV)
    v = torch.tensor(rng.standard_normal((nz, ny, nx)), device=DEV)
    for precision, tol, sfx, want in (("mixed", 1e-5, "f32", fused[0]), ("fp64", 1e-13, "f64", fused[1])):
        out = {}
        for sweep in ("half", "auto"):
            s = gm.GMGPoisson(a, precision=precision, fine_sweep=sweep)
            s.profile(True)
            out[sweep] = s.vcycle(v)
            assert ("sym_L1_" + sfx in s.profile_read()) == (sweep == "auto" and want)
        assert ((out["auto"] - out["half"]).norm() / out["half"].norm()).item() < tol
