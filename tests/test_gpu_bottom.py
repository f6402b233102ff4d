"""The one-workgroup bottom of the cycles against the oracle, at the shapes
where its pair ownership and coarsest solve change: a full first level (2048
pairs), several pairs per thread with a remainder, one to three smoothed
levels, coarsest inverses in LDS (up to 128 cells in float32, 96 in float64)
and beyond."""
import numpy as np
import pytest
import torch

from oracle.multigrid import build_hierarchy, fmg, vcycle

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")

# (nx, ny, nz): bottom levels 16^3 8^3 4^3 2^3; 32 x 16 x 8 ... 8 x 4 x 2;
# 14 x 14 x 14 over 7^3 (343 cells); 10 x 18 x 22 over 5 x 9 x 11; 12 x 20 x 12
# over 6 x 10 x 6 and 3 x 5 x 3; 8 x 8 x 64 (long z) ... 2 x 2 x 16; 6 x 4 x 10 over 3 x 2 x 5;
# 4 x 5 x 20 (400 cells) and 4 x 4 x 5 (80 cells) coarsest
SHAPES = [(16, 20, 80), (16, 16, 20), (32, 32, 32), (64, 32, 16), (28, 28, 28), (20, 36, 44), (24, 40, 24), (16, 16, 128), (12, 8, 20)]


@pytest.mark.parametrize("nu", [(2, 2), (0, 1), (1, 0), (2, 3)])
@pytest.mark.parametrize("shape", SHAPES)
def test_bottom_levels(shape, nu):
    """Tolerances of the same operations on other shapes: 1e-12 in float64
    (some 1e3 roundings amplified by the coarse solves), 2e-5 in float32
    (the same count of float32 ones)."""
    nx, ny, nz = shape
    print(f"bottom {shape} nu {nu}", flush=True)
    rng = np.random.default_rng(nx * ny + nz)
    a = np.exp(rng.uniform(-0.5, 0.5, (nz, ny, nx)) * np.log(1e2))
    f = rng.standard_normal(a.shape)
    h = (1.0 / nx, 1.3 / ny, 0.9 / nz)
    for precision, dtype, tol in (("fp64", np.float64, 1e-12), ("mixed", np.float32, 2e-5)):
        s = gm.GMGPoisson(torch.tensor(a, device=DEV), h=h, precision=precision, nu_pre=nu[0], nu_post=nu[1])
        hier = build_hierarchy(a, h, nu_pre=nu[0], nu_post=nu[1], dtype=dtype)
        assert [tuple(lv.shape) for lv in hier.levels] == s.levels and len(s.levels) >= 3
        s.profile(True)
        for fn, ref in ((s.vcycle, vcycle), (s.fmg, fmg)):
            z = fn(torch.tensor(f, device=DEV)).cpu().numpy()
            r = ref(hier, f.astype(dtype)).astype(np.float64)
            assert np.linalg.norm(z - r) <= tol * np.linalg.norm(r)
        assert any("vcycle_bottom" in k for k in s.profile_read())
