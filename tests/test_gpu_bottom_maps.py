"""Bottom kernel over a 4 x 4 x 4 level (its cycles as precomputed maps) and its
packed pairs, against the oracle, before and after a new coefficient."""
import numpy as np
import pytest
import torch

from oracle.multigrid import build_hierarchy, fmg, vcycle

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")


# maps below one and two smoothed bottom levels and below a level outside the
# bottom; no maps: the 4 x 4 x 4 level first of the bottom, another coarsest
@pytest.mark.parametrize("nu", [(2, 2), (0, 2), (1, 0)])
@pytest.mark.parametrize("shape", [(16, 16, 16), (32, 32, 32), (64, 64, 64), (8, 8, 8), (16, 16, 24)])
def test_maps_and_packed_pairs(shape, nu):
    """Tolerances of the same cycles run phase by phase: 1e-12 in float64 (some
    1e3 roundings amplified by the coarse solves), 2e-5 in float32; a column of
    a map carries the same roundings, its product 64 more of each sum."""
    nx, ny, nz = shape
    print(f"maps {shape} nu {nu}", flush=True)
    rng = np.random.default_rng(nx + nz)
    coef = [np.exp(rng.uniform(-0.5, 0.5, (nz, ny, nx)) * np.log(c)) for c in (1e2, 1e3)]
    f = rng.standard_normal((nz, ny, nx))
    h = (1.0 / nx, 1.3 / ny, 0.9 / nz)
    for precision, dtype, tol in (("fp64", np.float64, 1e-12), ("mixed", np.float32, 2e-5)):
        s = gm.GMGPoisson(torch.tensor(coef[0], device=DEV), h=h, precision=precision, nu_pre=nu[0], nu_post=nu[1])
        for a in coef:
            s.update_coefficient(torch.tensor(a, device=DEV))
            hier = build_hierarchy(a, h, nu_pre=nu[0], nu_post=nu[1], dtype=dtype)
            for fn, ref in ((s.vcycle, vcycle), (s.fmg, fmg)):
                z = fn(torch.tensor(f, device=DEV)).cpu().numpy()
                r = ref(hier, f.astype(dtype)).astype(np.float64)
                assert np.linalg.norm(z - r) <= tol * np.linalg.norm(r)


@pytest.mark.parametrize("shape,precision", [((112, 72, 40), "fp64"), ((120, 88, 40), "mixed")])
def test_packed_pairs_need_no_more_workspace(shape, precision):
    """Grids whose workspace comes within 256 KiB of the library's static array
    (which refuses larger ones): packed pairs and maps lie in the partials'
    tail, and the solve on the array equals the solve on a workspace."""
    nx, ny, nz = shape
    print(f"static limit {shape} {precision}", flush=True)
    rng = np.random.default_rng(nx)
    a = torch.tensor(np.exp(rng.uniform(-0.5, 0.5, (nz, ny, nx)) * np.log(1e2)), device=DEV)
    f = torch.tensor(rng.standard_normal((nz, ny, nx)), device=DEV)
    s = gm.GMGPoisson(a, precision=precision)
    limit = 64 << 20
    assert limit - (256 << 10) - 4096 < s.workspace_bytes <= limit
    out = torch.empty_like(f)
    r = gm.fgmres_solve_static(a, f, 0.2, 0.7, 1e-8, out=out, precision=precision)
    assert torch.equal(r.phi, s.solve(f, 0.2, 0.7, tol=1e-8).phi)
