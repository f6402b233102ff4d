"""The bottom kernel's solve of a coarsest level whose inverse does not fit LDS:
its groups of lanes at the edges of whole waves, against the oracle."""
import numpy as np
import pytest
import torch

from oracle.multigrid import build_hierarchy, fmg, vcycle

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")


# coarsest (nx, ny, nz) of three levels (2 stops the coarsening): 98 to 512
# cells, whole waves and a few cells more; five groups of lanes to one
@pytest.mark.parametrize("base", [(2, 7, 7), (2, 8, 8), (2, 5, 13), (2, 12, 8), (3, 5, 13), (2, 8, 16), (2, 3, 43),
                                  (2, 10, 16), (2, 7, 23), (2, 16, 14), (2, 9, 25), (2, 16, 16)])
def test_coarsest_solve_beyond_lds(base):
    """Tolerances of the bottom kernel's other tests: 1e-12 in float64, 2e-5 in
    float32."""
    nx, ny, nz = (4 * b for b in base)
    print(f"coarsest {base}", flush=True)
    rng = np.random.default_rng(nx + ny + nz)
    a = np.exp(rng.uniform(-0.5, 0.5, (nz, ny, nx)) * np.log(1e2))
    f = rng.standard_normal(a.shape)
    h = (1.0, 1.3, 0.9)
    for precision, dtype, tol in (("fp64", np.float64, 1e-12), ("mixed", np.float32, 2e-5)):
        s = gm.GMGPoisson(torch.tensor(a, device=DEV), h=h, precision=precision)
        assert s.levels[-1] == base and len(s.levels) == 3
        hier = build_hierarchy(a, h, dtype=dtype)
        s.profile(True)
        for fn, ref in ((s.vcycle, vcycle), (s.fmg, fmg)):
            z = fn(torch.tensor(f, device=DEV)).cpu().numpy()
            r = ref(hier, f.astype(dtype)).astype(np.float64)
            assert np.linalg.norm(z - r) <= tol * np.linalg.norm(r)
        assert any("vcycle_bottom" in k for k in s.profile_read())
