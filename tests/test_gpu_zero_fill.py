"""A solve without a guess that ends before any update leaves phi = 0, complete
when the call returns, for a reader on any stream."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("why", ["no steps", "loose tolerance", "non-finite right side", "zero right side"])
def test_phi_is_zero_on_return(why):
    print(f"zero fill: {why}", flush=True)
    shape = (384, 384, 384)
    a = torch.ones(shape, dtype=torch.float64, device=DEV)
    f = torch.ones_like(a)
    if why == "non-finite right side":
        f[7, 5, 3] = float("inf")
    elif why == "zero right side":
        f.zero_()
    s = gm.GMGPoisson(a, restart=1, max_iter=0 if why == "no steps" else 5)
    phi = torch.full_like(f, float("nan"))
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    r = s.solve(f, 0.0, 0.0, tol=2.0 if why == "loose tolerance" else 1e-8, out=phi, raise_on_error=False)
    with torch.cuda.stream(side):
        seen = phi.clone()
    torch.cuda.synchronize()
    assert (seen == 0.0).all()
    assert r.status == {"no steps": 1, "non-finite right side": -3}.get(why, 0)
