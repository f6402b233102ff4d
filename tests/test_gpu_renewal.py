"""A renewal is queued without a wait: a refused coefficient is reported after
the whole chain has run on it, and the next renewal starts clean."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape", [(20, 24, 16), (5, 7, 9), (65, 2, 3)])  # (nz, ny, nx): three levels, one level
def test_refused_then_renewed(shape, precision):
    """Statuses as before, and after them a handle gives a fresh handle's
    solution to the bit."""
    print(f"renewal {shape} {precision}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(1)
    a = torch.rand(shape, generator=gen, dtype=torch.float64, device=DEV) + 0.5
    f = torch.rand(shape, generator=gen, dtype=torch.float64, device=DEV)
    s = gm.GMGPoisson(a, precision=precision)
    for value, status in ((float("nan"), -3), (float("inf"), -3), (0.0, -1), (-1.0, -1)):
        bad = a.clone()
        bad[-1, -1, -1] = value
        with pytest.raises(gm.GMGError) as e:
            s.update_coefficient(bad)
        assert e.value.status == status
        with pytest.raises(gm.GMGError) as e:
            gm.GMGPoisson(bad, precision=precision)
        assert e.value.status == status
    b = 2.0 * a.flip(0)
    s.update_coefficient(b)
    assert torch.equal(s.solve(f, 0.1, 0.9).phi, gm.GMGPoisson(b, precision=precision).solve(f, 0.1, 0.9).phi)
