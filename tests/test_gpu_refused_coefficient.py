"""Between a refused coefficient and the next renewal a handle has no
hierarchy: whatever would read it reports the refusal and writes nothing."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("value,status", [(float("nan"), -3), (0.0, -1), (-1.0, -1)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape", [(20, 24, 16), (5, 7, 9)])  # (nz, ny, nx): three levels, one level
def test_calls_after_a_refused_coefficient(shape, precision, value, status):
    print(f"refused {shape} {precision} {value}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(3)
    a = torch.rand(shape, generator=gen, dtype=torch.float64, device=DEV) + 0.5
    f = torch.rand(shape, generator=gen, dtype=torch.float64, device=DEV)
    s = gm.GMGPoisson(a, precision=precision)
    phi = s.solve(f, 0.1, 0.9).phi
    field = s.electric_field(phi, 0.1, 0.9)
    bad = a.clone()
    bad[-1, -1, -1] = value
    with pytest.raises(gm.GMGError):
        s.update_coefficient(bad)
    out = torch.full_like(f, 7.0)
    guess = torch.full_like(f, 7.0)
    for call in (lambda: s.solve(f, 0.1, 0.9, out=out), lambda: s.solve(f, 0.1, 0.9, x0=guess, out=guess),
                 lambda: s.krylov_solve(f, 0.1, 0.9, "bicgstab"), lambda: s.krylov_solve(f, 0.1, 0.9, "gmres"), lambda: s.apply(f),
                 lambda: s.vcycle(f), lambda: s.fmg(f)):
        with pytest.raises(gm.GMGError) as e:
            call()
        assert e.value.status == status
    assert (out == 7.0).all() and (guess == 7.0).all()
    # what does not read the coefficient still answers
    for got, want in zip(s.electric_field(phi, 0.1, 0.9), field):
        assert torch.equal(got, want)
    s.update_coefficient(a)
    assert torch.equal(s.solve(f, 0.1, 0.9).phi, phi)
