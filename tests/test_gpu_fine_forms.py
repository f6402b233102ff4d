"""Which kernels smooth the finest level by default, and the row sweep in both
precisions against the half-sweeps where it is the default."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")
FORMS = {"leg": ("leg_pre_fine", "leg_post_fine"), "half": ("gs_fine",), "row": ("sym_row_fine", "sym_row_first_fine"),
         "split": ("sym_fine", "sym_first_fine", "sym_resid_fine")}


def _form(s):
    """Names of the finest level's smoothing kernels, as one of FORMS."""
    names = {n.rsplit("_", 1)[0] for n in s.profile_read()}
    used = [form for form, base in FORMS.items() if names & set(base)]
    assert len(used) == 1, (used, names)
    return used[0]


def _problem(shape):
    nx, ny, nz = shape
    gen = torch.Generator(device=DEV).manual_seed(nx + 3 * ny + 7 * nz)
    draw = lambda: torch.rand((nz, ny, nx), generator=gen, dtype=torch.float64, device=DEV)  # noqa: E731
    return torch.exp((draw() - 0.5) * np.log(1e2)), draw() - 0.5, draw()


# (nx, ny, nz): float32, float64.  Legs up to 4 MiB per iterate; rows of 64 and
# 128 pairs by the row sweep; longer rows by the 62-pair tiles.
@pytest.mark.parametrize("shape,f32,f64", [
    ((64, 64, 64), "leg", "leg"), ((128, 96, 96), "row", "row"), ((128, 128, 128), "row", "row"),
    ((256, 256, 256), "row", "row"), ((384, 384, 384), "split", "split")])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_default_kernels(shape, f32, f64, precision):
    print(f"default kernels {shape} {precision}", flush=True)
    a, v, _ = _problem(shape)
    s = gm.GMGPoisson(a, precision=precision, restart=1)
    s.profile(True)
    s.vcycle(v)
    assert _form(s) == (f32 if precision == "mixed" else f64)


@pytest.mark.parametrize("shape", [(128, 96, 96), (112, 112, 96), (256, 128, 64)])
def test_row_sweep_in_a_mixed_solve(shape):
    """From zero with the lazily scaled Krylov vector (float64) as right side of
    the float32 sweep.  The preconditioners differ by float32 rounding (1e-5
    of their results, the sweeps' tolerance), which each of the five steps of a
    converging solve carries into its part of the solution: 5e-5 of the first
    correction in all."""
    print(f"row sweep in a mixed solve {shape}", flush=True)
    a, f, x0 = _problem(shape)
    out = []
    for sweep in ("auto", "half"):
        s = gm.GMGPoisson(a, precision="mixed", fine_sweep=sweep, max_iter=5)
        s.profile(True)
        out.append(s.solve(f, 0.2, 0.7, tol=0.0, x0=x0.clone()).phi)
        assert _form(s) == ("row" if sweep == "auto" else "half")
        assert ("sym_row_first_fine_f32" in s.profile_read()) == (sweep == "auto")
    assert ((out[0] - out[1]).norm() / (out[1] - x0).norm()).item() < 5e-5
