"""The pair-lane operator (y = A x - lifting) against the oracle at the edges
of its 64-pair tiles, its rows of four and its z-chunks."""
import numpy as np
import pytest
import torch

from oracle.operator import apply_operator

pytestmark = pytest.mark.gpu

import paper_1812_08606_amd as gm  # noqa: E402  (fails loudly if the library is missing)

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("shape", [(2, 2, 2), (2, 1, 9), (126, 4, 2), (128, 6, 4), (130, 8, 10), (258, 4, 2)])
def test_apply_pairs(shape, offset):
    """Each value is a sum of six products of a few roundings each: 1e-14 of
    the largest magnitude summed.  offset 1: a buffer 8 bytes past a 16-byte
    boundary, which takes the one-cell kernel."""
    nx, ny, nz = shape
    print(f"apply {shape} offset {offset}", flush=True)
    rng = np.random.default_rng(nx + nz)
    a = np.exp(rng.uniform(-0.5, 0.5, (nz, ny, nx)) * np.log(1e2))
    x = rng.standard_normal(a.shape)
    h = (1.0 / nx, 1.3 / ny, 0.9 / nz)
    buf = torch.empty(x.size + 1, dtype=torch.float64, device=DEV)
    xd = buf[offset:offset + x.size].view(x.shape)
    xd.copy_(torch.tensor(x))
    s = gm.GMGPoisson(torch.tensor(a, device=DEV), h=h, precision="fp64")
    y = s.apply(xd, 0.3, -1.2).cpu().numpy()
    ref = apply_operator(x, a, h, 0.3, -1.2)
    scale = (np.abs(x).max() + 1.2) * a.max() * 4 * sum(1 / d ** 2 for d in h)
    assert np.all(np.abs(y - ref) <= 1e-14 * scale)
