"""The force gradient pass and its max |a| at every launch shape it has below 1024^3 (mesh
sides 8 to 512): the components against the float64 operator on the same density, within
the force tolerance (relative RMS 1e-4), and max |a| against the components themselves."""

import pytest
import torch

from gpu_util import ctx
from oracle import fp64_torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 16, 32, 64, 128, 256, 512])
def test_force_components_and_max(n):
    c = ctx(n, max(1, n // 4))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    rho = torch.rand((n, n, n), generator=gen, device="cuda")
    for scale in (0.25, 1.0, 0.5):  # each call clears the maximum of the one before
        acc, a_max = c.force(rho * scale)
        c.sync()
        assert float(a_max) == float(acc.abs().max())
    rhok = fp64_torch.spectrum((rho * 0.5).double(), slab=min(n, 32))
    for axis in range(3):
        want = fp64_torch.force_component(rhok, axis, slab=min(n, 32))
        err = ((acc[axis].double() - want) ** 2).mean() / (want ** 2).mean()
        assert float(err) ** 0.5 <= 1e-4
    c.close()
