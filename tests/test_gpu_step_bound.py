"""The velocity bound of a compressed step that kicks from the potential. Its gradient pass only
finds the largest |a|, in launch shapes of its own, and the bound is rounded up to a power of
two, so the maximum is compared by steps dt just below and just above 2^k / max |a| of the stored
force meshes: v_max' is 2^k for one and 2^(k + 1) for the other only if the two maxima agree to
1e-9. A clump of the particles puts the largest |a| at the edges of the pass's tiles."""

import math

import pytest
import torch

from gpu_util import ctx

pytestmark = pytest.mark.gpu


def _corners(n_mesh):
    n = n_mesh
    return [(0, 0, 0), (n - 1, n - 1, n - 1), (n // 2, 3, 4), (n - 2, 16, n // 2 - 1),
            (5, n - 3, 31 % n), (n // 4 + 1, n // 2 - 1, n // 2 + 2)]


@pytest.mark.parametrize("n_mesh", [32, 64, 128, 256, 512, 1024, 2048])
def test_bound_is_the_largest_force(n_mesh):
    c = ctx(n_mesh, n_mesh // 4)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_mesh)
    for node in _corners(n_mesh)[: 1 if n_mesh == 2048 else 6]:
        x = torch.rand((2000, 3), generator=gen, device="cuda")
        at = torch.tensor(node, device="cuda", dtype=torch.float32) + 0.5
        x[:500] = (at + 0.3 * x[:500]) / n_mesh % 1.0
        st = [c.encode(c.float_species(x, torch.zeros_like(x), 1.0 / 2000), cap_esc=64)]
        acc = torch.empty((3,) + (n_mesh,) * 3, device="cuda")
        a_max = c.force(c.deposit(st, acc[0]), acc)[1]
        a = float(a_max.item())
        assert a == max(max(float(t.max()), -float(t.min())) for t in acc)
        del acc
        torch.cuda.empty_cache()
        k = round(math.log2(a)) - 12
        for dt, want in ((2.0 ** k / a * (1 - 1e-9), 2.0 ** k),
                         (2.0 ** k / a * (1 + 1e-9), 2.0 ** (k + 1))):
            out = c.step(st, dt)
            c.sync()
            assert float(out[0].header()["v_max"]) == want, (node, dt * a)
    c.close()
    torch.cuda.empty_cache()
