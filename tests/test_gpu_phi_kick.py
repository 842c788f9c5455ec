"""A step whose kick reads the potential equals the step of its pieces, whose kick reads the
three force meshes, bit for bit: meshes of two and more bricks per side (the tile's ring of
planes wraps, and its halo crosses the box), all code widths, one to three species."""

import pytest
import torch

from gpu_util import ctx
from paper_1611_01545_amd.pm import widths_word

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_mesh", [32, 64, 128, 256])
@pytest.mark.parametrize("pos,vel", [(1, 2), (2, 2), (1, 1), (2, 1)])
@pytest.mark.parametrize("sizes", [(1,), (5000, 700), (30011, 1, 4096)])
def test_step_equals_its_pieces(n_mesh, pos, vel, sizes):
    c = ctx(n_mesh, n_mesh // 4)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    st = []
    for i, n in enumerate(sizes):
        x = torch.rand((n, 3), generator=gen, device="cuda")
        x[: n // 3] = 0.999 - 0.02 * x[: n // 3]  # a clump at the corner of the box
        v = torch.randn((n, 3), generator=gen, device="cuda") * (2.0 / n_mesh)
        st.append(c.encode(c.float_species(x, v, (1.0 + i) / n), cap_esc=4096,
                           widths=widths_word(pos, vel)))
    got = c.step(st, 0.3)
    acc, a_max = c.force(c.deposit(st))
    want = c.kick_drift(st, acc, a_max, 0.3, 0.3)
    c.sync()
    for a, b in zip(got, want):
        for f in ("count", "pos", "vel", "hdr"):
            assert torch.equal(getattr(a, f), getattr(b, f)), f
    c.close()
