"""pm_unpack around the edges of its device memory: bodies at the 1 MB that go through the
context's own room, more cell runs than a launch's table holds, and one cell of more records
than an upload takes, whose records are cut at an upload's end."""

import pytest
import torch

from gpu_util import ctx
from paper_1611_01545_amd.pm import widths_word

pytestmark = pytest.mark.gpu


def _round_trip(n_mesh, n_cell, n, pos=1, vel=2, one_cell=False):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    c = ctx(n_mesh, n_cell)
    x = torch.rand((n, 3), generator=gen, device="cuda")
    if one_cell:
        x = 0.5 + x * (0.99 / n_cell)
    v = torch.randn((n, 3), generator=gen, device="cuda")
    s = c.encode(c.float_species(x, v, 0.25), cap_esc=4096, widths=widths_word(pos, vel))
    data = c.pack(s, 5)
    back, sid = c.unpack(data, n, cap_esc=4096)
    assert sid == 5 and back.mass == 0.25
    for f in ("count", "pos", "vel", "hdr"):
        assert torch.equal(getattr(back, f), getattr(s, f)), f
    ne = s.header()["n_esc"]
    assert torch.equal(back.esc[:ne], s.esc[:ne])
    c.close()
    return len(data) - 64


@pytest.mark.parametrize("extra", [-1, 0, 1, 2])
def test_bodies_around_the_contexts_room(extra):
    # 32^3 count bytes and 9 a particle: 1 MB is 112867.6 particles
    body = _round_trip(64, 32, 112867 + extra)
    assert abs(body - (1 << 20)) < 32


@pytest.mark.parametrize("pos,vel", [(1, 2), (2, 2), (1, 1)])
def test_more_runs_than_a_table(pos, vel):
    assert 256 ** 3 // 64 > 65536
    _round_trip(256, 256, 100_003, pos, vel)


@pytest.mark.parametrize("n_cell", [2, 16])
def test_a_cell_longer_than_an_upload(n_cell):
    body = _round_trip(16, n_cell, 60_000_001, one_cell=True)
    assert body > 2 * (256 << 20)
