"""An encode keeps no memory for its records beyond the arrays that a step of as many particles
has, and replaces none that a captured step reads: such a step replays right after encodes,
packs and unpacks on the same context."""

import pytest
import torch

from gpu_util import ctx
from paper_1611_01545_amd.pm import widths_word

pytestmark = pytest.mark.gpu


def _float_species(c, n, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    x = torch.rand((n, 3), generator=gen, device="cuda")
    v = torch.randn((n, 3), generator=gen, device="cuda") * 0.01
    return c.float_species(x, v, 1.0 / n)


@pytest.mark.parametrize("n_cell", [8, 128])  # two and three digit passes
@pytest.mark.parametrize("pos,vel", [(1, 2), (2, 2), (1, 1)])
def test_encode_after_a_step_adds_no_record_copies(n_cell, pos, vel):
    n, w = 200_000, widths_word(pos, vel)
    c, other = ctx(2 * n_cell, n_cell), ctx(2 * n_cell, n_cell)
    data = other.pack(other.encode(_float_species(other, n, 1), cap_esc=4096, widths=w))
    other.close()
    st = c.unpack(data, n, cap_esc=4096)[0]
    c.step([st], 0.01)
    c.sync()
    before = c.scratch_bytes()
    c.encode(_float_species(c, n, 2), want_perm=True, cap_esc=4096, widths=w)
    c.sync()
    # the second copy of the keys, the digits' counts (4 bytes) and their places (8 bytes,
    # with the scan's sums) of each tile of 4096, two words and an offset per cell
    tiles = (n + 4095) // 4096
    own = 4 * n + tiles * 256 * (4 + 8 + 1) + (4 + 4 + 8) * n_cell ** 3 + 4096
    assert c.scratch_bytes() - before <= own * 9 // 8
    c.close()


@pytest.mark.parametrize("n_cell,sizes", [(8, (30011,)), (16, (2000, 300_000))])
def test_captured_step_outlives_an_encode(n_cell, sizes):
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        c, other = ctx(4 * n_cell, n_cell), ctx(4 * n_cell, n_cell)
        data = [other.pack(other.encode(_float_species(other, n, 5 + n), cap_esc=4096))
                for n in sizes]
        st = [c.unpack(d, n, cap_esc=4096)[0] for d, n in zip(data, sizes)]
        want = other.step([other.unpack(d, n, cap_esc=4096)[0] for d, n in zip(data, sizes)], 0.3)
        other.sync()
        out = c.step(st, 0.3)  # allocates what a capture may not
        c.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            c.step(st, 0.3, out=out)
        for k in range(3):
            for s in out:
                for t in (s.count, s.pos, s.vel, s.hdr):
                    t.zero_()
            for n in sizes:
                e, perm = c.encode(_float_species(c, n, 100 + k), want_perm=True, cap_esc=4096)
                assert torch.equal(c.unpack(c.pack(e), n, cap_esc=4096)[0].pos, e.pos)
            graph.replay()
            c.sync()
            for a, b in zip(out, want):
                for f in ("count", "pos", "vel", "hdr"):
                    assert torch.equal(getattr(a, f), getattr(b, f)), f
        c.close()
        other.close()
