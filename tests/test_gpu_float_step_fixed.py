"""A float step, whose transform reads the deposit's fixed-point sums, equals the step of its
pieces, which goes through the float density mesh, bit for bit; also when it is replayed from a
captured graph with eager deposits between the replays, which leave their sums in the mesh."""

import pytest
import torch

from gpu_util import ctx

pytestmark = pytest.mark.gpu


def species(c, sizes, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    out = []
    for i, n in enumerate(sizes):
        x = torch.rand((n, 3), generator=gen, device="cuda")
        v = torch.randn((n, 3), generator=gen, device="cuda") * 0.01
        out.append(c.float_species(x, v, (1.0 + i) / n))
    return out


def pieces(c, st, dt):
    acc, a_max = c.force(c.deposit(st))
    return c.kick_drift(st, acc, a_max, dt, dt)


def check(got, want):
    for a, b in zip(got, want):
        assert torch.equal(a.x, b.x) and torch.equal(a.v, b.v)


@pytest.mark.parametrize("n_mesh", [32, 64, 128, 256, 512, 1024])
@pytest.mark.parametrize("sizes", [(1,), (30011, 4097)])
def test_float_step_equals_its_pieces(n_mesh, sizes):
    c = ctx(n_mesh, n_mesh // 4)
    for seed in (1, 2):  # the second call finds the first one's sums
        st = species(c, sizes, seed)
        got, want = c.step(st, 0.3), pieces(c, st, 0.3)
        c.sync()
        check(got, want)
    c.close()


def test_float_step_in_a_graph():
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        c = ctx(64, 16)
        st = species(c, (5000, 77), 3)
        other = species(c, (4000,), 4)
        want = pieces(c, st, 0.3)
        out = c.step(st, 0.3)  # allocates what a capture may not
        c.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            c.step(st, 0.3, out=out)
        for _ in range(4):
            for s in out:
                s.x.zero_()
                s.v.zero_()
            graph.replay()
            c.sync()
            check(out, want)
            c.deposit(other)
            c.sync()
        c.close()
