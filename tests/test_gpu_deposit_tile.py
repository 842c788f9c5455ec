"""The tiled deposit against the integer definition of its weights, bit for bit: every corner's
weight is an exact multiple of 2^-27 (2-byte codes: rounded to one), a node's sum is an integer,
and the species' sums are rounded to float32 once each and added in order. Nodes with fewer and
with more particles than a 32-bit sum holds (32), one to four species, all tile shapes."""

import numpy as np
import pytest

from gpu_util import ctx
from oracle import codec
from paper_1611_01545_amd.pm import widths_word

pytestmark = pytest.mark.gpu

# (n_mesh, n_cell): tiles of 4^3 and 8^3 cells of 16^3 nodes, and the runtime shapes: one mesh
# cell per compression cell, eight, sixteen, and a box of fewer nodes than a tile
SHAPES = [(32, 8), (64, 32), (16, 16), (64, 8), (32, 2), (8, 4)]


def _positions(kind, n, n_mesh, rng):
    if kind == "uniform":
        return rng.random((n, 3), dtype=np.float32)
    if kind == "point":  # all on one spot, whose corners straddle the periodic boundary
        return np.full((n, 3), 1.0 - 0.25 / n_mesh, dtype=np.float32)
    # "clumps": spots at tile corners and faces, in tile interiors, and a uniform part
    c = rng.integers(0, n_mesh, (6, 3)) / n_mesh
    c[0] = (0.0, 0.0, 0.0)
    c[1] = (0.5, 0.0, 0.5)
    x = c[rng.integers(0, 6, n)] + rng.normal(0.0, 0.3 / n_mesh, (n, 3))
    x[: n // 4] = rng.random((n // 4, 3))
    return ((x % 1.0) % 1.0).astype(np.float32)


def _density(state, n_mesh, unit):
    """Integer weight sums of one species, as float32 densities."""
    u, _ = codec.decode_codes(state)
    pb = int(state.get("pos_bytes", 1))
    n_cell = state["n_c"]
    r, fb = n_mesh // n_cell, 8 * pb + 1
    g = (2 * u.astype(np.int64) + 1) * r
    i, f = g >> fb, (g & ((1 << fb) - 1)).astype(np.uint64)
    one = np.uint64(1 << fb)
    w = np.zeros(n_mesh ** 3, dtype=np.uint64)
    for d in range(8):
        c = [(d >> a) & 1 for a in range(3)]
        f3 = [f[:, a] if c[a] else one - f[:, a] for a in range(3)]
        p = f3[0] * f3[1] * f3[2]
        if pb == 2:
            p = (p + np.uint64(1 << 23)) >> np.uint64(24)
        k = [(i[:, a] + c[a]) % n_mesh for a in range(3)]
        np.add.at(w, (k[2] * n_mesh + k[1]) * n_mesh + k[0], p)
    return (w.astype(np.float64) * unit).astype(np.float32).reshape((n_mesh,) * 3)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("pos_bytes", [1, 2])
@pytest.mark.parametrize("kind,sizes", [("uniform", (3000, 500)), ("point", (31, 32)),
                                        ("point", (5000,)), ("clumps", (9000, 1, 4000, 700)),
                                        ("uniform", (1,)), ("clumps", (70001, 300))])
def test_deposit_is_the_integer_sum(shape, pos_bytes, kind, sizes):
    n_mesh, n_cell = shape
    rng = np.random.default_rng(11)
    c = ctx(n_mesh, n_cell)
    w = widths_word(pos_bytes, 2)
    st, want = [], np.zeros((n_mesh,) * 3, dtype=np.float32)
    for i, n in enumerate(sizes):
        x, mass = _positions(kind, n, n_mesh, rng), (0.3 + i) / n
        s = c.encode(c.float_species(x, np.ones_like(x), mass), cap_esc=256, widths=w)
        st.append(s)
        want = want + _density(c.to_host(s), n_mesh, mass * float(n_mesh) ** 3 * 2.0 ** -27)
    got = c.deposit(st)
    c.sync()
    assert np.array_equal(got.cpu().numpy(), want)
    c.close()


def test_unaligned_mesh():
    """A density mesh that starts at any float, not at a multiple of 16 bytes."""
    import torch

    c = ctx(32, 8)
    rng = np.random.default_rng(5)
    x = rng.random((4000, 3), dtype=np.float32)
    s = c.encode(c.float_species(x, np.ones_like(x), 1.0))
    want = c.deposit([s])
    buf = torch.full((32 ** 3 + 2,), -1.0, device="cuda")
    c.deposit([s], rho=buf[1:-1])
    c.sync()
    assert torch.equal(buf[1:-1].view(32, 32, 32), want)
    assert float(buf[0]) == -1.0 and float(buf[-1]) == -1.0
    c.close()
