"""The rules that spare a tile of the deposit its check or its 32-bit sums: particles of the eight
cells around a node, as many as no pair of neighbours, or just one, of more than seven leaves
unchecked, and far more, at every place of a tile; and cells around the count from which a tile
takes 64-bit sums at once. Against the integer sums of the exact weights."""

import numpy as np
import pytest
import torch

from gpu_util import ctx
from oracle import codec
from paper_1611_01545_amd.pm import widths_word
from test_gpu_deposit_tile import _density

pytestmark = pytest.mark.gpu


def _check(c, xs, pos_bytes):
    st, want = [], np.zeros((c.n_mesh,) * 3, dtype=np.float32)
    for i, x in enumerate(xs):
        x = x.astype(np.float32)
        s = c.encode(c.float_species(x, np.ones_like(x), (0.3 + i) / len(x)), cap_esc=256,
                     widths=widths_word(pos_bytes, 2))
        st.append(s)
        want = want + _density(c.to_host(s), c.n_mesh,
                               s.mass * float(c.n_mesh) ** 3 * 2.0 ** -27)
    got = c.deposit(st)
    c.sync()
    assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("n_mesh,n_cell", [(64, 16), (64, 32), (16, 16), (64, 8)])
@pytest.mark.parametrize("pos_bytes", [1, 2])
@pytest.mark.parametrize("species", [1, 2, 3])
def test_particles_around_a_node(n_mesh, n_cell, pos_bytes, species):
    """Counts (a, b) of the two cells of each pair along x, all of them next to the node, which
    is the corner of eight cells; every place of the corner in a tile."""
    rng = np.random.default_rng(3)
    c = ctx(n_mesh, n_cell)
    step = 1.0 / (256 * n_cell)
    for a, b in ((4, 3), (3, 4), (7, 0), (4, 4), (5, 5), (20, 20)):
        for corner in rng.integers(0, n_cell, (12, 3)):
            xs = []
            for k in range(species):
                x = []
                for dz in (-1, 1):
                    for dy in (-1, 1):
                        for dx, n in ((-1, a), (1, b)):
                            off = np.array([dx, dy, dz]) * step * (0.3 + 0.5 * rng.random((n, 3)))
                            x.append((corner / n_cell + off) % 1.0)
                xs.append(np.concatenate(x + [rng.random((5, 3))]))
            _check(c, xs, pos_bytes)
    c.close()


@pytest.mark.parametrize("n_mesh,n_cell", [(64, 16), (64, 32), (16, 16), (64, 8)])
@pytest.mark.parametrize("pos_bytes", [1, 2])
@pytest.mark.parametrize("others", [(), (700,), (700, 50)])
def test_cells_at_the_count_of_64_bit_sums(n_mesh, n_cell, pos_bytes, others):
    r = n_mesh // n_cell
    rng = np.random.default_rng(4)
    c = ctx(n_mesh, n_cell)
    for n in (16 * r ** 3 + 47, 16 * r ** 3 + 48, 16 * r ** 3 + 49):
        for shrink in (0.96, 0.2):  # all over the cell, and together
            cell = rng.integers(0, n_cell, 3)
            xs = [(cell + 0.02 + shrink * rng.random((n, 3))) / n_cell]
            xs += [rng.random((k, 3)) for k in others]
            _check(c, xs, pos_bytes)
    c.close()
