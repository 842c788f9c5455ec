"""Tiles whose cells hold more particles than 32-bit node sums can: the count at which the deposit
goes to 64-bit sums at once, one below and one above it, in cells at a tile's first corner and its
last one, which are also a neighbour's shell; alone, and as one of two and of three species."""

import numpy as np
import pytest

from gpu_util import ctx
from paper_1611_01545_amd.pm import widths_word
from test_gpu_deposit_tile import _density

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_mesh,n_cell", [(32, 8), (64, 32), (16, 16), (64, 8)])
@pytest.mark.parametrize("pos_bytes", [1, 2])
@pytest.mark.parametrize("cell", [0, -1])
@pytest.mark.parametrize("others", [(), (600,), (600, 50)])
def test_crowded_cell(n_mesh, n_cell, pos_bytes, cell, others):
    r = n_mesh // n_cell
    most = 32 * (r + 1) ** 3 + 32
    rng = np.random.default_rng(17)
    c = ctx(n_mesh, n_cell)
    for n in (most - 1, most, most + 1, 3 * most):
        st, want = [], np.zeros((n_mesh,) * 3, dtype=np.float32)
        for i, k in enumerate((n,) + others):
            x = rng.random((k, 3)) * 0.98 + 0.01
            if i == 0:  # all in one cell
                x = (x + cell % n_cell) / n_cell
            x, mass = x.astype(np.float32), (0.3 + i) / k
            s = c.encode(c.float_species(x, np.ones_like(x), mass), cap_esc=256,
                         widths=widths_word(pos_bytes, 2))
            st.append(s)
            want = want + _density(c.to_host(s), n_mesh, mass * float(n_mesh) ** 3 * 2.0 ** -27)
        got = c.deposit(st)
        c.sync()
        assert np.array_equal(got.cpu().numpy(), want), n
    c.close()
