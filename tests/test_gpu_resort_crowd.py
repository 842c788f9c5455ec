"""The re-sort of crowded states: escapes in many tiles of bricks. With a zero force the new
position codes are u + floor(v c_d S + 1/2) exactly, and the stream has to be the stable sort
of the old one by the new cells."""

import numpy as np
import pytest
import torch

from gpu_util import ctx
from oracle import codec

pytestmark = pytest.mark.gpu


def _check(n_mesh, n_cell, brick, loads, cap_esc=4096):
    """loads: (x, to) per species; the kick moves particles from x to `to`."""
    c = ctx(n_mesh, n_cell, brick=brick)
    st = [c.encode(c.float_species(x.astype(np.float32), (to - x).astype(np.float32), 1.0),
                   cap_esc=cap_esc) for x, to in loads]
    acc = torch.zeros((3, n_mesh, n_mesh, n_mesh), device="cuda")
    a_max = torch.zeros(1, device="cuda")
    out, perms = c.kick_drift_perm(st, acc, a_max, 1.0, 1.0)
    c.sync()
    S = codec.pos_scale(n_cell)
    for s, o, p in zip(st, out, perms):
        old, new = c.to_host(s), c.to_host(o)
        u, _ = codec.decode_codes(old)
        u1 = (u + np.floor(codec.decode(old)[1].astype(np.float64) * S + 0.5)
              .astype(np.int64)) % S
        keys = codec.cell_keys(u1 >> 8, n_cell, brick)
        order = np.argsort(keys, kind="stable")
        assert np.array_equal(p.cpu().numpy(), order)
        un, _ = codec.decode_codes(new)
        assert np.array_equal(un, u1[order])
        cnt, esc = codec.build_counts(keys[order], n_cell)
        assert np.array_equal(new["count"], cnt)
        assert np.array_equal(new["esc"], np.asarray(esc, dtype=np.uint64).reshape(-1, 2))
        assert new["j_min"] == new["vel"].min() and new["j_max"] == new["vel"].max()
    c.close()


# 8 and 512 tiles of 4096 bricks
@pytest.mark.parametrize("n_mesh,n_cell,brick", [(64, 64, 2), (128, 128, 1)])
def test_escapes_all_over_the_box(n_mesh, n_cell, brick):
    rng = np.random.default_rng(5)
    loads = []
    for clumps in (40, 1):
        cells = rng.integers(0, n_cell, (clumps, 3))
        cells[0] = n_cell - 1  # the last tile
        to = np.concatenate([(np.repeat(cells, 300, axis=0) +
                              0.02 + 0.96 * rng.random((300 * clumps, 3))) / n_cell,
                             rng.random((20000, 3))])
        x = (to + rng.normal(0.0, 1.5 * brick / n_cell, to.shape)) % 1.0
        keep = rng.permutation(len(x))
        loads.append((x[keep], to[keep]))
    _check(n_mesh, n_cell, brick, loads)
