"""The re-sort of a compressed kick, for every form of it (one wave or four per brick, arrival
lists sorted in LDS or in memory, with and without cells of 255 particles and more): with a
zero force the new position codes are u + floor(v c_d S + 1/2) exactly, and the stream has
to be the stable sort of the old one by the new cells."""

import numpy as np
import pytest
import torch

from gpu_util import ctx
from oracle import codec

pytestmark = pytest.mark.gpu

# (n_mesh, n_cell, brick): 16-node bricks of 4^3 and 8^3 cells, odd shapes down to one cell
SHAPES = [(64, 16, 4), (64, 32, 8), (32, 16, 8), (64, 16, 2), (32, 8, 1), (16, 4, 4), (64, 64, 8),
          (256, 128, 2)]


def _particles(kind, n, n_cell, brick, rng):
    x = rng.random((n, 3), dtype=np.float32)
    if kind == "gather":  # every particle ends in one brick: lists far beyond the LDS sort
        to = (0.5 + rng.random((n, 3)) * (brick / n_cell)) % 1.0
    elif kind == "cells":  # and in a few of its cells: counts beyond 255
        to = (0.25 + rng.integers(0, 2, (n, 3)) / n_cell + 1e-3) % 1.0
    elif kind == "shuffle":  # anywhere
        to = rng.random((n, 3))
    else:  # "drift": few leave their brick
        to = x + rng.normal(0.0, 0.1 / n_cell, (n, 3))
    return x, (to - x).astype(np.float32)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind,n", [("gather", 5000), ("cells", 3001), ("shuffle", 20011),
                                    ("drift", 40000), ("drift", 1)])
def test_resort_is_the_stable_sort_by_new_cell(shape, kind, n):
    n_mesh, n_cell, brick = shape
    rng = np.random.default_rng(7)
    c = ctx(n_mesh, n_cell, brick=brick)
    st = []
    for size in (n, max(1, n // 3)):  # two species of different lengths in one call
        x, v = _particles(kind, size, n_cell, brick, rng)
        st.append(c.encode(c.float_species(x, v, 1.0 / size), cap_esc=64))
    acc = torch.zeros((3, n_mesh, n_mesh, n_mesh), device="cuda")
    a_max = torch.zeros(1, device="cuda")
    out, perms = c.kick_drift_perm(st, acc, a_max, 1.0, 1.0)
    again = c.kick_drift(st, acc, a_max, 1.0, 1.0)
    c.sync()
    S = codec.pos_scale(n_cell)
    for s, o, p, o2 in zip(st, out, perms, again):
        old, new = c.to_host(s), c.to_host(o)
        u, j = codec.decode_codes(old)
        vel = codec.decode(old)[1].astype(np.float64)
        u1 = (u + np.floor(vel * S + 0.5).astype(np.int64)) % S
        keys = codec.cell_keys(u1 >> 8, n_cell, brick)
        order = np.argsort(keys, kind="stable")
        assert np.array_equal(p.cpu().numpy(), order)
        un, _ = codec.decode_codes(new)
        assert np.array_equal(un, u1[order])
        cnt, esc = codec.build_counts(keys[order], n_cell)
        assert np.array_equal(new["count"], cnt)
        assert np.array_equal(new["esc"], np.asarray(esc, dtype=np.uint64).reshape(-1, 2))
        assert new["j_min"] == new["vel"].min() and new["j_max"] == new["vel"].max()
        for t in ("count", "pos", "vel"):  # the order of the atomics does not show
            assert torch.equal(getattr(o, t), getattr(o2, t))
    c.close()


def test_more_bricks_than_one_scan_block():
    """32^3 one-cell bricks: the block sums of the scans over cells and over bricks."""
    c = ctx(64, 32, brick=1)  # 32768 bricks
    rng = np.random.default_rng(3)
    x, v = _particles("shuffle", 50021, 32, 1, rng)
    st = [c.encode(c.float_species(x, v, 1.0))]
    acc = torch.zeros((3, 64, 64, 64), device="cuda")
    out, perms = c.kick_drift_perm(st, acc, torch.zeros(1, device="cuda"), 1.0, 1.0)
    c.sync()
    old = c.to_host(st[0])
    u, _ = codec.decode_codes(old)
    u1 = (u + np.floor(codec.decode(old)[1].astype(np.float64) * codec.pos_scale(32) + 0.5)
          .astype(np.int64)) % codec.pos_scale(32)
    order = np.argsort(codec.cell_keys(u1 >> 8, 32, 1), kind="stable")
    assert np.array_equal(perms[0].cpu().numpy(), order)
    assert int(c.to_host(out[0])["count"].astype(np.int64).sum()) == 50021
    c.close()
