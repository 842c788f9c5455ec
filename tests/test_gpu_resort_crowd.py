"""The re-sort at the edges of its forms for crowded states: arrival lists of a brick around
the lengths that are ranked in LDS (256 a wave), sorted in registers (1024) and sorted by a
whole workgroup; bricks of many times the mean of old particles; escapes in many tiles of
bricks. With a zero force the new
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
    arrivals = []
    for s, o, p in zip(st, out, perms):
        old, new = c.to_host(s), c.to_host(o)
        u, _ = codec.decode_codes(old)
        u1 = (u + np.floor(codec.decode(old)[1].astype(np.float64) * S + 0.5)
              .astype(np.int64)) % S
        was, keys = (codec.cell_keys(q >> 8, n_cell, brick) for q in (u, u1))
        order = np.argsort(keys, kind="stable")
        assert np.array_equal(p.cpu().numpy(), order)
        un, _ = codec.decode_codes(new)
        assert np.array_equal(un, u1[order])
        cnt, esc = codec.build_counts(keys[order], n_cell)
        assert np.array_equal(new["count"], cnt)
        assert np.array_equal(new["esc"], np.asarray(esc, dtype=np.uint64).reshape(-1, 2))
        assert new["j_min"] == new["vel"].min() and new["j_max"] == new["vel"].max()
        b, b0 = keys // brick ** 3, was // brick ** 3
        arrivals.append(np.bincount(b[b != b0], minlength=(n_cell // brick) ** 3))
    c.close()
    return arrivals


def _box(rng, n, lo, side):
    return lo + side * (0.02 + 0.96 * rng.random((n, 3)))


@pytest.mark.parametrize("n_mesh,n_cell,brick", [(64, 16, 4), (64, 32, 8), (32, 16, 2)])
@pytest.mark.parametrize("m", [255, 256, 257, 511, 1023, 1024, 1025, 5000])
def test_lists_of_many_lengths(n_mesh, n_cell, brick, m):
    rng = np.random.default_rng(m)
    side = brick / n_cell
    loads = []
    for k in (m, m // 3):  # k particles from all over the box into one brick, among others
        x = rng.random((k + 3000, 3))
        to = x.copy()
        x[:k] = 0.5 * x[:k] + np.array([0.0, 0.0, 0.5]) * rng.integers(0, 2, (k, 1))
        to[:k] = _box(rng, k, 2 * side if brick < n_cell // 2 else side, side)
        keep = rng.permutation(k + 3000)
        loads.append((x[keep], to[keep]))
    got = _check(n_mesh, n_cell, brick, loads)
    assert got[0].max() >= m - m // 8  # (a few were there before)


@pytest.mark.parametrize("n_mesh,n_cell,brick,n", [(64, 16, 4, 2600), (64, 16, 4, 30011),
                                                   (64, 32, 8, 40003), (128, 64, 2, 9001)])
@pytest.mark.parametrize("hop", [0.02, 0.4, 3.0])  # drift in bricks: stay, cross, scatter
def test_bricks_of_many_times_the_mean(n_mesh, n_cell, brick, n, hop):
    rng = np.random.default_rng(n)
    side = brick / n_cell
    loads = []
    for k, lo in ((n, side), (n // 2, 0.0), (100, 0.0)):
        x = np.concatenate([_box(rng, k, lo, side), rng.random((500, 3))])
        to = x + rng.normal(0.0, hop * side, x.shape)
        keep = rng.permutation(len(x))
        loads.append((x[keep], to[keep]))
    _check(n_mesh, n_cell, brick, loads)


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
