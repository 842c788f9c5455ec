"""The encode's sort of whole records: one to four digit passes (one cell to 2^24 cells and
more), tiles full, short and of one particle, all code widths, with and without the
permutation, all particles in one cell or in a few, against a stable sort of the codes."""

import numpy as np
import pytest
import torch

from gpu_util import ctx
from oracle import codec
from paper_1611_01545_amd.pm import widths_word

pytestmark = pytest.mark.gpu


def _load(kind, n, rng):
    if kind == "uniform":
        x = rng.random((n, 3), dtype=np.float32)
    elif kind == "one":
        x = np.full((n, 3), 0.7, dtype=np.float32)
    else:  # descending cells, with ties
        x = np.repeat(np.linspace(0.999, 0.0, n // 3 + 1, dtype=np.float32), 3)[:n, None]
        x = np.ascontiguousarray(np.broadcast_to(x, (n, 3)))
    v = rng.standard_normal((n, 3)).astype(np.float32)
    v[0] = (-7.0, 0.0, 7.0)
    return x, v


@pytest.mark.parametrize("n_mesh,n_cell,brick", [(8, 1, 1), (8, 4, 2), (64, 32, 8),
                                                 (128, 128, 8), (256, 256, 4)])
@pytest.mark.parametrize("pos,vel", [(1, 2), (2, 2), (1, 1), (2, 1)])
@pytest.mark.parametrize("kind,n", [("uniform", 1), ("uniform", 4095), ("uniform", 4096),
                                    ("descending", 4097), ("one", 9001), ("uniform", 100003)])
def test_encode_is_the_stable_sort_by_cell(n_mesh, n_cell, brick, pos, vel, kind, n):
    rng = np.random.default_rng(17)
    c = ctx(n_mesh, n_cell, brick=brick)
    x, v = _load(kind, n, rng)
    w = widths_word(pos, vel)
    fs = c.float_species(x, v, 1.0)
    got, perm = c.encode(fs, want_perm=True, cap_esc=4096, widths=w)
    plain = c.encode(fs, cap_esc=4096, widths=w)
    h = c.to_host(got)
    S = codec.pos_scale(n_cell, pos)
    u = np.floor(x.astype(np.float64) * S).astype(np.int64) % S
    keys = codec.cell_keys(u >> (8 * pos), n_cell, brick)
    order = np.argsort(keys, kind="stable")
    assert np.array_equal(perm.cpu().numpy(), order)
    un, j = codec.decode_codes(h)
    assert np.array_equal(un, u[order])
    half = 2.0 ** (8 * vel - 1)
    vm = np.abs(v).max()
    assert h["v_max"] == vm
    jj = np.clip(np.floor(v.astype(np.float64) * (half / float(vm)) + half), 0, 2 * half - 1)
    assert np.array_equal(j, jj[order].astype(np.int64))
    assert h["j_min"] == jj.min() and h["j_max"] == jj.max()
    for f in ("count", "pos", "vel", "hdr"):
        assert torch.equal(getattr(got, f), getattr(plain, f)), f
    c.close()
