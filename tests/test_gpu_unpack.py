"""pm_unpack takes records apart on the GPU from places that the host finds along the counts:
every byte of the species and its header come back, for odd sizes, escapes, all code widths
and bodies on either side of the upload buffer's 256 MB; a damaged stream is refused with the
destination untouched."""

import ctypes

import numpy as np
import pytest
import torch

from gpu_util import ctx
from paper_1611_01545_amd.pm import widths_word

pytestmark = pytest.mark.gpu

FIELDS = ("count", "pos", "vel", "hdr")


def _state(c, n, kind, widths, seed=3):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    x = torch.rand((n, 3), generator=gen, device="cuda")
    if kind == "clumps" and n:
        x[: n // 2] = x[:1] * 0.999  # one cell of n / 2: an escape beyond 255 particles
        x[n // 2: n // 2 + n // 4] *= 0.3
    v = torch.randn((n, 3), generator=gen, device="cuda")
    return c.encode(c.float_species(x, v, 0.25), cap_esc=4096, widths=widths)


@pytest.mark.parametrize("n_mesh,n_cell", [(16, 4), (16, 16), (64, 32)])
@pytest.mark.parametrize("pos,vel", [(1, 2), (2, 2), (1, 1), (2, 1)])
@pytest.mark.parametrize("kind,n", [("uniform", 1), ("uniform", 63), ("clumps", 1021),
                                    ("uniform", 20000), ("clumps", 200003)])
def test_round_trip(n_mesh, n_cell, pos, vel, kind, n):
    c = ctx(n_mesh, n_cell)
    s = _state(c, n, kind, widths_word(pos, vel))
    data = c.pack(s, 5)
    for blob in (data, bytearray(data), memoryview(data)):
        back, sid = c.unpack(blob, n, cap_esc=4096)
        assert sid == 5 and back.mass == 0.25
        for f in FIELDS:
            assert torch.equal(getattr(back, f), getattr(s, f)), f
        ne = s.header()["n_esc"]
        assert torch.equal(back.esc[:ne], s.esc[:ne])
    c.close()


@pytest.mark.parametrize("n_cell", [8, 4])
def test_bodies_beyond_the_upload_buffer(n_cell):
    """270 MB of records: in several uploads (8 runs of 64 cells), and in one run that is
    itself longer than the buffer (4^3 cells)."""
    c = ctx(16, n_cell)
    n = 30_000_001
    s = _state(c, n, "uniform", 0)
    data = c.pack(s, 0)
    back, _ = c.unpack(data, n, cap_esc=4096)
    for f in FIELDS:
        assert torch.equal(getattr(back, f), getattr(s, f)), f
    c.close()


@pytest.mark.parametrize("n", [600, 300000])  # walked before and beside the upload
def test_damaged_streams_are_refused(n):
    c = ctx(64, 32)
    s = _state(c, n, "clumps", 0)
    data = bytearray(c.pack(s, 0))

    def refused(blob, cap=4096, n_out=n):
        out = c.empty_compressed(n_out, 0.0, cap)
        for t in (out.count, out.pos, out.vel, out.esc, out.hdr):
            t.fill_(7)
        a = out.c()
        raw = np.frombuffer(bytes(blob), dtype=np.uint8)
        code = c.lib.pm_unpack(c.h, ctypes.c_void_p(raw.ctypes.data), len(raw), ctypes.byref(a),
                               None, None)
        c.sync()
        for t in (out.count, out.pos, out.vel, out.esc, out.hdr):
            assert bool((t == 7).all())
        return code

    def with_checksum(body):
        b = np.frombuffer(bytes(body), dtype=np.uint8).astype(np.uint64)
        cs = int(((2 * np.arange(len(b), dtype=np.uint64) + 1) * b).sum(dtype=np.uint64))
        head = bytearray(data[:64])
        head[48:56] = cs.to_bytes(8, "little")
        head[56:64] = len(b).to_bytes(8, "little")
        return bytes(head) + bytes(body)

    corrupt = 6
    body = data[64:]
    flip = bytearray(data)
    flip[-1] ^= 1
    assert refused(flip) == corrupt                       # the checksum
    assert refused(data[:-1]) == corrupt                  # the length
    assert refused(data, n_out=n + 1) == corrupt          # the particle number
    assert refused(with_checksum(body[:-9])) == corrupt   # records missing
    assert refused(with_checksum(body + b"\0")) == corrupt
    more = bytearray(body)
    more[0] = 254                                         # a count too large
    assert refused(with_checksum(more)) == corrupt
    short = bytearray(body)
    k = short.index(255)
    while int.from_bytes(short[k + 1:k + 5], "little") != int(s.esc[0, 1]):
        k = short.index(255, k + 1)
    short[k + 1:k + 5] = (254).to_bytes(4, "little")      # an escape that needs none
    assert refused(with_checksum(short)) == corrupt
    assert refused(data, cap=0) == 5                      # PM_ERR_CAPACITY
    assert c.last_error_detail() == s.header()["n_esc"]
    assert refused(with_checksum(body)[:40]) == corrupt
    c.close()


@pytest.mark.parametrize("n", [0, 1, (2 << 20) - 1, 2 << 20, (16 << 20) - 1, 16 << 20,
                               (32 << 20) + 5, 50_000_003])
def test_device_bytes(n):
    """Around the pieces and the threads' cuts of the copy into a bytes object."""
    from paper_1611_01545_amd.pm import _device_bytes
    t = torch.randint(0, 256, (n + 3,), dtype=torch.uint8, device="cuda")[1: n + 1]
    assert _device_bytes(t) == t.cpu().numpy().tobytes()
