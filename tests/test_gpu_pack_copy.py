"""The copy of a packed stream into a bytes object around the size from which it goes in pieces,
and where no page-locked memory is to be had."""

import pytest
import torch

from paper_1611_01545_amd import pm

pytestmark = pytest.mark.gpu


def _bytes(n):
    return torch.randint(0, 256, (n + 3,), dtype=torch.uint8, device="cuda")[1: n + 1]


@pytest.mark.parametrize("n", [(6 << 20) - 1, 6 << 20, (6 << 20) + 7])
def test_where_pieces_start(n):
    t = _bytes(n)
    assert pm._device_bytes(t) == t.cpu().numpy().tobytes()


def test_without_page_locked_memory(monkeypatch):
    t = _bytes(9_000_001)
    want = t.cpu().numpy().tobytes()
    empty = torch.empty

    def refuse(*a, **k):
        if k.get("pin_memory"):
            raise RuntimeError("out of page-locked memory")
        return empty(*a, **k)

    monkeypatch.setattr(torch, "empty", refuse)
    assert pm._device_bytes(t) == want
