"""The binding's flat operand checks against its general ones, on stand-in
tensors (no device): both accept the same operands and return the same
pointers, and refuse the same ones with the same error."""
import itertools

import pytest
import torch

from paper_1908_06649_amd import tcu


class Fake:
    """What the binding asks of a tensor, with a device index of its own."""

    def __init__(self, t, dev=0, ptr=64):
        self.t, self.dev, self.ptr = t, dev, ptr

    is_cuda = property(lambda self: self.dev >= 0)
    shape = property(lambda self: self.t.shape)

    def get_device(self):
        return self.dev

    def data_ptr(self):
        return self.ptr

    def __getattr__(self, name):
        return getattr(self.t, name)


@pytest.fixture
def device0(monkeypatch):
    monkeypatch.setattr(tcu, "_GET_DEVICE", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)


def outcome(f):
    try:
        return f()
    except ValueError as e:
        return str(e)


ARRAYS = [torch.zeros(4, 6), torch.zeros(24), torch.zeros(6, 4).t(), torch.zeros(4, 8)[:, :6],
          torch.zeros(4, 7), torch.zeros(0), torch.zeros(1, 24)[:, ::2], torch.zeros(1, 6)]


@pytest.mark.parametrize("want", [24, 0, 6])
def test_contiguous_operands(device0, want):
    for a, b in itertools.product(ARRAYS, ARRAYS):
        for devs in ((0, 0, 0), (1, 1, 1), (0, 1, 0), (-1, -1, -1), (0, 0, -1)):
            ts = [Fake(x, d, 64 + i) for i, (x, d) in enumerate(zip((a, b, ARRAYS[0]), devs))]

            def general():
                dev, (x, y, z) = tcu._marshal("call", ts, (24, want, 24))
                return dev, x, y, z
            assert outcome(lambda: tcu._marshal3("call", *ts, 24, want, 24)) == outcome(general)


VIEWS = [torch.zeros(4, 6), torch.zeros(4, 9)[:, :6], torch.zeros(6, 4).t(), torch.zeros(4, 12)[:, ::2],
         torch.zeros(1, 6), torch.zeros(4, 1), torch.zeros(8, 1)[::2], torch.zeros(24), torch.zeros(0, 6)]


@pytest.mark.parametrize("ld", [6, 9, 1, 4])
def test_view_operands(device0, ld):
    B, C = torch.zeros(6, 5), torch.zeros(4, 5)
    for a, M, K, dev in itertools.product(VIEWS, (4, 1, 0), (6, 1), (0, 1, -1)):
        ts = Fake(a, dev), Fake(B[:K]), Fake(C[:M])

        def general():
            d, (x, y, z) = tcu._marshal_views(
                "call", ((ts[0], M, K, ld), (ts[1], K, 5, 5), (ts[2], M, 5, 5)))
            return d, x, y, z
        assert outcome(lambda: tcu._marshal_views3("call", ts[0], ld, ts[1], 5, ts[2], 5, M, K,
                                                   5)) == outcome(general)
