"""A value that is infinite, NaN or past bfloat16's range in one vector of a
batch leaves every other vector's bits as they are without it, on every path
whose last level shares matrix-core columns between transforms, and makes its
own vector NaN (its lo word, v - hi, is NaN or Inf in every product)."""
import numpy as np
import pytest
import torch

from paper_1908_06649_amd import inputs, tcu

import gpu_util as gu

pytestmark = pytest.mark.gpu


def run_dft(x, s):
    dx = x.to(gu.DEV)
    y, work = torch.zeros_like(dx), torch.empty_like(dx)
    tcu.tcu_dft_ex(dx, y, work, x.shape[1], x.shape[0], s)
    torch.cuda.synchronize()
    return y.cpu().numpy()


@pytest.mark.parametrize("single", [0, 1])
@pytest.mark.parametrize("s", [16, 32])
@pytest.mark.parametrize("lg,batch", [(0, 70), (1, 70), (2, 70), (3, 70), (4, 70), (5, 70), (6, 70),
                                      (7, 35), (8, 35), (9, 19), (11, 5), (13, 3), (14, 3)])
def test_dft_vectors_apart(knobs, lg, batch, s, single):
    knobs(tcu.TCU_KNOB_DFT_PAIRS, single)
    n = 1 << lg
    x = inputs.complex_signal(batch, n, seed=lg + s)
    clean = run_dft(x, s)
    bad = {0: complex(0.0, float("nan")), batch // 2: complex(float("-inf"), 1.0),
           batch - 1: complex(1.0, 3.4e38)}
    for b, v in bad.items():
        x[b, (b * 7 + 1) % n] = v
    got = run_dft(x, s)
    rest = [b for b in range(batch) if b not in bad]
    assert np.array_equal(got[rest].view(np.uint64), clean[rest].view(np.uint64))
    assert np.isnan(got[list(bad)].view(np.float32)).all()


def test_dft_largest_finite_words():
    """The largest magnitude that stays finite as a bfloat16 word is not taken
    for one that does not."""
    x = torch.zeros((40, 2), dtype=torch.complex64)
    big = float(np.uint32(0x7F7F7FFF).view(np.float32))
    x[3, 0] = complex(big, -big)
    got = run_dft(x, 32)
    want = np.zeros((40, 2), np.complex64)
    want[3] = complex(big, -big)
    assert np.abs(got / big - want / big).max() <= 2.0 ** -15
