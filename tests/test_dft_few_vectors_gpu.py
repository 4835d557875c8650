"""Few and many long vectors.  With s = 16 on both sides of the batch from which they are
transformed whole (a quarter of 256 compute units): one launch per level gives the
same bits, and the result is within the oracle's bar; with a last level of radix below s
and more columns than its workgroups take at once, a vector's bits do not depend on
its place among the others, nor on an infinity in one of them."""
import numpy as np
import pytest

from oracle import compare
from paper_1908_06649_amd import inputs, tcu

from test_dft_gpu import run_dft

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lg", [12, 13])
@pytest.mark.parametrize("batch", [1, 63, 64, 65])
def test_dft_few_vectors(knobs, lg, batch):
    x = inputs.complex_signal(batch, 1 << lg, seed=lg + batch)
    got = run_dft(x, 16)
    knobs(tcu.TCU_KNOB_DFT_PAIRS, 1)
    assert np.array_equal(got.view(np.uint64), run_dft(x, 16).view(np.uint64))
    rep = compare.check_dft(x.numpy(), got)
    assert rep["max_rel_frob"] <= 1e-4, rep


@pytest.mark.parametrize("s", [16, 32])
@pytest.mark.parametrize("batch", [130, 517])
def test_dft_many_vectors(s, batch):
    n = 1 << 14
    x = inputs.complex_signal(batch, n, seed=s + batch)
    x[batch - 2, 77] = complex(float("inf"), 1.0)
    got = run_dft(x, s).view(np.uint64)
    for i in (0, batch // 2, batch - 3, batch - 1):
        assert np.array_equal(got[i], run_dft(x[i:i + 1], s).view(np.uint64)[0]), i
    assert np.isnan(got[batch - 2].view(np.complex64)).all()
