"""Long vectors with s = 16 on both sides of the batch from which they are
transformed whole (a quarter of 256 compute units): one launch per level gives the
same bits, and the result is within the oracle's bar."""
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
