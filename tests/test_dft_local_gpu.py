"""The DFT's division into launches: short vectors whole in LDS (several per
tile, a last tile that is not full), last levels narrower than the unit, and
pairs of levels apart, bit for bit against one launch per level
(TCU_KNOB_DFT_PAIRS = 1) and within the oracle's bar."""
import numpy as np
import pytest

from oracle import compare
from paper_1908_06649_amd import inputs, tcu

from test_dft_gpu import run_dft

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [16, 32])
@pytest.mark.parametrize("lg,batch", [(0, 5), (1, 4099), (2, 3), (3, 517), (4, 257), (5, 129),
                                      (6, 65), (7, 33), (8, 17), (9, 9), (10, 5), (11, 3),
                                      (12, 2), (13, 3), (14, 1), (17, 1)])
def test_dft_divisions_bit_identical(knobs, lg, batch, s):
    n = 1 << lg
    x = inputs.complex_signal(batch, n, seed=lg + 31 * batch + s)
    whole = run_dft(x, s)
    knobs(tcu.TCU_KNOB_DFT_PAIRS, 1)
    single = run_dft(x, s)
    assert np.array_equal(whole.view(np.uint64), single.view(np.uint64))
    rep = compare.check_dft(x.numpy(), whole)
    assert rep["max_rel_frob"] <= 1e-4, rep


def test_dft_more_tiles_than_workgroups():
    """1100 tiles of two vectors: workgroups walk several."""
    x = inputs.complex_signal(2200, 2048, seed=8)
    got = run_dft(x, 32)
    want = np.fft.fft(x.numpy().astype(np.complex128), axis=1)
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    assert err <= 1e-4, err       # the hi/lo products keep ~2^-16 per level
