"""Polynomial evaluation on both sides of every choice of its kernel: 16 and
32 powers per column (n = 1024), block edges, the small and the large stage of
coefficients (and more than one stage of each), and few and many points."""
import pytest

from oracle import compare
from paper_1908_06649_amd import inputs

from test_poly_gpu import PAIRS, draw, run_poly

pytestmark = pytest.mark.gpu

# n around the blocks (512, 1024), the choice of powers (1024), the stages of
# 32 KiB (8192 binary16, 16384 bfloat16 coefficients) and 128 KiB (four times
# that); p below one chunk and a chunk's neighbours, few points, and enough
# of them (16 waves per CU, two chunks each) for the large stage.
SMALL = [(15, 31), (17, 33), (511, 65), (513, 1), (1023, 100), (1025, 70000), (2047, 63),
         (8193, 129), (16385, 95), (70000, 33)]
LARGE = [(8200, 300000), (16400, 270001), (40000, 263000)]


@pytest.mark.parametrize("din,out", PAIRS)
@pytest.mark.parametrize("n,p", SMALL)
def test_poly_edges(n, p, din, out):
    coef, pts = draw(n, p, din, seed=n + p)
    got = run_poly(coef, pts, 32, out)
    compare.check_poly(din, out, inputs.bits(coef), inputs.bits(pts), got, 32)


@pytest.mark.parametrize("din,out", PAIRS)
@pytest.mark.parametrize("n,p", LARGE)
def test_poly_large_stage(n, p, din, out):
    """The first 700, middle and last points against the oracle."""
    coef, pts = draw(n, p, din, seed=n + 3 * p)
    got = run_poly(coef, pts, 16, out)
    for a in (0, p // 2, p - 700):
        compare.check_poly(din, out, inputs.bits(coef), inputs.bits(pts[a:a + 700]),
                           got[a:a + 700], 16)
