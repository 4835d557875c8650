"""The ring kernel of the product on every tile size, fill and edge: DMA and
register-staged (any row pitch), chunks that cross the ends of rows, rows
shorter than a chunk, partial last stages and K ranges added atomically.

TCU_KNOB_PP_GRID sets the number of compute units the tile choice assumes, so
that a few workgroups make it take 128 x 128 tiles on small shapes."""
import pytest

from paper_1908_06649_amd import tcu

import gpu_util as gu
from test_rect_gpu import PAIRS, run_and_check

pytestmark = pytest.mark.gpu

# (M, K, N): below a chunk in every dimension, one chunk and one more element,
# one tile and its neighbours, a stage and its neighbours (64 and 128
# elements), several tiles with every remainder, and a long K.
SHAPES = [(1, 1, 1), (3, 5, 7), (5, 9, 17), (17, 7, 129), (130, 65, 6), (64, 64, 64), (65, 63, 65),
          (127, 129, 136), (129, 128, 257), (200, 333, 190), (256, 191, 384), (70, 2055, 75)]


@pytest.mark.parametrize("cus", [1, 256])
@pytest.mark.parametrize("kernel", ["general", "auto"])
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("din,out", PAIRS)
@pytest.mark.parametrize("M,K,N", SHAPES)
def test_ring_edges(M, K, N, din, out, accumulate, kernel, cus, knobs):
    knobs(tcu.TCU_KNOB_GEMM_KERNEL, gu.PATHS[kernel])
    knobs(tcu.TCU_KNOB_PP_GRID, cus)
    pitch = "padded" if (M + N) % 2 else "contiguous"
    run_and_check(M, K, N, din, out, 16, pitch, accumulate, seed=M * 7 + K * 3 + N)


@pytest.mark.parametrize("nsplit", [2, 5, 16])
@pytest.mark.parametrize("kernel", ["general", "ring"])
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("din,out", PAIRS)
@pytest.mark.parametrize("M,K,N", [(64, 1024, 64), (150, 1111, 203), (65, 640, 200)])
def test_ring_split_k(M, K, N, din, out, accumulate, kernel, nsplit, knobs):
    """Forced K ranges (bfloat16 outputs stay whole); 16 ranges leave one
    stage or less apiece."""
    knobs(tcu.TCU_KNOB_GEMM_KERNEL, gu.PATHS[kernel])
    knobs(tcu.TCU_KNOB_SPLIT_K, nsplit)
    run_and_check(M, K, N, din, out, 32, "padded", accumulate, seed=M + K + N + nsplit)


@pytest.mark.parametrize("cus", [1, 256])
@pytest.mark.parametrize("din,out", [p for p in PAIRS if p[1] != "bf16"])
def test_ring_split_k_chosen_by_size(din, out, cus, knobs):
    """A few tiles with a long K are split without forcing."""
    knobs(tcu.TCU_KNOB_PP_GRID, cus)
    run_and_check(131, 8200, 140, din, out, 16, "contiguous", True, seed=9)


# On 2 compute units a round is 4 tiles of 128 x 128 and a last round of one is cut
# into quarters of 64 x 64: 5 and 9 tiles whose last has four, two or one quarter
# inside C, one of them a row or a column wide; DMA and register-staged.
@pytest.mark.parametrize("pitch", ["contiguous", "padded"])
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("din,out", PAIRS)
@pytest.mark.parametrize("M,K,N", [(640, 128, 128), (600, 130, 101), (577, 2055, 112),
                                   (321, 333, 384), (384, 64, 321), (300, 70, 304), (1030, 99, 90)])
def test_ring_quarters(M, K, N, din, out, accumulate, pitch, knobs):
    knobs(tcu.TCU_KNOB_GEMM_KERNEL, gu.PATHS["auto"])
    knobs(tcu.TCU_KNOB_PP_GRID, 2)
    run_and_check(M, K, N, din, out, 16, pitch, accumulate, seed=M + K * 3 + N)
