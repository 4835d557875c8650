"""The full-tile kernel on ragged shapes, forced, on a few workgroups: rows,
columns and stages cut by the edge in the kernel (N a whole number of 16-byte
chunks), or its 256-aligned interior with the ring kernel on the strips; the
last round's tiles whole or split, with C's edge through them.  Pitches are
multiples of 16 bytes, the unused columns poisoned (tests/test_dispatch.py checks
that these calls take the kernel)."""
import pytest

from paper_1908_06649_amd import tcu

from test_rect_gpu import PAIRS, run_and_check

pytestmark = pytest.mark.gpu

# (M, K, N): K tail alone, M, N, all; one tile smaller than C's edge; several
# tiles and a long K; then N that is no whole number of chunks (strips right and
# below, one of them alone).
EDGES = [(256, 70, 256), (300, 128, 256), (256, 64, 272), (515, 200, 528), (100, 97, 48),
         (700, 1030, 784)]
STRIPS = [(515, 200, 521), (512, 96, 259), (300, 65, 777)]


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("din,out", PAIRS)
@pytest.mark.parametrize("M,K,N", EDGES + STRIPS)
def test_full_ragged(M, K, N, din, out, accumulate, knobs):
    knobs(tcu.TCU_KNOB_GEMM_KERNEL, tcu.TCU_PATH_FULL_TILE)
    knobs(tcu.TCU_KNOB_PP_GRID, 2)
    knobs(tcu.TCU_KNOB_TAIL_SPLIT, 1)
    run_and_check(M, K, N, din, out, 32, "padded", accumulate, seed=M + K + N)


# 9 and 12 tiles on 8 and 5 workgroups: one tail tile (the corner) and two.
@pytest.mark.parametrize("M,K,N,grid", [(700, 1030, 656, 8), (700, 1030, 784, 5),
                                        (800, 1001, 777, 4)])
@pytest.mark.parametrize("din,out", PAIRS)
@pytest.mark.parametrize("accumulate", [False, True])
def test_full_ragged_tail_split(M, K, N, grid, din, out, accumulate, knobs):
    knobs(tcu.TCU_KNOB_GEMM_KERNEL, tcu.TCU_PATH_FULL_TILE)
    knobs(tcu.TCU_KNOB_PP_GRID, grid)
    knobs(tcu.TCU_KNOB_TAIL_SPLIT, 3)
    run_and_check(M, K, N, din, out, 32, "padded", accumulate, seed=M + K + N + 1)
