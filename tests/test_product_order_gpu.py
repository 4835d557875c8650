"""Binary32 products with K below 2048: their sums are formed in a fixed order,
so every call gives the same bits, and C's old value is added once.  Shapes of few
tiles take the kernel whose waves share K (16- and 32-row tiles; by DMA and
through registers), at the edges of its tiles, stages and waves."""
import numpy as np
import pytest
import torch

from paper_1908_06649_amd import tcu

import gpu_util as gu
from test_rect_gpu import run_and_check

pytestmark = pytest.mark.gpu

FLOATS = [("f16", torch.float16), ("bf16", torch.bfloat16)]


@pytest.mark.parametrize("height", [16, 32])
@pytest.mark.parametrize("pitch", ["contiguous", "padded"])
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("din", ["f16", "bf16"])
@pytest.mark.parametrize("M,K,N", [(1, 1, 1), (3, 5, 7), (17, 63, 33), (31, 64, 64), (16, 512, 32),
                                   (33, 513, 31), (64, 575, 96), (65, 577, 40), (200, 1100, 72),
                                   (190, 2047, 301), (100, 1984, 136)])
def test_shared_k_edges(M, K, N, din, accumulate, pitch, height, knobs):
    """As many compute units assumed as there are tiles of that height, so that
    they are one round."""
    knobs(tcu.TCU_KNOB_PP_GRID, -(-M // height) * -(-N // 32))
    run_and_check(M, K, N, din, "f32", 16, pitch, accumulate, seed=M + 3 * K + N)


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("name,dt", FLOATS)
@pytest.mark.parametrize("M,K,N", [(320, 1024, 320), (300, 2000, 300), (16, 2047, 16), (64, 1536, 512),
                                   (192, 2047, 320), (640, 1900, 640), (256, 2016, 256)])
def test_same_bits_every_call(M, K, N, name, dt, pad, accumulate):
    g = torch.Generator(device=gu.DEV).manual_seed(M + K + N)
    A = torch.randn(M, K + pad, generator=g, device=gu.DEV).to(dt)[:, :K]
    B = torch.randn(K, N + pad, generator=g, device=gu.DEV).to(dt)[:, :N]
    C0 = torch.randn(M, N + pad, generator=g, device=gu.DEV)[:, :N]
    first = None
    for _ in range(24):
        C = C0.clone(memory_format=torch.preserve_format)
        tcu.tcu_gemm_rect_ex(A, K + pad, B, N + pad, C, C.stride(0), M, K, N,
                             tcu.TCU_ACCUMULATE if accumulate else 0, 16)
        bits = C.contiguous().view(torch.int32)
        if first is None:
            first = bits
        assert torch.equal(bits, first)


@pytest.mark.parametrize("M,K,N,pad", [(192, 2000, 320, 0), (300, 2000, 300, 3), (64, 1024, 64, 0)])
def test_old_value_added_once(M, K, N, pad):
    """|C| of 2^20 and sums below 2^9: one rounding of the result, half a unit of
    2^-3 there, and the sums' own error (below 2^-8)."""
    g = torch.Generator(device=gu.DEV).manual_seed(K)
    A = torch.rand(M, K + pad, generator=g, device=gu.DEV).sub_(0.5).half()[:, :K]
    B = torch.rand(K, N + pad, generator=g, device=gu.DEV).sub_(0.5).half()[:, :N]
    C = torch.randn(M, N, generator=g, device=gu.DEV).add_(float(1 << 20))
    want = A.double() @ B.double() + C.double()
    tcu.tcu_gemm_rect_ex(A, K + pad, B, N + pad, C, N, M, K, N, tcu.TCU_ACCUMULATE, 16)
    assert (C.double() - want).abs().max().item() <= 2.0 ** -4 + 2.0 ** -8
