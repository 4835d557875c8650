"""The library's choice of kernels, read off the launches it would make
(tests/recording.py), on a device of 256 compute units."""
import random
import shutil

import pytest

from paper_1908_06649_amd import tcu

import recording as rec

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")

F16, BF16, BF16OUT, I8 = (tcu.TCU_F16_F32, tcu.TCU_BF16_F32, tcu.TCU_BF16_BF16, tcu.TCU_I8_I32)


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return rec.build(tmp_path_factory.mktemp("recording"))


def kernels(answer):
    """Names without the namespace and the argument types."""
    assert answer["rc"] == tcu.TCU_OK
    out = []
    for la in answer["launches"]:
        name = la["name"].split("_GLOBAL__N_1")[1].lstrip("0123456789")
        out.append(name.split("EEv")[0])
    return out


# Sizes on both sides of the lines where the full-tile kernel and the 128 x 128
# ring tiles take turns, the faster one on the card: a ragged last round that
# is split, rows that start inside a line, many rounds, large outputs.
@pytest.mark.parametrize("M,K,N,dtype,want", [
    (4350, 4096, 4352, F16, "gemm_pp"), (4350, 8192, 4352, BF16, "gemm_pp"),
    (4350, 4096, 4352, BF16OUT, "ring128"), (4350, 1024, 4352, F16, "ring128"),
    (6000, 6000, 6000, F16, "gemm_pp"), (6000, 6000, 6000, I8, "gemm_pp"),
    (6000, 1000, 6000, BF16OUT, "gemm_pp"),
    (7000, 4096, 7008, F16, "gemm_pp"), (8192, 8192, 8192, BF16, "gemm_pp"),
    (3072, 1024, 3072, BF16OUT, "ring128"), (3072, 3072, 3072, I8, "ring128"),
    (2560, 2560, 2560, BF16, "ring128"), (4096, 4096, 4096, BF16, "gemm_pp"),
    (4101, 1000, 4173, BF16OUT, "ring128"), (1024, 1024, 1024, F16, "ring64"),
    (192, 8192, 320, F16, "ring64"), (192, 1024, 320, F16, "gemm_wave")])
def test_tile_choice(so, M, K, N, dtype, want):
    names = kernels(rec.run(so, [rec.product(M, K, N, dtype)])[0])
    part = {"ring128": f"gemm_ring_kernelILi{dtype}ELi128", "ring64": f"gemm_ring_kernelILi{dtype}ELi64"}
    assert any(part.get(want, want) in n for n in names), names


# Few long vectors with s = 16 are faster divided among launches (2^12: a pair
# and a level; 2^13: a pair and two levels), more of them, shorter ones and s = 32
# whole in one.
@pytest.mark.parametrize("n,batch,s,launches", [
    (1 << 13, 1, 16, 3), (1 << 13, 63, 16, 3), (1 << 13, 64, 16, 1), (1 << 12, 4, 16, 2),
    (1 << 12, 64, 16, 1), (1 << 11, 1, 16, 1), (1 << 13, 1, 32, 1), (1, 7, 32, 1)])
def test_dft_division(so, n, batch, s, launches):
    job = dict(fn="tcu_dft_ex", args=[rec.ptr(0), rec.ptr(1), rec.ptr(2), n, batch, s, None])
    names = kernels(rec.run(so, [job])[0])
    assert len(names) == launches, names
    assert (launches == 1) == names[0].startswith("dft_local")
