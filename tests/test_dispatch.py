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


# The first pair reads its input past the caches from 32 MiB on with s = 32, past 64
# MiB with s = 16.
@pytest.mark.parametrize("n,batch,s,past", [
    (1 << 20, 3, 32, 0), (1 << 20, 4, 32, 1), (1 << 20, 8, 16, 0), (1 << 20, 9, 16, 1),
    (1 << 14, 512, 16, 0), (1 << 14, 513, 16, 1)])
def test_dft_input_past_caches(so, n, batch, s, past):
    job = dict(fn="tcu_dft_ex", args=[rec.ptr(0), rec.ptr(1), rec.ptr(2), n, batch, s, None])
    assert kernels(rec.run(so, [job])[0])[0] == f"dft_pair_kernelILi{s}ELb0ELb{past}E"


# The last level of radix below s: three workgroups per compute unit, 12 for arrays
# of more than 64 MiB; a workgroup of four waves takes 64 s elements.
@pytest.mark.parametrize("n,batch,s,blocks", [
    (1 << 14, 4, 32, 32), (1 << 14, 97, 32, 768), (1 << 14, 512, 32, 768),
    (1 << 14, 513, 32, 3072), (1 << 14, 200, 16, 768), (1 << 14, 1024, 16, 3072)])
def test_dft_narrow_grid(so, n, batch, s, blocks):
    job = dict(fn="tcu_dft_ex", args=[rec.ptr(0), rec.ptr(1), rec.ptr(2), n, batch, s, None])
    answer = rec.run(so, [job])[0]
    assert kernels(answer)[-1] == f"dft_level_kernelILi{s}ELb1E"
    assert answer["launches"][-1]["blocks"] == blocks


def aligned(cols, dtype_bytes, extra):
    """The padded pitches of the GPU tests."""
    step = 16 // dtype_bytes
    return (cols + step - 1) // step * step + extra * step


def padded(M, K, N, dtype, knobs, acc=False):
    es, ob = (1 if dtype == I8 else 2), (2 if dtype == BF16OUT else 4)
    return rec.product(M, K, N, dtype, lda=aligned(K, es, 1), ldb=aligned(N, es, 2),
                       ldc=aligned(N, ob, 1), acc=acc, knobs=knobs)


def test_forced_full_tiles_on_ragged_shapes(so):
    """What tests/test_full_ragged_gpu.py names is what it runs."""
    import test_full_ragged_gpu as t
    for dtype in (F16, BF16, BF16OUT, I8):
        for shapes, strips in ((t.EDGES, False), (t.STRIPS, True)):
            for M, K, N in shapes:
                if dtype == I8 and (N % 16 != 0) != strips:
                    continue
                knobs = [(tcu.TCU_KNOB_GEMM_KERNEL, tcu.TCU_PATH_FULL_TILE),
                         (tcu.TCU_KNOB_PP_GRID, 2), (tcu.TCU_KNOB_TAIL_SPLIT, 1)]
                names = kernels(rec.run(so, [padded(M, K, N, dtype, knobs)])[0])
                whole = M % 256 == 0 and N % 256 == 0 and K % (64 if dtype == I8 else 32) == 0
                assert names[0] == f"gemm_pp_kernelILi{dtype}ELi5ELb{int(not whole)}E", names
                assert (len(names) > 1) == strips, names
    for M, K, N, grid in ((700, 1030, 656, 8), (700, 1030, 784, 5), (800, 1001, 777, 4)):
        knobs = [(tcu.TCU_KNOB_GEMM_KERNEL, tcu.TCU_PATH_FULL_TILE), (tcu.TCU_KNOB_PP_GRID, grid),
                 (tcu.TCU_KNOB_TAIL_SPLIT, 3)]
        names = kernels(rec.run(so, [padded(M, K, N, F16, knobs)])[0])
        assert names[0].startswith("zero_tiles") and names[1].startswith("gemm_pp"), names


def test_quarters_are_taken(so):
    """The shapes of tests/test_ring_gpu.py's quarters cut a last round."""
    import test_ring_gpu as t
    shapes = [m.args[1] for m in t.test_ring_quarters.pytestmark
              if m.name == "parametrize" and m.args[0] == "M,K,N"][0]
    jobs = [padded(M, K, N, d, [(tcu.TCU_KNOB_PP_GRID, 2)]) for M, K, N in shapes
            for d in (F16, BF16, BF16OUT, I8)]
    for answer in rec.run(so, jobs):
        names = kernels(answer)
        assert "ELi128ELi2ELb" in names[0] and names[0].endswith("ELb1E"), names


def test_shared_k_is_taken(so):
    """The shapes of tests/test_product_order_gpu.py take the tile of the height
    they name, except the ones of at most two stages."""
    import test_product_order_gpu as t
    shapes = [m.args[1] for m in t.test_shared_k_edges.pytestmark
              if m.name == "parametrize" and m.args[0] == "M,K,N"][0]
    for M, K, N in shapes:
        for height in (16, 32):
            tiles = -(-M // height) * -(-N // 32)
            name = kernels(rec.run(so, [padded(M, K, N, BF16, [(tcu.TCU_KNOB_PP_GRID, tiles)])])[0])[0]
            if K > 128 and (height == 16 or M > 16):
                assert name.startswith(f"gemm_wave_kernelILi{BF16}ELi{height}E"), (M, K, N, name)


def test_binary32_repeats_below_2048(so):
    """No binary32 product with K below 2048 is cut into ranges, whatever its
    sizes, pitches and type, and some from 2048 on are."""
    rng = random.Random(5)
    arity = [("gemm_ring", 15), ("gemm_pp", 12)]

    def ranges(K, acc):
        M, N = (max(1, int(2 ** rng.uniform(0, 13.2))) for _ in range(2))
        if rng.random() < 0.5:
            M, N = max(256, M // 256 * 256), max(256, N // 256 * 256)
        pad = rng.choice([0, 0, 8, 1])
        return rec.product(M, K, N, rng.choice([F16, BF16]), lda=K + pad, ldb=N + pad, ldc=N + pad,
                           acc=acc, arity=arity)

    def cut(answer):
        return any(la["name"].find("zero_") >= 0
                   or (la["name"].find("gemm_ring") >= 0 and la["ints"][12] > 1)
                   or (la["name"].find("gemm_pp") >= 0 and la["ints"][11] > 1)
                   for la in answer["launches"])

    below = [ranges(rng.choice([2047, 2016, int(2 ** rng.uniform(0, 11))]), rng.random() < 0.5)
             for _ in range(1500)]
    answers = rec.run(so, below)
    assert not any(cut(a) for a in answers)
    assert any(a["launches"][0]["name"].find("gemm_pp") >= 0 for a in answers)
    assert sum(cut(a) for a in rec.run(so, [ranges(4096, True) for _ in range(200)])) > 20


@pytest.mark.parametrize("M,K,N,dtype", [(1 << 30, 8, 1, BF16), ((1 << 30) - 63, 3, 5, F16),
                                         (1 << 30, 1, 129, BF16OUT), (5, 8, 1 << 30, I8),
                                         (1 << 29, 40, 16, F16)])
def test_largest_dimensions(so, M, K, N, dtype):
    """Products whose tiles exceed a launch's 32-bit count of work items are
    accepted and every tile is taken once."""
    answer = rec.run(so, [rec.product(M, K, N, dtype, arity=[("gemm_ring", 15)])])[0]
    kernels(answer)
    rings = [la for la in answer["launches"] if "gemm_ring" in la["name"]]
    assert all(la["status"] == 0 for la in answer["launches"])
    at = 0
    for la in rings:
        assert la["ints"][14] == at
        at += la["blocks"]
    tiles_m, tiles_n, whole = rings[0]["ints"][10], rings[0]["ints"][11], rings[0]["ints"][13]
    whole = min(whole, tiles_m * tiles_n)
    assert at == whole + 4 * (tiles_m * tiles_n - whole)


@pytest.mark.parametrize("fail", [0, 1, 2, 4])
def test_closure_unpacks_after_a_failed_launch(so, fail):
    """Whichever launch fails, no more bands are walked and X does not stay
    packed: the last launch turns it back into bytes."""
    job = dict(fn="tcu_transitive_closure_ex", args=[rec.ptr(0), 1000, 1000, 16, None])
    ok = rec.run(so, [job])[0]
    names = kernels(ok)
    assert [n.split("_kernel")[0] for n in names] == (
        ["tc_pack", "tc_diag"] + ["tc_band"] * 4 + ["tc_unpack"])
    bad = rec.run(so, [dict(job, fail=fail)])[0]
    assert bad["rc"] == tcu.TCU_ERR_HIP
    tried = [la["name"] for la in bad["launches"]]
    assert [la["status"] != 0 for la in bad["launches"]].count(True) == 1
    assert len(tried) == (1 if fail == 0 else fail + 2)
    assert fail == 0 or "tc_unpack" in tried[-1]


@pytest.mark.parametrize("n,p,s,powers", [(1000, 1 << 20, 16, 16), (1000, 1 << 20, 32, 16),
                                          (1025, 1 << 20, 16, 16), (1025, 1 << 20, 32, 32),
                                          (20000, 1 << 20, 16, 16), (20000, 1 << 20, 32, 32),
                                          (5000, 100, 16, 16), (5000, 100, 32, 32)])
def test_poly_powers_per_column(so, n, p, s, powers):
    """With s = 16 a column never holds more than 16 powers (32 cost precision)."""
    job = dict(fn="tcu_poly_eval_ex", args=[rec.ptr(0), n, rec.ptr(1), p, rec.ptr(2), s, BF16, None])
    assert kernels(rec.run(so, [job])[0])[0].startswith(f"poly_kernelILi{BF16}ELi{powers}E")
