"""The work the library is timed on: every computing entry point of the Python
binding, from the smallest calls to the largest, in the shapes, types and
options a program uses them in.

A case is a dict of plain values; ``kind`` names the entry point:

    tall      tcu_mm_tall_ex             n, s, dtype
    product   tcu_gemm_ex                N, s, dtype
    rect      tcu_gemm_rect_ex           M, K, N, s, dtype, acc, pad (extra elements per row)
    poly      tcu_poly_eval_ex           n, p, s, dtype
    closure   tcu_transitive_closure_ex  n, deg (mean out-degree), pad
    dft       tcu_dft_ex                 n, batch, s

The stateless forms are used, so that a pass does not depend on the calls of
another case.  Inputs have the distributions of the library's own workloads
(uniform or normal values rounded once to the storage type, uniform int8, a
random digraph, a normal complex signal).
"""
import math

import torch

from paper_1908_06649_amd import tcu

# dtype name -> (input type, output type)
DTYPES = {"f16": (torch.float16, torch.float32),
          "bf16": (torch.bfloat16, torch.float32),
          "bf16out": (torch.bfloat16, torch.bfloat16),
          "i8": (torch.int8, torch.int32)}

DEVICE = "cuda"


def listed():
    return [
        # One native call on a few thousand rows: launch latency.
        dict(name="tall_f16_n4096_s16", kind="tall", n=4096, s=16, dtype="f16"),
        # A native call over far more rows than the caches hold: a projection
        # of a large table by a small matrix, memory bandwidth.
        dict(name="tall_bf16_n16777216_s32", kind="tall", n=1 << 24, s=32, dtype="bf16out"),
        # The small square product a solver or a small network calls in a loop.
        dict(name="product_f16_N1024_s16", kind="product", N=1024, s=16, dtype="f16"),
        # An ordinary quantised product.
        dict(name="product_i8_N3072_s32", kind="product", N=3072, s=32, dtype="i8"),
        # The largest dense product.
        dict(name="product_bf16_N8192_s32", kind="product", N=8192, s=32, dtype="bf16"),
        # A small block built up over a long contracted dimension (covariances,
        # gradients of a narrow layer), accumulated into a view of a larger array.
        dict(name="rect_f16_192x8192x320_acc", kind="rect", M=192, K=8192, N=320, s=16,
             dtype="f16", acc=True, pad=32),
        # Sizes as data has them: no dimension a multiple of anything, rows of
        # B and C that start at any 2-byte address.
        dict(name="rect_bf16_4101x1000x4173", kind="rect", M=4101, K=1000, N=4173, s=32,
             dtype="bf16out", acc=False, pad=0),
        # Evaluation of one polynomial at many points.
        dict(name="poly_bf16_n4096_p16777216", kind="poly", n=4096, p=1 << 24, s=32, dtype="bf16"),
        # Reachability in a small graph, its size not a multiple of a block.
        dict(name="closure_n1000", kind="closure", n=1000, deg=2.0, pad=0),
        # Reachability in the largest graph.
        dict(name="closure_n8192", kind="closure", n=8192, deg=2.0, pad=0),
        # Many short transforms (frames of a signal).
        dict(name="dft_n4096_b512_s32", kind="dft", n=4096, batch=512, s=32),
        # A few long transforms.
        dict(name="dft_n1048576_b16_s32", kind="dft", n=1 << 20, batch=16, s=32),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _any_or_round(rng, v, unit):
    """v as it is, or as a multiple of `unit`: programs pass both."""
    return max(unit, v // unit * unit) if rng.random() < 0.5 else v


def draw(rng):
    kind = rng.choice(["tall", "product", "rect", "poly", "closure", "dft"])
    s = rng.choice([16, 32])
    if kind == "tall":
        return dict(kind=kind, n=_any_or_round(rng, _log_int(rng, 256, 1 << 24), 64), s=s,
                    dtype=rng.choice(list(DTYPES)))
    if kind == "product":
        return dict(kind=kind, N=_log_int(rng, 64, 8192) // s * s, s=s,
                    dtype=rng.choice(list(DTYPES)))
    if kind == "rect":
        M, K, N = (_any_or_round(rng, _log_int(rng, 16, 8192), 64) for _ in range(3))
        pad = rng.choice([0, 0, 64, rng.randint(1, 63)])
        # keep the work below the largest listed case's, with room for the
        # element-wise paths of odd pitches
        K = max(16, min(K, (1 << 35) // (M * N)))
        return dict(kind=kind, M=M, K=K, N=N, s=s, dtype=rng.choice(list(DTYPES)),
                    acc=rng.random() < 0.5, pad=pad)
    if kind == "poly":
        n = _any_or_round(rng, _log_int(rng, 16, 1 << 16), 64)
        p = _any_or_round(rng, _log_int(rng, 256, min(1 << 24, (1 << 35) // n)), 64)
        return dict(kind=kind, n=n, p=p, s=s, dtype=rng.choice(["f16", "bf16", "bf16out"]))
    if kind == "closure":
        # ragged graphs and odd pitches cost more per vertex
        if rng.random() < 0.5:
            n, pad = _log_int(rng, 64, 1500), rng.choice([0, 0, 16, rng.randint(1, 31)])
        else:
            n, pad = max(1, _log_int(rng, 128, 8192) // 256) * 256, rng.choice([0, 16])
        return dict(kind=kind, n=n, deg=round(rng.uniform(0.5, 4.0), 2), pad=pad)
    lg = rng.randint(4, 20)
    batch = _log_int(rng, 1, 1 << (24 - lg))
    return dict(kind=kind, n=1 << lg, batch=batch, s=s)


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _values(shape, dtype, dist, g):
    if dtype == torch.int8:
        return torch.randint(-128, 128, shape, generator=g, dtype=torch.int8, device=DEVICE)
    if dist == "uniform":
        x = torch.rand(shape, generator=g, device=DEVICE).mul_(2.0).sub_(1.0)
    else:
        x = torch.randn(shape, generator=g, device=DEVICE)
    return x.to(dtype)


def _view(rows, cols, pad, dtype):
    return torch.zeros((rows, cols + pad), dtype=dtype, device=DEVICE)[:, :cols]


def prepare(case, seed):
    kind = case["kind"]
    g = _gen(seed)
    st = dict(case)
    if kind in ("tall", "product", "rect"):
        it, ot = DTYPES[case["dtype"]]
        dist = "uniform" if case["dtype"] == "f16" else "normal"
        if kind == "tall":
            M, K, N = case["n"], case["s"], case["s"]
        elif kind == "product":
            M = K = N = case["N"]
        else:
            M, K, N = case["M"], case["K"], case["N"]
        pad = case.get("pad", 0)
        A, B, C = _view(M, K, pad, it), _view(K, N, pad, it), _view(M, N, pad, ot)
        A.copy_(_values((M, K), it, dist, g))
        B.copy_(_values((K, N), it, dist, g))
        if case.get("acc"):
            if ot == torch.int32:
                C.copy_(torch.randint(-(1 << 20), 1 << 20, (M, N), generator=g,
                                      dtype=torch.int32, device=DEVICE))
            else:
                C.copy_(torch.randn((M, N), generator=g, device=DEVICE))
        st.update(A=A, B=B, C=C)
    elif kind == "poly":
        it, ot = DTYPES[case["dtype"]]
        coef = _values((case["n"],), it, "normal", g)
        pts = _values((case["p"],), it, "uniform", g)
        st.update(coef=coef, pts=pts, out=torch.zeros(case["p"], dtype=ot, device=DEVICE))
    elif kind == "closure":
        n = case["n"]
        graph = (torch.rand((n, n), generator=g, device=DEVICE) < case["deg"] / n).to(torch.int8)
        st.update(graph=graph, X=_view(n, n, case["pad"], torch.int8))
    else:
        n, batch = case["n"], case["batch"]
        x = torch.view_as_complex(torch.randn((batch, n, 2), generator=g, device=DEVICE))
        st.update(x=x, y=torch.zeros_like(x), work=torch.empty_like(x))
    return st


def run(st):
    kind = st["kind"]
    if kind == "tall":
        tcu.tcu_mm_tall_ex(st["A"], st["n"], st["s"], st["B"], st["C"])
        return st["C"]
    if kind == "product":
        tcu.tcu_gemm_ex(st["A"], st["B"], st["C"], st["N"], st["s"])
        return st["C"]
    if kind == "rect":
        pad, K, N = st["pad"], st["K"], st["N"]
        tcu.tcu_gemm_rect_ex(st["A"], K + pad, st["B"], N + pad, st["C"], N + pad, st["M"], K, N,
                             tcu.TCU_ACCUMULATE if st["acc"] else 0, st["s"])
        return st["C"]
    if kind == "poly":
        tcu.tcu_poly_eval_ex(st["coef"], st["n"], st["pts"], st["p"], st["out"], st["s"])
        return st["out"]
    if kind == "closure":
        # the call works in place: the program keeps its graph
        st["X"].copy_(st["graph"])
        tcu.tcu_transitive_closure_ex(st["X"], st["n"], st["n"] + st["pad"], 32)
        return st["X"]
    tcu.tcu_dft_ex(st["x"], st["y"], st["work"], st["n"], st["batch"], st["s"])
    return st["y"]


# ------------------------------------------------- what a pass cannot avoid
def _product_work(M, K, N, dtype, acc):
    it, ot = DTYPES[dtype]
    out = M * N * ot.itemsize
    return {"bytes": (M * K + K * N) * it.itemsize + out * (2 if acc else 1),
            "flops": 2.0 * M * K * N}


def work(case):
    kind = case["kind"]
    if kind == "tall":
        return _product_work(case["n"], case["s"], case["s"], case["dtype"], False)
    if kind == "product":
        N = case["N"]
        return _product_work(N, N, N, case["dtype"], False)
    if kind == "rect":
        return _product_work(case["M"], case["K"], case["N"], case["dtype"], case["acc"])
    if kind == "poly":
        it, ot = DTYPES[case["dtype"]]
        return {"bytes": case["n"] * it.itemsize + case["p"] * (it.itemsize + ot.itemsize),
                "flops": 2.0 * case["n"] * case["p"]}
    if kind == "closure":
        n = case["n"]
        return {"bytes": 2.0 * n * n, "flops": 2.0 * n ** 3}
    n, batch = case["n"], case["batch"]
    return {"bytes": 2.0 * 8 * n * batch, "flops": 5.0 * n * max(1, n.bit_length() - 1) * batch}


def tolerance(case):
    kind = case["kind"]
    if kind == "closure" or case.get("dtype") == "i8":
        return "exact"
    if case.get("dtype") == "bf16out":
        return {"rel": 1e-2}
    if kind in ("tall", "product", "rect"):
        return {"rel": 2.5e-6}   # binary32 sums of up to 8192 products
    if kind == "poly":
        return {"rel": 1e-5}     # powers carried to about 2^-17
    return {"rel": 3e-5}         # data and roots carried to about 2^-16 per level


# --------------------------------------------------------- the same in 64 bits
def exact(case, seed):
    kind = case["kind"]
    st = prepare(case, seed)
    if kind in ("tall", "product", "rect"):
        C = st["A"].double() @ st["B"].double()
        if case.get("acc"):
            C += st["C"].double()
        if case["dtype"] == "i8":
            C = C.to(torch.int64).to(torch.int32)    # sums below 2^53; int32 wraps
        return C
    if kind == "poly":
        x = st["pts"].double()
        y = torch.zeros_like(x)
        for a in reversed(st["coef"].double().tolist()):
            y.mul_(x).add_(a)
        return y
    if kind == "closure":
        # paths of up to 2^k edges, doubled until nothing is added
        R = st["graph"].double()
        edges = R.sum()
        while True:
            R = ((R + R @ R) > 0).double()
            now = R.sum()
            if bool(now == edges):
                return R.to(torch.int8)
            edges = now
    return torch.fft.fft(st["x"].to(torch.complex128))
