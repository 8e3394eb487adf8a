"""Products on pre-split operands (reduced precision), every tile height whole
and cut along k, at the edges of the tiles, against numpy.

Bars, relative in the Frobenius norm: each operand keeps 2^-18 of a component
(two bf16 parts, rounded to nearest) or 2^-9 (B in X2), FP32 2^-24 and one more
rounding of its sum planes; FP32 accumulation over K terms and the rounding of
a partial sum add at most about sqrt(2 K) 2^-23.  X3: (2 + 1) 2^-18 (two
operands, the dropped lo*lo term) + sqrt(2K) 2^-23; X2: 2^-9 + the same; FP32,
whose Gauss terms are up to twice the result: 4 (2^-23 + sqrt(2K) 2^-23)."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
P, I, D = ctypes.c_void_p, ctypes.c_int, ctypes.c_double
CODES = {"fp32": 1, "bf16x3": 2, "bf16x2": 3}


def bar(prec, K):
    acc = np.sqrt(2.0 * K) * 2.0 ** -23
    return {"fp32": 4 * (2.0 ** -23 + acc), "bf16x3": 3 * 2.0 ** -18 + acc, "bf16x2": 2.0 ** -9 + 3 * 2.0 ** -18 + acc}[prec]


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_14296_amd as cc
    L = cc.lib()
    L.cclr_dbg_split_product.argtypes = [I] * 6 + [P] * 3 + [D, D, I, ctypes.POINTER(I)]
    return L


def run(L, prec, bm, cutters, M, N, K, beta, wants_cut=None):
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    A, B, C0 = (rng.normal(size=(x, y)) + 1j * rng.normal(size=(x, y)) for x, y in ((M, K), (K, N), (M, N)))
    Ad, Bd, Cd = (torch.as_tensor(x).cuda() for x in (A, B, C0))
    alpha, cut = 0.7 - 0.3j, I(-1)
    print(f"{prec} bm {bm} cutters {cutters}: {M}x{N}x{K} beta {beta}", flush=True)
    rc = L.cclr_dbg_split_product(CODES[prec], bm, cutters, M, N, K, Ad.data_ptr(), Bd.data_ptr(), Cd.data_ptr(),
                                  alpha.real, alpha.imag, beta, ctypes.byref(cut))
    assert rc == 0
    prod = alpha * (A @ B)
    e = np.linalg.norm(Cd.cpu().numpy() - (C0 if beta else 0) - prod) / np.linalg.norm(prod)
    print(f"{cut.value} tiles cut, rel err {e:.2e}, bar {bar(prec, K):.2e}", flush=True)
    assert e < bar(prec, K)
    if wants_cut is not None:
        assert (cut.value > 0) == wants_cut


# one entry; tile edges in m and n; K of one step, a step and one, ragged; one
# run per few steps; whole rounds of 256 tiles with a cut rest
@pytest.mark.parametrize("prec", list(CODES))
@pytest.mark.parametrize("bm", [64, 96, 128])
@pytest.mark.parametrize("M,N,K,cutters", [(1, 1, 1, 256), (64, 128, 32, 256), (65, 129, 33, 0), (97, 130, 300, 256),
                                           (128, 127, 1000, 7), (129, 257, 2047, 256), (200, 1300, 515, 200),
                                           (1700, 2600, 260, 256)])
def test_split_tiles(lib, prec, bm, M, N, K, cutters):
    run(lib, prec, bm, cutters, M, N, K, (M + bm) % 2)


# the plan the library makes, with room for partial sums and without
@pytest.mark.parametrize("prec", list(CODES))
@pytest.mark.parametrize("M,N,K,cut", [(66, 1500, 4000, True), (264, 1200, 3000, True), (30, 40, 50, None)])
def test_split_plan(lib, prec, M, N, K, cut):
    run(lib, prec, 0, 256, M, N, K, 0, cut)
    run(lib, prec, 0, 0, M, N, K, 1, False)
