"""The partial sums of cut tiles keep what the accumulators hold: products whose
accumulators are whole numbers below 2^24, exact in FP32, but whose real parts
over one run need 25 bits.  Operands are whole numbers of at most 8 bits (exact
in bf16), so the result is the exact product, bit for bit."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
P, I, D = ctypes.c_void_p, ctypes.c_int, ctypes.c_double
CODES = {"fp32": 1, "bf16x3": 2, "bf16x2": 3}


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_14296_amd as cc
    L = cc.lib()
    L.cclr_dbg_split_product.argtypes = [I] * 6 + [P] * 3 + [D, D, I, ctypes.POINTER(I)]
    return L


@pytest.mark.parametrize("prec", list(CODES))
@pytest.mark.parametrize("bm", [64, 96, 128])
# K and the number of runs: 256 values of k in each run of the one tile
@pytest.mark.parametrize("K,cutters", [(512, 2), (1024, 4)])
def test_exact_partial_sums(lib, prec, bm, K, cutters):
    M, N = 50, 120
    rng = np.random.default_rng(K + bm)
    draw = lambda lo, hi, *s: rng.integers(lo, hi + 1, size=s).astype(np.float64)  # noqa: E731
    A = draw(254, 255, M, K) - 1j * draw(29, 35, M, K)
    B = draw(254, 255, K, N) + 1j * draw(29, 35, K, N)
    # per run: Ar Br and k1 at most 256 * 255^2 < 2^24, Re = Ar Br - Ai Bi above it
    runs = [slice(k, k + 256) for k in range(0, K, 256)]
    for r in runs:
        assert (A.real[:, r] @ B.real[r]).max() < 2 ** 24
    parts = np.stack([(A[:, r] @ B[r]).real for r in runs])
    assert parts.min() > 2 ** 24 and (parts % 2 == 1).any()
    Ad, Bd = torch.as_tensor(A).cuda(), torch.as_tensor(B).cuda()
    Cd, cut = torch.zeros((M, N), dtype=torch.complex128, device="cuda"), I(-1)
    print(f"{prec} bm {bm} K {K} cutters {cutters}", flush=True)
    rc = lib.cclr_dbg_split_product(CODES[prec], bm, cutters, M, N, K, Ad.data_ptr(), Bd.data_ptr(), Cd.data_ptr(),
                                    1.0, 0.0, 0, ctypes.byref(cut))
    assert rc == 0 and cut.value == 1
    assert np.array_equal(Cd.cpu().numpy(), A @ B)
