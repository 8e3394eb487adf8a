"""The record of large FP64 products holds products of 1e10 flop and more by
their own shape; the parts of one that is split along K are not among them."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu
P, I, L, D = ctypes.c_void_p, ctypes.c_int, ctypes.c_longlong, ctypes.c_double


# flop: 4.1e9, split along K in 74 parts (no room for the partial sums of the even split); 1.4e10, whole
@pytest.mark.parametrize("M,N,K,fails,recorded", [(160, 160, 20000, 6, False), (6000, 6000, 50, 0, True)])
def test_recorded_products(M, N, K, fails, recorded):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_14296_amd as cc
    lib = cc.lib()
    lib.cclr_dbg_run_gemm.argtypes = [P] + [I] * 4 + [P, L, L, L, I] * 2 + [P, L, L, L, D, D, I]
    lib.cclr_dbg_tuning.argtypes = [P, I, ctypes.c_char_p, L]
    lib.cclr_dbg_gemm_trace.argtypes = [P, I, ctypes.c_char_p, L]
    lib.cclr_dbg_fail_allocs.argtypes = [P, I]
    A, B = (torch.ones(s, dtype=torch.complex128, device="cuda") for s in ((M, K), (K, N)))
    C = torch.empty((M, N), dtype=torch.complex128, device="cuda")
    ctx = cc.cclr_create(4, 16)
    try:
        assert lib.cclr_dbg_gemm_trace(ctx, 1, None, 0) == 0
        assert lib.cclr_dbg_fail_allocs(ctx, fails) == 0
        assert lib.cclr_dbg_run_gemm(ctx, M, N, K, 1, A.data_ptr(), 0, K, 1, 0, B.data_ptr(), 0, N, 1, 0, C.data_ptr(), 0,
                                     N, 1, 1.0, 0.0, 0) == 0
        assert bool((C == K).all())
        buf = ctypes.create_string_buffer(1 << 14)
        assert lib.cclr_dbg_gemm_trace(ctx, 0, buf, len(buf)) == 0
        trace = buf.value.decode()
        assert ("form -2" in trace) == (fails > 0), trace
        assert lib.cclr_dbg_tuning(ctx, -1, buf, len(buf)) == 0
        lines = buf.value.decode().splitlines()
        print(trace, lines, flush=True)
        assert [ln.split(":")[0] for ln in lines] == ([f"{M}x{N}x{K} b1"] if recorded else [])
    finally:
        cc.cclr_destroy(ctx)
