"""A reduced-precision product under a memory cap that holds its split operands
but not the partial sums of cut tiles runs whole."""
import ctypes

import pytest
import torch

from test_gpu_split_products import bar

pytestmark = pytest.mark.gpu
P, I, L, D = ctypes.c_void_p, ctypes.c_int, ctypes.c_longlong, ctypes.c_double


def test_split_operands_before_partial_sums():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_14296_amd as cc
    lib = cc.lib()
    lib.cclr_dbg_run_gemm.argtypes = [P] + [I] * 4 + [P, L, L, L, I] * 2 + [P, L, L, L, D, D, I]
    lib.cclr_dbg_set_sigma_prec.argtypes = [P, I]
    # FP32 planes: 12 bytes an entry, 195 MB of B and 28 of A, in a cap of 268; the partial sums take 50
    M, N, K = 576, 3968, 4096
    opt = cc.cclr_default_options()
    opt.device_mem_cap = 256 << 20
    ctx = cc.cclr_create(4, 16, opt)
    try:
        assert lib.cclr_dbg_set_sigma_prec(ctx, cc.CCLR_FP32) == 0
        g = torch.Generator(device="cuda").manual_seed(3)
        draw = lambda *s: torch.view_as_complex(torch.randn(*s, 2, dtype=torch.float64, device="cuda", generator=g))  # noqa: E731
        A, B = draw(M, K), draw(K, N)
        C = torch.zeros((M, N), dtype=torch.complex128, device="cuda")
        print(f"{M}x{N}x{K} under {opt.device_mem_cap} bytes", flush=True)
        rc = lib.cclr_dbg_run_gemm(ctx, M, N, K, 1, A.data_ptr(), 0, K, 1, 0, B.data_ptr(), 0, N, 1, 0, C.data_ptr(), 0,
                                   N, 1, 1.0, 0.0, 0)
        assert rc == 0
        ref = A @ B
        assert float(torch.linalg.norm(C - ref) / torch.linalg.norm(ref)) < bar("fp32", K)
    finally:
        cc.cclr_destroy(ctx)
