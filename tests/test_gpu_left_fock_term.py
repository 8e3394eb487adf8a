"""The one-body term P(ij) P(ab) l^i_a F^j_b of the left transform is FP64 in
every arithmetic: with a Fock matrix alone (no integrals, no amplitudes) and
singles alone it is the whole of the doubles."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["CCLR_FP64", "CCLR_FP32", "CCLR_BF16X3", "CCLR_BF16X2"])
@pytest.mark.parametrize("o,v,n", [(6, 64, 3), (4, 16, 1)])  # on the GEMM tiles, and as a small product
def test_fock_term_of_the_left_transform(prec, o, v, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_14296_amd as cc
    lib = cc.lib()
    lib.cclr_dbg_set_sigma_prec.argtypes = [ctypes.c_void_p, ctypes.c_int]
    g = torch.Generator(device="cuda").manual_seed(o + v)
    draw = lambda *s: torch.view_as_complex(torch.randn(*s, 2, dtype=torch.float64, device="cuda", generator=g))  # noqa: E731
    zeros = lambda *s: torch.zeros(s, dtype=torch.complex128, device="cuda")  # noqa: E731
    f = draw(o + v, o + v)
    f = f + f.conj().T.contiguous()
    ctx = cc.cclr_create(o, v)
    try:
        cc.cclr_set_hamiltonian(ctx, f, *[zeros(*[o if c == "o" else v for c in k])
                                          for k in ("oooo", "ooov", "oovv", "ovov", "ovvv", "vvvv")])
        cc.cclr_set_amplitudes(ctx, zeros(o, v), zeros(o, o, v, v))
        assert lib.cclr_dbg_set_sigma_prec(ctx, getattr(cc, prec)) == 0
        l1, l2 = draw(n, o, v), zeros(n, o, o, v, v)
        s1, s2 = torch.empty_like(l1), torch.empty_like(l2)
        print(f"{prec} o={o} v={v} n={n}", flush=True)
        cc.cclr_jacobian_left(ctx, [0.0] * n, [0.0] * n, l1, l2, s1, s2)
        t = l1[:, :, None, :, None] * f[None, None, :o, None, o:]
        t = t - t.transpose(3, 4)
        ref = t - t.transpose(1, 2)
        # at most four products and three sums of entries below max|l| max|f|
        err = float((s2 - ref).abs().max() / (l1.abs().max() * f.abs().max()))
        print(f"largest error {err:.1e}", flush=True)
        assert err < 16 * 2.0 ** -53
    finally:
        cc.cclr_destroy(ctx)
