"""The strided copy's transposing tiles at short and ragged extents, against
torch's permute: bit for bit as a copy, one rounding when it accumulates."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_14296_amd as cc
    L = cc.lib()
    LL, P, I, D = ctypes.c_longlong, ctypes.c_void_p, ctypes.c_int, ctypes.c_double
    L.cclr_dbg_tcopy.argtypes = [I, P, P, P, P, P, D, D, I, I]
    return L


# the source's last extent becomes the stride, the destination's last one the
# unit: 3 and 4 (the shortest tiled), 15 to 17 and 63 to 65 (tile edges), both
# short (12 x 12 tiled, 8 x 11 not), and with a batch between them
SHAPES = [((40, 3), (1, 0)), ((40, 4), (1, 0)), ((4, 17), (1, 0)), ((65, 15), (1, 0)), ((63, 16), (1, 0)),
          ((64, 17), (1, 0)), ((15, 64), (1, 0)), ((16, 129), (1, 0)), ((33, 31), (1, 0)), ((12, 9, 12), (2, 1, 0)),
          ((8, 7, 11), (2, 1, 0)), ((19, 5, 3, 12), (3, 1, 2, 0)), ((12, 3, 5, 70), (3, 2, 1, 0)),
          ((18, 2, 3, 5, 6), (4, 3, 2, 1, 0))]


@pytest.mark.parametrize("shape,perm", SHAPES)
def test_transposing_copy(lib, shape, perm):
    LL = ctypes.c_longlong
    src = torch.randn(shape, dtype=torch.complex128, generator=torch.Generator().manual_seed(1)).cuda()
    out = [shape[p] for p in perm]
    nd = len(shape)
    st = [int(np.prod(shape[d + 1:])) for d in range(nd)]
    dims = (LL * nd)(*out)
    sd = (LL * nd)(*[int(np.prod(out[d + 1:])) for d in range(nd)])
    ss = (LL * nd)(*[st[p] for p in perm])
    dst = torch.full(out, 7.0 + 0j, dtype=torch.complex128, device="cuda")
    print(shape, perm, flush=True)
    assert lib.cclr_dbg_tcopy(nd, dims, sd, ss, dst.data_ptr(), src.data_ptr(), 1.0, 0.0, 0, 0) == 0
    want = src.permute(*perm)
    assert torch.equal(dst, want)
    assert lib.cclr_dbg_tcopy(nd, dims, sd, ss, dst.data_ptr(), src.data_ptr(), 1.0, 0.0, 1, 1) == 0
    assert torch.equal(dst, want + want.conj())
