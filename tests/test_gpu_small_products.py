"""The engine's kernels for small and unevenly filling FP64 products, at the
edges of their tiles and of the rules that choose them, against numpy.

Tolerance: each of the two sides sums K complex products (four real ones
each) in FP64 in some order, so an entry differs by at most
2 (2 K + 16) 2^-53 |alpha| (|A| |B|) plus two roundings of the result."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
LL, P, I, D = ctypes.c_longlong, ctypes.c_void_p, ctypes.c_int, ctypes.c_double
EPS = 2.0 ** -53


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_14296_amd as cc
    L = cc.lib()
    L.cclr_dbg_run_gemm.argtypes = [P] + [I] * 4 + [P, LL, LL, LL, I, P, LL, LL, LL, I, P, LL, LL, LL, D, D, I]
    L.cclr_dbg_run_gemm_b2.argtypes = [P] + [I] * 5 + [P, LL, LL, LL, LL, P, LL, LL, LL, LL, P, LL, LL, LL, LL, D, D, I]
    L.cclr_dbg_gemm_trace.argtypes = [P, I, ctypes.c_char_p, LL]
    ctx = cc.cclr_create(3, 6, cc.cclr_default_options())
    yield L, ctx
    cc.cclr_destroy(ctx)


def crand(rng, *shape):
    return rng.normal(size=shape) + 1j * rng.normal(size=shape)


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


def forms(L, ctx):
    buf = ctypes.create_string_buffer(1 << 16)
    assert L.cclr_dbg_gemm_trace(ctx, 0, buf, len(buf)) == 0
    return [int(ln.split(" form ")[1].split()[0]) for ln in buf.value.decode().splitlines() if ln]


def check(got, A, B, C0, alpha, K):
    ref = alpha * (A @ B) + C0
    bound = 2 * (2 * K + 16) * EPS * abs(alpha) * (np.abs(A) @ np.abs(B)) + 2 * EPS * (np.abs(ref) + np.abs(C0))
    worst = (np.abs(got - ref) / bound).max()
    print(f"worst entry at {worst:.2f} of its bound", flush=True)
    assert worst <= 1.0


def product(L, ctx, M, N, K, batch, ta, tb, tc, conjA, conjB, beta, form):
    rng = np.random.default_rng(M + 3 * N + 7 * K + batch)
    A, B, C0 = crand(rng, batch, M, K), crand(rng, batch, K, N), crand(rng, batch, M, N)
    Ad = dev(A.transpose(0, 2, 1) if ta else A)
    Bd = dev(B.transpose(0, 2, 1) if tb else B)
    Cd = dev(C0.transpose(0, 2, 1) if tc else C0)
    sA, sB, sC = (1, M) if ta else (K, 1), (1, K) if tb else (N, 1), (1, M) if tc else (N, 1)
    alpha = 0.7 - 0.4j
    print(f"{M}x{N}x{K} b{batch} ta={ta} tb={tb} tc={tc} conj=({conjA},{conjB}) beta={beta}", flush=True)
    assert L.cclr_dbg_gemm_trace(ctx, 1, None, 0) == 0
    rc = L.cclr_dbg_run_gemm(ctx, M, N, K, batch, Ad.data_ptr(), M * K, *sA, conjA, Bd.data_ptr(), K * N, *sB, conjB,
                             Cd.data_ptr(), M * N, *sC, alpha.real, alpha.imag, beta)
    assert rc == 0
    assert forms(L, ctx) == [form]
    got = Cd.cpu().numpy()
    check(got.transpose(0, 2, 1) if tc else got, A.conj() if conjA else A, B.conj() if conjB else B,
          C0 if beta else 0 * C0, alpha, K)


LAYOUTS = [(False, False, False, 0, 1, 0), (True, False, True, 1, 0, 1), (False, True, False, 1, 1, 1)]

# register kernel: one entry; one block and one beyond it; K of one tile, one
# more, a ragged tile in a cut reduction; the last size of the 5120 block-tile
# rule; tiles of 32 x 16, 16 x 32 and 32 x 32; long reductions at their limits
FRAG = [(1, 1, 1, 1), (16, 16, 16, 1), (17, 15, 17, 3), (4, 4, 480, 1), (33, 16, 33, 2), (16, 256, 4096, 1),
        (256, 320, 256, 1), (500, 40, 40, 1), (2, 3000, 31, 2), (48, 640, 601, 1), (80, 128, 5000, 1),
        (10, 10, 70001, 1), (83850, 10, 10, 1), (9, 120, 20000, 2), (64, 64, 64, 16), (128, 192, 3001, 1),
        (200, 160, 1600, 1), (80, 80, 3600, 3), (40, 33, 513, 14),
        (70001, 12, 90, 1), (16, 40003, 129, 1), (9, 6000, 511, 4), (70000, 16, 33, 2)]


@pytest.mark.parametrize("M,N,K,batch", FRAG)
@pytest.mark.parametrize("ta,tb,tc,conjA,conjB,beta", LAYOUTS)
def test_register_kernel(lib, M, N, K, batch, ta, tb, tc, conjA, conjB, beta):
    product(*lib, M, N, K, batch, ta, tb, tc, conjA, conjB, beta, -7)


def test_register_kernel_two_level_batch(lib):
    """b = b1 nb2 + b2 with B shared over b2; a cut reduction among them."""
    L, ctx = lib
    for M, N, K, nb1, nb2 in ((20, 12, 33, 3, 2), (12, 20, 3000, 2, 2)):
        rng = np.random.default_rng(K)
        A, B, C0 = crand(rng, nb1, nb2, M, K), crand(rng, nb1, 1, K, N), crand(rng, nb1, nb2, M, N)
        Ad, Bd, Cd = dev(A), dev(B), dev(C0)
        assert L.cclr_dbg_gemm_trace(ctx, 1, None, 0) == 0
        rc = L.cclr_dbg_run_gemm_b2(ctx, M, N, K, nb1, nb2, Ad.data_ptr(), nb2 * M * K, M * K, K, 1, Bd.data_ptr(),
                                    K * N, 0, N, 1, Cd.data_ptr(), nb2 * M * N, M * N, N, 1, 0.5, 0.25, 1)
        assert rc == 0 and forms(L, ctx) == [-7]
        check(Cd.cpu().numpy(), A, B, C0, 0.5 + 0.25j, K)


# chunk sums: one to 32 threads per output, chunk counts that leave remainders
# (the vector kernels' cut reductions and the split-K tiles)
@pytest.mark.parametrize("M,N,K,batch,form", [(300, 1, 100003, 1, -6), (2000, 3, 9001, 2, -6), (3, 3000, 5000, 1, -4),
                                              (70, 2, 40000, 3, -6)])
def test_chunk_sums(lib, M, N, K, batch, form):
    product(*lib, M, N, K, batch, False, False, False, 1, 0, 1, form)


# even split: every row count of the tile in both orientations (45, 66, 91,
# 130, 180 rows against long sides), K tails and K of whole tiles, whole
# rounds with a cut rest, fewer runs than workgroups, batches
EVEN = [(45, 1000, 1530, 1), (1000, 66, 728, 1), (91, 700, 900, 1), (180, 513, 2047, 1), (130, 190, 9000, 1),
        (1500, 1500, 300, 1), (65, 65, 2401, 4), (200, 200, 700, 3), (33, 2000, 900, 1), (500, 300, 260, 2)]


@pytest.mark.parametrize("M,N,K,batch", EVEN)
@pytest.mark.parametrize("ta,tb,tc,conjA,conjB,beta", LAYOUTS)
def test_even_split(lib, M, N, K, batch, ta, tb, tc, conjA, conjB, beta):
    product(*lib, M, N, K, batch, ta, tb, tc, conjA, conjB, beta, -8)


# the tile rule: each tile it names (10: 64x64, 15 and 16: 128x128 in plain and
# grouped order, 19: 128x32, 20: 64x32, 100 + v: on the transposed product),
# ragged in every extent, and 32 and 33 columns and 64 and 65 rows
TILES = [(1301, 1289, 101, 1, 10), (2047, 2041, 239, 1, 15), (2041, 2047, 333, 1, 16), (90, 89, 201, 80, 19),
         (701, 690, 99, 1, 20), (70, 1000, 239, 10, 119), (70, 1999, 99, 8, 120), (3000, 32, 250, 1, 19),
         (64, 32, 90, 130, 20), (65, 32, 90, 130, 19), (3000, 33, 250, 1, 20)]


@pytest.mark.parametrize("M,N,K,batch,form", TILES)
@pytest.mark.parametrize("ta,tb,tc,conjA,conjB,beta", LAYOUTS)
def test_tile_rule(lib, M, N, K, batch, form, ta, tb, tc, conjA, conjB, beta):
    product(*lib, M, N, K, batch, ta, tb, tc, conjA, conjB, beta, form)


@pytest.mark.parametrize("fm", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("M,N,K,batch,cutters", [(97, 70, 300, 1, 512), (97, 70, 300, 1, 0), (161, 1, 129, 2, 512),
                                                 (16, 64, 4100, 1, 7), (700, 3000, 140, 1, 512),
                                                 (700, 3000, 17, 1, 512), (33, 65, 15, 3, 512)])
def test_even_split_tiles(lib, fm, M, N, K, batch, cutters):
    """Each tile height with whole tiles only, a cut rest, a cut rest after
    whole rounds, few runs, and K below one tile."""
    L, _ = lib
    L.cclr_dbg_zgemm_even.argtypes = [I] * 6 + [P, LL, LL, LL, P, LL, LL, LL, P, LL, LL, LL, I, I]
    rng = np.random.default_rng(fm + M + K)
    A, B, C0 = crand(rng, batch, M, K), crand(rng, batch, K, N), crand(rng, batch, M, N)
    for ta, tb, conjA, beta in ((False, False, 1, 0), (True, True, 0, 1)):
        Ad, Bd, Cd = dev(A.transpose(0, 2, 1) if ta else A), dev(B.transpose(0, 2, 1) if tb else B), dev(C0)
        sA, sB = (1, M) if ta else (K, 1), (1, K) if tb else (N, 1)
        print(f"fm={fm} {M}x{N}x{K} b{batch} cutters {cutters} ta={ta}", flush=True)
        rc = L.cclr_dbg_zgemm_even(fm, cutters, M, N, K, batch, Ad.data_ptr(), M * K, *sA, Bd.data_ptr(), K * N, *sB,
                                   Cd.data_ptr(), M * N, N, 1, conjA, beta)
        assert rc == 0
        check(Cd.cpu().numpy(), A.conj() if conjA else A, B, C0 if beta else 0 * C0, 1.0, K)


def test_even_split_without_room():
    """A context whose memory cap leaves no room for partial sums runs the
    product in whole tiles."""
    import paper_2307_14296_amd as cc
    L = cc.lib()
    opt = cc.cclr_default_options()
    opt.device_mem_cap = 1 << 20
    ctx = cc.cclr_create(3, 6, opt)
    try:
        product(L, ctx, 300, 5000, 300, 1, False, False, False, 0, 0, 1, -8)
    finally:
        cc.cclr_destroy(ctx)


@pytest.mark.parametrize("shared", [1, 2])
def test_batch_innermost_input_shared_over_a_level(lib, shared):
    """An input whose unit stride is one batch index and which does not vary
    over the other (stride 0), in either order of the levels."""
    L, ctx = lib
    M, N, K, nv, ns = 90, 40, 70, 24, 9  # nv entries of A along its unit stride, shared by ns products each
    rng = np.random.default_rng(shared)
    A, C0 = crand(rng, M, K, nv), crand(rng, nv, ns, M, N)
    B = crand(rng, nv, ns, K, N)
    if shared == 1:  # the shared level is the first
        B, C0 = B.transpose(1, 0, 2, 3).copy(), C0.transpose(1, 0, 2, 3).copy()
    nb1, nb2 = (ns, nv) if shared == 1 else (nv, ns)
    Ad, Bd, Cd = dev(A), dev(B), dev(C0)
    sA1, sA2 = (0, 1) if shared == 1 else (1, 0)
    rc = L.cclr_dbg_run_gemm_b2(ctx, M, N, K, nb1, nb2, Ad.data_ptr(), sA1, sA2, K * nv, nv, Bd.data_ptr(),
                                nb2 * K * N, K * N, N, 1, Cd.data_ptr(), nb2 * M * N, M * N, N, 1, 0.5, 0.25, 1)
    assert rc == 0
    Ab = A.transpose(2, 0, 1)
    Ab = Ab[None] if shared == 1 else Ab[:, None]
    check(Cd.cpu().numpy(), Ab, B, C0, 0.5 + 0.25j, K)
