"""The contraction engine's choice between one product with copied tensors and
batched products without: every order of labels of random contractions, unit
extents and odd sizes among them, against numpy's einsum.

Tolerance: as for a product of inner length K, 2 (2 K + 16) 2^-53 |alpha|
sum |A| |B| per entry plus two roundings of the result."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
LL, P, D = ctypes.c_longlong, ctypes.c_void_p, ctypes.c_double
EPS = 2.0 ** -53


@pytest.fixture(scope="module")
def engine():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_14296_amd as cc
    L = cc.lib()
    L.cclr_dbg_contract.argtypes = [P, D, D, P, ctypes.c_char_p, ctypes.POINTER(LL), P, ctypes.c_char_p,
                                    ctypes.POINTER(LL), P, ctypes.c_char_p, ctypes.POINTER(LL)]
    ctx = cc.cclr_create(3, 6, cc.cclr_default_options())
    yield L, ctx
    cc.cclr_destroy(ctx)


def run(L, ctx, rng, la, lb, lc, ext):
    A, B, C = (rng.normal(size=[ext[x] for x in l]) + 1j * rng.normal(size=[ext[x] for x in l]) for l in (la, lb, lc))
    Ad, Bd, Cd = (torch.as_tensor(x).cuda() for x in (A, B, C))
    dims = lambda x: (LL * x.ndim)(*x.shape)  # noqa: E731
    alpha = -0.5 + 0.25j
    assert L.cclr_dbg_contract(ctx, alpha.real, alpha.imag, Ad.data_ptr(), la.encode(), dims(A), Bd.data_ptr(),
                               lb.encode(), dims(B), Cd.data_ptr(), lc.encode(), dims(C)) == 0
    K = int(np.prod([ext[x] for x in la if x not in lc]))
    ref = C + alpha * np.einsum(f"{la},{lb}->{lc}", A, B)
    bound = (2 * (2 * K + 16) * EPS * abs(alpha) * np.einsum(f"{la},{lb}->{lc}", np.abs(A), np.abs(B))
             + 2 * EPS * (np.abs(ref) + np.abs(C)))
    worst = (np.abs(Cd.cpu().numpy() - ref) / bound).max()
    assert worst <= 1.0, (la, lb, lc, ext, worst)


@pytest.mark.parametrize("seed", range(6))
def test_random_label_orders(engine, seed):
    L, ctx = engine
    rng = np.random.default_rng(seed)
    for n in range(60):
        nm, nn, nk = rng.integers(1, 4), rng.integers(0, 3), rng.integers(1, 3)
        m, nl, k = "abc"[:nm], "ij"[:nn], "xy"[:nk]
        mix = lambda s: "".join(rng.permutation(list(s)))  # noqa: E731
        la, lb, lc = mix(m + k), mix(nl + k), mix(m + nl)
        ext = {x: int(rng.choice([1, 2, 3, 5, 17, 33] if x in "abcij" else [1, 4, 7, 40])) for x in "abcijxy"}
        print(f"{la},{lb}->{lc} {ext}", flush=True)
        run(L, ctx, rng, la, lb, lc, ext)


# the shapes of the transforms: k vectors, P = pair of m and n, Q = pair of e and f
@pytest.mark.parametrize("la,lb,lc", [
    ("mbP", "kma", "kPab"), ("Pie", "kPea", "kia"), ("Paf", "kbf", "kPab"), ("Pef", "kPeb", "kbf"), ("mi", "kma", "kia"),
    ("nmQ", "kjmQ", "knj"), ("jeQ", "kie", "kijQ"), ("inQ", "knj", "kijQ"), ("bmef", "kme", "kbf"), ("imab", "kjm", "kijab")])
@pytest.mark.parametrize("k,o,v", [(1, 3, 7), (3, 4, 33), (5, 9, 20)])
def test_transform_contractions(engine, la, lb, lc, k, o, v):
    ext = {x: o for x in "ijmn"} | {x: v for x in "abef"} | {"k": k, "P": o * (o - 1) // 2, "Q": v * (v - 1) // 2}
    run(*engine, np.random.default_rng(o + v), la, lb, lc, ext)
