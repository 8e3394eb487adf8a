"""Work memory that contexts keep between calls is given back where an
allocation finds no room: the context's own, and that of another context on
the device.  Where it fits it stays for the next call.  That an allocation
finds no room is set from the host."""
import ctypes
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu
CHUNK = 256 << 20  # the least a context takes at a time
O, V = 4, 60


def zeros(*dims):
    return torch.zeros(dims, dtype=torch.complex128, device="cuda")


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_14296_amd as cc
    cc.lib().cclr_dbg_fail_allocs.argtypes = [ctypes.c_void_p, ctypes.c_int]
    cc.lib().cclr_dbg_allocated.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_longlong)]
    n = O + V
    H = [zeros(n, n)] + [zeros(*[O if c == "o" else V for c in k]) for k in ("oooo", "ooov", "oovv", "ovov", "ovvv", "vvvv")]
    big = zeros(1600, O, V), zeros(1600, O, O, V, V)
    out = torch.empty_like(big[0]), torch.empty_like(big[1])
    big[0].fill_(1.0)
    return cc, H, big, out


def context(cc, H):
    ctx = cc.cclr_create(O, V)
    cc.cclr_set_hamiltonian(ctx, *H)
    cc.cclr_set_amplitudes(ctx, zeros(O, V), zeros(O, O, V, V))
    return ctx


def transform(lib, ctx, n):
    """n vectors; the Hamiltonian and the amplitudes are zero, so A = 0."""
    cc, _, (r1, r2), (s1, s2) = lib
    cc.cclr_jacobian_right(ctx, [0.5] * n, [0.25] * n, r1[:n], r2[:n], s1[:n], s2[:n])
    assert bool((s1[:n] == -(0.5 + 0.25j)).all()) and not bool(s2[:n].any())


def held(cc, ctx):
    n = ctypes.c_longlong()
    assert cc.lib().cclr_dbg_allocated(ctx, ctypes.byref(n)) == 0
    return n.value


def test_own_idle_memory(lib):
    # 100 vectors leave two chunks; with 1600 the packed doubles (272 MB) fit neither
    cc, H = lib[:2]
    taken = []
    for fails in (0, 1):
        ctx = context(cc, H)
        transform(lib, ctx, 100)
        before = held(cc, ctx)
        assert cc.lib().cclr_dbg_fail_allocs(ctx, fails) == 0
        transform(lib, ctx, 1600)
        taken.append(held(cc, ctx) - before)
        transform(lib, ctx, 100)
        transform(lib, ctx, 1600)
        cc.cclr_destroy(ctx)
    print(f"taken {taken[0]} bytes, {taken[1]} with the idle chunk released", flush=True)
    assert taken[1] == taken[0] - CHUNK


def test_idle_memory_of_another_context(lib):
    cc, H = lib[:2]
    keeper = context(cc, H)
    idle = held(cc, keeper)
    transform(lib, keeper, 100)
    other = context(cc, H)
    before = held(cc, keeper)
    assert cc.lib().cclr_dbg_fail_allocs(other, 2) == 0
    cc.cclr_set_amplitudes(other, zeros(O, V), zeros(O, O, V, V))  # same sizes: keeps what it has
    transform(lib, other, 1600)
    after = held(cc, keeper)
    cc.cclr_destroy(other)
    transform(lib, keeper, 100)
    again = held(cc, keeper)
    cc.cclr_destroy(keeper)
    print(f"{before} bytes before, {after} after", flush=True)
    assert before == idle + CHUNK and after == before - 2 * CHUNK and again == before


def test_no_room_at_all(lib):
    # a call that finds none fails, hands back what it took, and the next one runs
    cc, H = lib[:2]
    ctx = context(cc, H)
    transform(lib, ctx, 1600)
    transform(lib, ctx, 100)
    for _ in range(3):
        small = context(cc, H)
        assert cc.lib().cclr_dbg_fail_allocs(small, 3) == 0
        with pytest.raises(cc.CclrError) as e:
            transform(lib, small, 1600)
        assert e.value.code == cc.CCLR_ENOMEM
        transform(lib, small, 1600)
        cc.cclr_destroy(small)
    transform(lib, ctx, 100)
    cc.cclr_destroy(ctx)


def test_second_solve_allocates_nothing(lib):
    # 300 right-hand sides with 48 slots each, 5 GB of subspace: A = 0, so x = b / z
    cc, H, (r1, r2), (s1, s2) = lib
    ctx, n = context(cc, H), 300
    for fails in (0, 3):
        assert cc.lib().cclr_dbg_fail_allocs(ctx, fails) == 0
        rc, info = cc.cclr_solve_damped(ctx, cc.CCLR_RIGHT, [0.5] * n, [0.25] * n, r1[:n], r2[:n], s1[:n], s2[:n])
        assert rc == 0, info.as_dict()
        assert torch.allclose(s1[:n], r1[:n] / (0.5 + 0.25j), rtol=0, atol=1e-9) and not bool(s2[:n].any())
    cc.cclr_destroy(ctx)


def test_new_amplitudes_keep_it(lib):
    # the 5 GB that 300 right-hand sides leave are there for the solve after
    # new amplitudes, which may then allocate nothing
    cc, H, (r1, r2), (s1, s2) = lib
    ctx, n = context(cc, H), 300
    taken = []
    for fails in (0, 3):
        cc.cclr_set_amplitudes(ctx, zeros(O, V), zeros(O, O, V, V))
        assert cc.lib().cclr_dbg_fail_allocs(ctx, fails) == 0
        cc.cclr_solve_damped(ctx, cc.CCLR_RIGHT, [0.5] * n, [0.25] * n, r1[:n], r2[:n], s1[:n], s2[:n])
        taken.append(held(cc, ctx))
    cc.cclr_destroy(ctx)
    assert taken[0] > 4 << 30 and taken[1] == taken[0]


def test_two_threads(lib):
    # one thread's allocations keep finding no room while the other's transforms run
    cc, H = lib[:2]
    ctxs = [context(cc, H) for _ in range(2)]
    errors = []

    def work(k):
        try:
            r1, r2 = torch.ones((100, O, V), dtype=torch.complex128, device="cuda"), zeros(100, O, O, V, V)
            s1, s2 = torch.empty_like(r1), torch.empty_like(r2)
            for i in range(20):
                if k:
                    cc.cclr_destroy(ctxs[1])
                    ctxs[1] = context(cc, H)
                    assert cc.lib().cclr_dbg_fail_allocs(ctxs[1], 2) == 0
                cc.cclr_jacobian_right(ctxs[k], [0.5] * 100, [0.25] * 100, r1, r2, s1, s2)
                assert bool((s1 == -(0.5 + 0.25j)).all()) and not bool(s2.any())
        except BaseException as e:  # noqa: BLE001 (reported by the main thread)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for c in ctxs:
        cc.cclr_destroy(c)
    assert not errors, errors
