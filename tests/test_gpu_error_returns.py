"""Calls that fail after work has been queued: they return only when the stream
has finished with the caller's arrays.  And a rejected input of one context
means nothing to the next, also while the null stream is busy."""
import numpy as np
import pytest
import torch

from helpers import config_problem, vec

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).to(torch.complex128).cuda()


@pytest.fixture(scope="module")
def setup():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_14296_amd as cc
    from gen import synth as s
    pb, _, H, t1, t2 = config_problem(4, 16, 2)
    ctx = cc.cclr_create(4, 16)
    blocks = [dev(H.f)] + [dev(H.blocks[k]) for k in s.CANONICAL_BLOCKS]
    cc.cclr_set_hamiltonian(ctx, *blocks)
    cc.cclr_set_amplitudes(ctx, dev(t1), dev(t2))
    yield cc, ctx, pb, blocks
    cc.cclr_destroy(ctx)


def busy():
    """About a tenth of a second of earlier work on the stream the context uses."""
    torch.cuda.synchronize()
    torch.cuda._sleep(10 ** 7)
    assert not torch.cuda.current_stream().query()


def drained():
    return torch.cuda.current_stream().query()


def test_missing_output_array(setup):
    cc, ctx, pb, _ = setup
    L = cc.lib()
    r1, r2 = (dev(x[None]) for x in vec(pb, 0))
    s1 = torch.full_like(r1, 3.0)
    z = cc._dbl([0.1])
    for fn in (L.cclr_jacobian_right, L.cclr_jacobian_left):
        busy()
        assert fn(ctx, 1, z, z, r1.data_ptr(), r2.data_ptr(), s1.data_ptr(), None) == cc.CCLR_EINVAL
        assert drained()
    assert bool((s1 == 3.0).all())


def test_missing_integral_block(setup):
    cc, ctx, pb, blocks = setup
    ptrs = [x.data_ptr() for x in blocks]
    busy()
    assert cc.lib().cclr_set_hamiltonian(ctx, *ptrs[:-1], None) == cc.CCLR_EINVAL
    assert drained()
    cc.cclr_set_hamiltonian(ctx, *blocks)


def test_marks_of_a_destroyed_context(setup):
    cc, _, _, blocks = setup
    stream = torch.cuda.Stream()
    bad = [blocks[0].clone()] + blocks[1:]
    bad[0][0, 0] = float("nan")
    for _ in range(3):
        old = cc.cclr_create(4, 16, stream=stream)
        with pytest.raises(cc.CclrError):
            cc.cclr_set_hamiltonian(old, *bad)
        cc.cclr_destroy(old)
        busy()
        ctx = cc.cclr_create(4, 16, stream=stream)  # its marks may lie where the old ones did
        try:
            cc.cclr_set_hamiltonian(ctx, *blocks)
        finally:
            cc.cclr_destroy(ctx)
