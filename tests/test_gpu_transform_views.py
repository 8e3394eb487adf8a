"""Both transforms at the edges of the 32 x 32 virtual tiles in which the
vectors are unpacked and the result is packed, and at the smallest sizes,
against the oracle with the suite's parity bar."""
import numpy as np
import pytest
import torch

from helpers import assert_blocks, small_problem, vec
from oracle import cclr_ref as O

pytestmark = pytest.mark.gpu
TOL = 1e-10


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).to(torch.complex128).cuda()


@pytest.mark.parametrize("o,v,nvec", [(2, 2, 1), (2, 3, 3), (3, 31, 2), (3, 32, 1), (2, 33, 2), (2, 65, 1)])
def test_transforms_at_tile_edges(o, v, nvec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_14296_amd as cc
    from gen import synth as s
    pb, _, f, H, t1, t2 = small_problem(o, v)
    ref = O.CCLR(H, t1, t2)
    ctx = cc.cclr_create(o, v)
    try:
        cc.cclr_set_hamiltonian(ctx, dev(H.f), *[dev(H.blocks[k]) for k in s.CANONICAL_BLOCKS])
        cc.cclr_set_amplitudes(ctx, dev(t1), dev(t2))
        xs, zs = [vec(pb, k) for k in range(nvec)], [0.1 + 0.005j, -0.2 + 0.3j, 0.0j][:nvec]
        r1, r2 = dev(np.stack([x[0] for x in xs])), dev(np.stack([x[1] for x in xs]))
        for fn, side in ((cc.cclr_jacobian_right, ref.right), (cc.cclr_jacobian_left, ref.left)):
            s1, s2 = torch.full_like(r1, 7.0), torch.full_like(r2, 7.0)
            fn(ctx, [z.real for z in zs], [z.imag for z in zs], r1, r2, s1, s2)
            for k in range(nvec):
                assert_blocks((s1.cpu().numpy()[k], s2.cpu().numpy()[k]), side(*xs[k], zs[k]), TOL,
                              f"{side.__name__} o={o} v={v} vector {k}")
    finally:
        cc.cclr_destroy(ctx)
