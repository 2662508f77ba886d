"""Coarse apply and solve on a stencil beyond the last-level cache with more than 16
right-hand sides (the blocks are then read again, through the caches): a right-hand side
has the same bits as in a batch of at most 16, whose launch streams them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_more_than_sixteen_same_bits():
    import torch
    from paper_1811_00355_amd import Context, Gauge, MG, default_params
    from workloads import su3_random
    L, n, blk = (24, 24, 24, 32), 24, (4, 4, 4, 4)
    V = int(np.prod(L))
    ctx = Context(0)
    g = Gauge(ctx, L, blk, np.resize(su3_random(4096 * 4 + 12, 0.3, 7), (V * 4, 3, 3)).reshape(V, 4, 3, 3), -0.1, 1.0)
    assert 9 * g.Vc * (2 * n) ** 2 * 8 > 256e6
    mg = MG(g, default_params(block=blk, n_vec=n, setup_iters=0, init_sap_apps=1, inner_dtype=1, store_dtype=1,
                              coarse_fixed_iters=3))
    gen = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn((33, g.Vc, 2 * n), generator=gen, device="cuda", dtype=torch.complex64)
    for call in (mg.dd_coarse_apply, mg.dd_coarse_solve):
        def out(v):
            y = torch.empty_like(v)
            call(1, v.shape[0], v, y)
            torch.cuda.synchronize()
            return y
        few = torch.cat([out(x[:16].contiguous()), out(x[16:32].contiguous()), out(x[32:].contiguous())])
        for nrhs in (17, 33):
            print(f"{call.__name__} nrhs={nrhs}", flush=True)
            assert torch.equal(out(x[:nrhs].contiguous()), few[:nrhs])
    mg.destroy()
    g.destroy()
    ctx.close()
