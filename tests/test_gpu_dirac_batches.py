"""Half-precision D apply with several right-hand sides: blocks beyond whole rounds of
the chip are split over the right-hand sides.  Few blocks (every right-hand side by
itself), none left over, and remainders split in one, two and three; every
right-hand side the same bits in every batch of two or more, and within 1e-5 of the
largest entry (the repository's bar for FP32 arithmetic) of its apply alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1811_00355_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dtype", [2, 3])
@pytest.mark.parametrize("L,batches", [((8, 8, 8, 8), (2, 3, 13)), ((8, 8, 8, 24), (2, 7)), ((16, 16, 16, 32), (2, 3)),
                                       ((24, 24, 24, 24), (2, 5, 12)), ((16, 16, 24, 32), (2, 3, 12))])
def test_every_batch_same_bits(ctx, dtype, L, batches):
    import torch
    from paper_1811_00355_amd import Gauge
    from workloads import su3_random
    V = int(np.prod(L))
    g = Gauge(ctx, L, (4, 4, 4, 4), np.resize(su3_random(4096 * 4 + 12, 0.3, 7), (V * 4, 3, 3)).reshape(V, 4, 3, 3),
              -0.1, 1.0)
    gen = torch.Generator(device="cuda").manual_seed(dtype)
    x = torch.randn((max(batches), 12, V), generator=gen, device="cuda", dtype=torch.complex64)

    def apply(v):
        y = torch.full_like(v, float("nan"))
        g.dd_dirac_apply(dtype, v.shape[0], v, y)
        torch.cuda.synchronize()
        return y

    alone = torch.cat([apply(x[r:r + 1].contiguous()) for r in range(max(batches))])
    for n in batches:
        y = apply(x[:n].contiguous())
        err = float((y - alone[:n]).abs().max() / alone.abs().max())
        print(f"L={L} dtype={dtype} nrhs={n}: against one by one {err:.1e}", flush=True)
        assert err < 1e-5
        for r in range(0, n - 1, 3):
            assert torch.equal(apply(x[r:r + 2].contiguous()), y[r:r + 2])
    g.destroy()
