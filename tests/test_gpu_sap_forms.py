"""Every form of the smoother on 4^4 domains gives the same bits: per-RHS layouts,
domain-resident with two or four right-hand sides per workgroup, FP32, FP16 and BF16
operands, batches that fill a group of right-hand sides and that do not; and a
right-hand side has the same bits alone and in a batch where the form depends on
the batch (FP32 operands on more than 512 domains per colour)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1811_00355_amd import Context
    c = Context(0)
    yield c
    c.close()


def _gauge(ctx, L):
    from paper_1811_00355_amd import Gauge
    from workloads import su3_random
    V = int(np.prod(L))
    U = np.resize(su3_random(4096 * 4 + 12, 0.3, 7), (V * 4, 3, 3)).reshape(V, 4, 3, 3)
    return Gauge(ctx, L, (4, 4, 4, 4), U, -0.1, 1.0)


def _smooth(g, dtype, b, x0, sweeps=2, mr=3):
    import torch
    from paper_1811_00355_amd import default_params
    x = x0.clone()
    g.dd_sap_smooth(default_params(block=(4, 4, 4, 4), sap_sweeps=sweeps, sap_mr_iters=mr), dtype, b.shape[0], b, x)
    torch.cuda.synchronize()
    return x


@pytest.mark.parametrize("dtype", [1, 2, 3])
@pytest.mark.parametrize("nrhs", [1, 3, 4, 6])
def test_forms_same_bits(ctx, dtype, nrhs):
    import torch
    L = (8, 8, 16, 8)
    g = _gauge(ctx, L)
    gen = torch.Generator(device="cuda").manual_seed(dtype * 10 + nrhs)
    b, x0 = (torch.randn((nrhs, 12, int(np.prod(L))), generator=gen, device="cuda", dtype=torch.complex64) for _ in "bx")
    ref = None
    for layout in (dict(sap_wpe=2, sap_dom_rhs=0), dict(sap_wpe=3, sap_dom_rhs=0), dict(sap_dom_rhs=2), dict(sap_dom_rhs=4)):
        g.dd_gauge_set_tuning(**dict(g.dd_gauge_get_tuning(), **layout))
        x = _smooth(g, dtype, b, x0)
        ref = x if ref is None else ref
        print(f"dtype {dtype} nrhs {nrhs} {layout}: same bits {torch.equal(x, ref)}", flush=True)
        assert torch.isfinite(torch.view_as_real(x)).all() and torch.equal(x, ref)
    g.destroy()


@pytest.mark.parametrize("L", [(24, 24, 24, 24), (16, 16, 16, 24)])
def test_fp32_alone_and_in_a_batch_same_bits(ctx, L):
    import torch
    g = _gauge(ctx, L)
    gen = torch.Generator(device="cuda").manual_seed(3)
    b, x0 = (torch.randn((3, 12, int(np.prod(L))), generator=gen, device="cuda", dtype=torch.complex64) for _ in "bx")
    both = _smooth(g, 1, b, x0)
    for r in (0, 2):
        print(f"L={L} rhs {r}", flush=True)
        assert torch.equal(_smooth(g, 1, b[r:r + 1].contiguous(), x0[r:r + 1].contiguous())[0], both[r])
    g.destroy()
