"""The coarse apply against R D P through the library's own transfer and operator
entry points, at every block size, both splits of the kernel (stencil blocks
within and beyond the last-level cache) and around the 16 right-hand sides of a
pass.  Bars: FP64 1e-12; FP32 blocks and vectors 1e-5, the repository's bars for
the coarse apply (a few hundred FP32 products per entry, relative to the largest)."""
import pytest

pytestmark = pytest.mark.gpu

SMALL = [((8, 8, 8, 8), n, store, nrhs) for n in (6, 8, 12, 16, 20, 24) for store, nrhs in ((0, 17), (1, 1), (1, 16), (1, 17))]
LARGE = [((24, 24, 24, 48), 24, 1, 3), ((24, 24, 24, 48), 20, 1, 17), ((24, 24, 24, 32), 24, 0, 2)]


@pytest.fixture(scope="module")
def ctx():
    from paper_1811_00355_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("L,n,store,nrhs", SMALL + LARGE)
def test_coarse_apply_is_r_d_p(ctx, L, n, store, nrhs):
    import numpy as np
    import torch
    from paper_1811_00355_amd import Gauge, MG, default_params
    from workloads import su3_random
    blk = (4, 4, 4, 4)
    V = int(np.prod(L))
    # links repeat a short random stretch: the identity holds for any links
    U = np.resize(su3_random(4096 * 4 + 12, 0.3, 7), (V * 4, 3, 3)).reshape(V, 4, 3, 3)
    g = Gauge(ctx, L, blk, U, -0.1, 1.0)
    vt = 0 if store == 0 else 1
    mg = MG(g, default_params(block=blk, n_vec=n, setup_iters=0, init_sap_apps=1, inner_dtype=vt, store_dtype=store))
    ct = torch.complex128 if vt == 0 else torch.complex64
    gen = torch.Generator(device="cuda").manual_seed(n * 100 + nrhs)
    x = torch.randn((nrhs, g.Vc, 2 * n), generator=gen, device="cuda", dtype=ct)
    y = torch.empty_like(x)
    ref = torch.empty_like(x)
    print(f"coarse apply L={L} n={n} store={store} nrhs={nrhs}", flush=True)
    mg.dd_coarse_apply(vt, nrhs, x, y)
    f = torch.empty((nrhs, 12, V), device="cuda", dtype=ct)
    h = torch.empty_like(f)
    mg.dd_prolong(vt, nrhs, x, f)
    g.dd_dirac_apply(vt, nrhs, f, h)
    mg.dd_restrict(vt, nrhs, h, ref)
    torch.cuda.synchronize()
    err = float((y - ref).abs().max() / ref.abs().max())
    print(f"  error against R D P {err:.2e}", flush=True)
    assert err < (1e-12 if vt == 0 else 1e-5)
    mg.destroy()
    g.destroy()
