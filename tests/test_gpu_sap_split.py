"""The smoother on small domains, a site's work split over the waves of a workgroup:
domains of 16 to 128 sites, every operand type, workgroups filled with right-hand
sides and domains (up to eight pairs) and not.  Against the oracle in FP64, 1e-12 of
the largest entry (the repository's bar for the smoother); every right-hand side the
same bits alone and in a batch, which on the larger lattices packs a workgroup
differently."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1811_00355_amd import Context
    c = Context(0)
    yield c
    c.close()


def _smooth(g, blk, dtype, b, x0, sweeps, mr):
    import torch
    from paper_1811_00355_amd import default_params
    x = x0.clone()
    g.dd_sap_smooth(default_params(block=blk, sap_sweeps=sweeps, sap_mr_iters=mr), dtype, b.shape[0], b, x)
    torch.cuda.synchronize()
    return x


@pytest.mark.parametrize("L,blk,nrhs,bc", [
    ((4, 4, 4, 4), (2, 2, 2, 2), 1, -1), ((4, 8, 4, 4), (2, 2, 2, 2), 9, 1), ((4, 8, 4, 8), (2, 4, 2, 2), 5, -1),
    ((8, 4, 8, 4), (4, 2, 4, 2), 3, -1), ((8, 8, 8, 4), (4, 4, 4, 2), 2, 1)])
def test_against_the_oracle(ctx, L, blk, nrhs, bc):
    import _gpu
    import torch
    from paper_1811_00355_amd import Gauge
    from oracle.lattice import Lattice
    from oracle.dirac import WilsonClover
    from oracle import amg
    from workloads import su3_field, gauss_spinor
    U = su3_field(L, 0.3, 21)
    lat = Lattice(L, blk, bc_t=bc)
    g = Gauge(ctx, L, blk, U, -0.2, 1.2, bc)
    W = WilsonClover(U, lat, -0.2, 1.2)
    b, x0 = gauss_spinor(L, nrhs, 3), gauss_spinor(L, nrhs, 4) * 0.1
    pb, px = g.new_packed(0, nrhs), g.new_packed(0, nrhs)
    g.pack(0, nrhs, _gpu.to_dev(b.reshape(nrhs, -1)), pb)
    g.pack(0, nrhs, _gpu.to_dev(x0.reshape(nrhs, -1)), px)
    got = _smooth(g, blk, 0, pb.reshape(nrhs, -1), px.reshape(nrhs, -1), 3, 4)
    out = torch.zeros((nrhs, lat.V * 12), dtype=torch.complex128, device="cuda")
    g.unpack(0, nrhs, got.reshape(px.shape), out)
    torch.cuda.synchronize()
    got = _gpu.to_host(out).reshape(nrhs, lat.V, 4, 3)
    for r in range(nrhs):
        err = _gpu.max_rel(got[r], amg.sap(W, b[r], x0[r], 3, 4))
        print(f"L={L} block={blk} bc={bc} rhs {r}: {err:.2e}", flush=True)
        assert err < 1e-12
    g.destroy()


@pytest.mark.parametrize("dtype", [0, 1, 2, 3])
@pytest.mark.parametrize("L,blk", [((4, 4, 4, 4), (2, 2, 2, 2)), ((8, 8, 8, 8), (2, 2, 2, 2)), ((16, 16, 16, 8), (2, 2, 2, 2)),
                                   ((16, 8, 16, 16), (2, 2, 2, 4)), ((16, 8, 16, 16), (4, 2, 4, 2)),
                                   ((8, 8, 8, 16), (4, 4, 4, 2))])
def test_alone_and_in_a_batch_same_bits(ctx, dtype, L, blk):
    import torch
    from paper_1811_00355_amd import Gauge
    from workloads import su3_random
    V, nrhs = int(np.prod(L)), 11
    g = Gauge(ctx, L, blk, np.resize(su3_random(4096 * 4 + 12, 0.3, 7), (V * 4, 3, 3)).reshape(V, 4, 3, 3), -0.1, 1.0)
    gen = torch.Generator(device="cuda").manual_seed(dtype)
    ct = torch.complex64 if dtype else torch.complex128
    b, x0 = (torch.randn((nrhs, 12, V), generator=gen, device="cuda", dtype=ct) for _ in "bx")
    print(f"L={L} block={blk} dtype={dtype}", flush=True)
    batch = _smooth(g, blk, dtype, b, x0, 2, 3)
    assert torch.isfinite(torch.view_as_real(batch)).all()
    for r in (0, 7, 10):
        assert torch.equal(_smooth(g, blk, dtype, b[r:r + 1].contiguous(), x0[r:r + 1].contiguous(), 2, 3)[0], batch[r])
    g.destroy()
