"""D apply with the face halos in LDS (lattices of more than 256 blocks) against the
oracle: FP64 and FP32 operands, one and several right-hand sides, extents of two
blocks (both faces of a direction belong to the same block) and more.  Bars as for
the other applies: FP64 1e-12, FP32 1e-5 against the oracle on FP32 operands.  A
right-hand side has the same bits alone and in a batch, with and without halos."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("L,nrhs", [((8, 16, 16, 40), 1), ((8, 16, 24, 24), 2)])
def test_dirac_with_faces_staged(L, nrhs, dtype):
    import numpy as np
    import _gpu
    from oracle.dirac import WilsonClover
    from oracle.lattice import Lattice
    from paper_1811_00355_amd import Context, Gauge
    from workloads import su3_field, gauss_spinor
    blk, m0, csw = (4, 4, 4, 4), -0.1, 1.2
    assert np.prod(L) // 256 > 256
    U = su3_field(L, 0.25, 3)
    lat = Lattice(L, blk)
    ctx = Context(0)
    g = Gauge(ctx, L, blk, U, m0, csw)
    psi = gauss_spinor(L, nrhs, 8)
    if dtype == 1:
        psi = _gpu.round_f32(psi)
        a, _ = g.export_clover()
        W = WilsonClover(_gpu.round_f32(U), lat, m0, csw, A=_gpu.stored_clover_dense(a, 1))
    else:
        W = WilsonClover(U, lat, m0, csw)
    print(f"D apply L={L} nrhs={nrhs} dtype={dtype}", flush=True)
    out = _gpu.fine_apply(g, dtype, nrhs, psi, lambda i, o: g.dd_dirac_apply(dtype, nrhs, i, o))
    for r in {0, nrhs - 1}:
        err = _gpu.max_rel(out[r], W.apply(psi[r]))
        print(f"  rhs {r}: error {err:.2e}", flush=True)
        assert err < (1e-12 if dtype == 0 else 1e-5)
    g.destroy()
    ctx.close()


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("L", [(8, 8, 8, 16), (8, 16, 16, 40)])
def test_alone_and_in_a_batch_same_bits(L, dtype):
    import torch
    from paper_1811_00355_amd import Context, Gauge
    from workloads import su3_field
    import numpy as np
    ctx = Context(0)
    g = Gauge(ctx, L, (4, 4, 4, 4), su3_field(L, 0.25, 3), -0.1, 1.0)
    n, V = 12, int(np.prod(L))
    gen = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randn((n, 12, V), generator=gen, device="cuda", dtype=torch.complex128 if dtype == 0 else torch.complex64)
    both = torch.empty_like(x)
    g.dd_dirac_apply(dtype, n, x, both)
    one = torch.empty_like(x[:1])
    for r in (0, 7, 11):
        g.dd_dirac_apply(dtype, 1, x[r].contiguous(), one)
        torch.cuda.synchronize()
        assert torch.equal(one[0], both[r])
    g.destroy()
    ctx.close()
