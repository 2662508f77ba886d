"""D apply on blocks of 256 sites whose edges are not all four, on lattices of more than
256 blocks (where 4^4 blocks stage their faces in LDS), against the oracle: FP64 and
FP32 operands, one and two right-hand sides, extents of two blocks and more.  Bars as
for the other applies: FP64 1e-12, FP32 1e-5 against the oracle on FP32 operands.  A
solve with an FP32 preconditioner on such blocks (its outer operator reads FP32
vectors) ends with the residual that it reports: the two differ by the rounding of
one FP64 apply, about 1e-15 |D| |x| / |b| < 1e-12."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FIELDS = [((8, 4, 4, 2), (16, 16, 16, 20)), ((2, 4, 4, 8), (8, 16, 16, 48)), ((4, 4, 8, 2), (8, 16, 16, 40))]


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("blk,L", FIELDS)
def test_dirac_on_other_blocks_of_256_sites(blk, L, dtype):
    import _gpu
    from oracle.dirac import WilsonClover
    from oracle.lattice import Lattice
    from paper_1811_00355_amd import Context, Gauge
    from workloads import su3_field, gauss_spinor
    assert np.prod(blk) == 256 and np.prod(L) // 256 > 256
    U, m0, csw = su3_field(L, 0.25, 3), -0.1, 1.2
    ctx = Context(0)
    g = Gauge(ctx, L, blk, U, m0, csw)
    psi = gauss_spinor(L, 2, 8)
    lat = Lattice(L, blk)
    if dtype == 1:
        psi = _gpu.round_f32(psi)
        W = WilsonClover(_gpu.round_f32(U), lat, m0, csw, A=_gpu.stored_clover_dense(g.export_clover()[0], 1))
    else:
        W = WilsonClover(U, lat, m0, csw)
    ref = [W.apply(psi[r]) for r in range(2)]
    for nrhs in (1, 2):
        print(f"D apply block={blk} L={L} nrhs={nrhs} dtype={dtype}", flush=True)
        out = _gpu.fine_apply(g, dtype, nrhs, psi[:nrhs], lambda i, o: g.dd_dirac_apply(dtype, nrhs, i, o))
        for r in range(nrhs):
            err = _gpu.max_rel(out[r], ref[r])
            print(f"  rhs {r}: error {err:.2e}", flush=True)
            assert err < (1e-12 if dtype == 0 else 1e-5)
    g.destroy()
    ctx.close()


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("L", [(16, 16, 16, 64), (16, 16, 16, 72)])
def test_batches_around_the_face_rules_same_bits(L, dtype):
    """4^4 blocks, 1024 and 1152 of them: in FP64 one to four right-hand sides read the faces ahead, five do so on the larger
    lattice only; every form the same bits."""
    import torch
    from paper_1811_00355_amd import Context, Gauge
    from workloads import su3_random
    V = int(np.prod(L))
    ctx = Context(0)
    g = Gauge(ctx, L, (4, 4, 4, 4), np.resize(su3_random(4096 * 4 + 12, 0.3, 7), (V * 4, 3, 3)).reshape(V, 4, 3, 3), -0.1, 1.0)
    gen = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randn((5, 12, V), generator=gen, device="cuda", dtype=torch.complex128 if dtype == 0 else torch.complex64)
    out = []
    for n in (5, 4, 2, 1):
        print(f"D apply L={L} dtype={dtype} nrhs={n}", flush=True)
        y = torch.empty_like(x[:n])
        g.dd_dirac_apply(dtype, n, x[:n].contiguous(), y)
        torch.cuda.synchronize()
        out.append(y)
        assert torch.equal(y, out[0][:n])
    g.destroy()
    ctx.close()


@pytest.mark.parametrize("dtype", [2, 3])
def test_half_operands_alone_and_in_a_batch_same_bits(dtype):
    """One right-hand side takes the form of the other operand types, several the one that keeps the operator in registers."""
    import torch
    from paper_1811_00355_amd import Context, Gauge
    from workloads import su3_field
    L, n = (8, 8, 8, 16), 5
    ctx = Context(0)
    g = Gauge(ctx, L, (4, 4, 4, 4), su3_field(L, 0.3, 11), -0.1, 1.0)
    gen = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn((n, 12, int(np.prod(L))), generator=gen, device="cuda", dtype=torch.complex64)
    y, one = torch.empty_like(x), torch.empty_like(x[:1])
    g.dd_dirac_apply(dtype, n, x, y)
    for r in range(n):
        g.dd_dirac_apply(dtype, 1, x[r:r + 1].contiguous(), one)
        torch.cuda.synchronize()
        assert torch.equal(one[0], y[r])
    g.destroy()
    ctx.close()


def test_solve_alone_and_in_a_batch_same_bits_on_384_blocks():
    """The outer operator (FP64 on FP32 spinors, and FP64 on FP64 at the restarts) takes other face forms for one to four
    right-hand sides than for six: the solutions are the same bits."""
    import torch
    from paper_1811_00355_amd import Context, Gauge, MG, default_params
    from workloads import su3_random
    L = (16, 16, 16, 24)
    V = int(np.prod(L))
    ctx = Context(0)
    g = Gauge(ctx, L, (4, 4, 4, 4), np.resize(su3_random(4096 * 4 + 12, 0.2, 7), (V * 4, 3, 3)).reshape(V, 4, 3, 3), -0.1, 1.0)
    mg = MG(g, default_params(block=(4, 4, 4, 4), n_vec=8, setup_iters=1, inner_dtype=1, store_dtype=3, seed=5))
    gen = torch.Generator(device="cuda").manual_seed(9)
    b = torch.randn((6, V * 12), generator=gen, device="cuda", dtype=torch.complex128)
    out = []
    for n in (6, 3, 1):
        print(f"solve L={L} nrhs={n}", flush=True)
        x = torch.zeros_like(b[:n])
        info, _ = mg.dd_solve(n, b[:n].contiguous(), x, 1e-8)
        torch.cuda.synchronize()
        assert all(i["converged"] for i in info[:n])
        out.append(x)
        assert torch.equal(x, out[0][:n])
    mg.destroy()
    g.destroy()
    ctx.close()


def test_solve_on_other_blocks_of_256_sites():
    import torch
    import _gpu
    from oracle.dirac import WilsonClover
    from oracle.lattice import Lattice
    from paper_1811_00355_amd import Context, Gauge, MG, default_params
    from workloads import su3_field, gauss_spinor
    blk, L = FIELDS[0]
    U, m0, csw, nrhs = su3_field(L, 0.2, 23), -0.1, 1.0, 2
    ctx = Context(0)
    g = Gauge(ctx, L, blk, U, m0, csw)
    p = default_params(block=blk, n_vec=8, setup_iters=1, inner_dtype=1, store_dtype=1, seed=5)
    print(f"setup and solve block={blk} L={L}", flush=True)
    mg = MG(g, p)
    b = gauss_spinor(L, nrhs, 65)
    bd = _gpu.to_dev(b.reshape(nrhs, -1))
    x = torch.zeros_like(bd)
    info, _ = mg.dd_solve(nrhs, bd, x, 1e-10)
    torch.cuda.synchronize()
    W = WilsonClover(U, Lattice(L, blk), m0, csw)
    xs = _gpu.to_host(x).reshape(b.shape)
    for r in range(nrhs):
        res = np.linalg.norm(b[r] - W.apply(xs[r])) / np.linalg.norm(b[r])
        print(f"  rhs {r}: residual {res:.3e}, reported {info[r]['true_relres']:.3e}", flush=True)
        assert info[r]["converged"] and info[r]["true_relres"] <= 1e-10
        assert abs(res - info[r]["true_relres"]) < 1e-12
    mg.destroy()
    g.destroy()
    ctx.close()
