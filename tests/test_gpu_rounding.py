"""Rounding of the FP64 setup arithmetic against 80-bit arithmetic on the same inputs.  A
chain of N products of random sign is 0.4 u sqrt(N / 2) off (u = 2^-53, the partial
sums growing as sqrt(k)), which the bars below follow from the kernels' chains."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
LD = np.clongdouble
L, BLK = (8, 8, 8, 8), (4, 4, 4, 4)
U53 = 2.0 ** -53


def chain(n):
    return 0.4 * U53 * np.sqrt(n / 2)


def norm(z):
    return float(np.sqrt((np.abs(z) ** 2).sum()))


@pytest.fixture(scope="module")
def ctx():
    from paper_1811_00355_amd import Context
    c = Context(0)
    yield c
    c.close()


def setup(ctx, n, inner=0):
    from paper_1811_00355_amd import Gauge, MG, default_params
    from oracle.lattice import Lattice
    from workloads import gauss_vectors, su3_field
    lat = Lattice(L, BLK)
    U = su3_field(L, 0.25, 3)
    g = Gauge(ctx, L, BLK, U, -0.25, 1.0)
    p = default_params(block=BLK, n_vec=n, setup_iters=0, init_sap_apps=2, inner_dtype=inner, store_dtype=inner)
    return lat, U, g, MG(g, p, tv_host=gauss_vectors(n, lat.V, 5).reshape(n, lat.V, 4, 3))


@pytest.mark.parametrize("n,inner", [(8, 0), (20, 0), (20, 1)])
def test_galerkin_operator(ctx, n, inner):
    """Two columns of D_c from the stored P and clover.  Chains of 96 products, the links' products add 1.2 u: 3.3e-16 of
    a block of hops; of the self block as much of each of its parts, which cancel (P is smooth)."""
    import _gpu
    from oracle import amg
    from oracle.dirac import apply_clover, hop_one
    lat, U, g, mg = setup(ctx, n, inner)
    P = mg.export_vectors()
    P = (_gpu.round_f32(P) if inner else P).astype(LD)
    A = _gpu.stored_clover_dense(g.export_clover()[0], 0).astype(LD)
    Pa = np.moveaxis(amg.to_aggregates(lat, P), 0, 2)                     # [Vc][2][n][K]
    bar = float(np.hypot(chain(96), 1.2 * U53))
    dc = mg.export_coarse()
    U = U.astype(LD)
    for t, j in ((0, n - 1), (1, 3)):
        phi = np.zeros_like(P[0])
        phi[:, 2 * t:2 * t + 2] = P[j][:, 2 * t:2 * t + 2]
        parts, face = [apply_clover(A, phi)], []
        for mu in range(4):
            for sign, keep in ((+1, lat.inside_fwd[mu]), (-1, lat.inside_bwd[mu])):
                h = hop_one(U, lat, phi, mu, sign)
                parts.append(h * keep[:, None, None])
                face.append(h * ~keep[:, None, None])

        def restrict(f):
            return (Pa.conj() * amg.to_aggregates(lat, f)[:, :, None]).sum(-1).reshape(lat.Vc, 2 * n)

        got = dc[:, :, :, t * n + j]
        parts = [restrict(f) for f in parts]
        e0 = norm(got[:, 0] - sum(parts)) / np.sqrt(sum(norm(f) ** 2 for f in parts))
        refs = [restrict(face[2 * mu + b]) for b in range(2) for mu in range(4)]
        e = max(norm(got[:, 1 + d] - refs[d]) / norm(refs[d]) for d in range(8))
        print(f"D_c n={n} inner={inner} column {t, j}: self {e0:.2e}, hops {e:.2e}, bar {bar:.2e}", flush=True)
        assert max(e0, e) < bar
    mg.destroy()
    g.destroy()


@pytest.mark.parametrize("n", [8, 20])
def test_orthonormality(ctx, n):
    """P^dag P - 1 of every aggregate and chirality, rms per vector: the last normalisation's norm is one within its
    rounding (at most u) and the sums' (a third of u and less), the vectors' own rounding averages out: 1.6 u."""
    from oracle import amg
    lat, _, g, mg = setup(ctx, n)
    Q = np.moveaxis(amg.to_aggregates(lat, mg.export_vectors().astype(LD)), 0, 2)
    dev = (Q.conj()[:, :, :, None] * Q[:, :, None]).sum(-1) - np.eye(n)
    e = norm(dev) / np.sqrt(2.0 * lat.Vc * n)
    print(f"P^dag P - 1, n={n}: {e:.2e} a vector, bar {1.6 * U53:.2e}", flush=True)
    assert e < 1.6 * U53
    mg.destroy()
    g.destroy()


@pytest.mark.parametrize("n", [8, 20])
def test_coarse_apply(ctx, n):
    """The FP64 coarse apply on its own D_c: two chains of 2n products a block, nine blocks added up (0.4 u sqrt(5)), and
    15 % for the spread."""
    import torch
    lat, _, g, mg = setup(ctx, n)
    nc = 2 * n
    D = mg.export_coarse().astype(LD)
    x = np.random.default_rng(3).standard_normal((4, lat.Vc, nc, 2)).view(np.complex128)[..., 0]
    cin = torch.from_numpy(np.ascontiguousarray(x).reshape(4, -1)).cuda()
    pin = torch.empty((4, lat.Vc, nc), dtype=torch.complex128, device="cuda")
    pout, out = torch.empty_like(pin), torch.empty_like(cin)
    mg.pack_coarse(0, 4, cin, pin)
    mg.dd_coarse_apply(0, 4, pin, pout)
    mg.unpack_coarse(0, 4, pout, out)
    torch.cuda.synchronize()
    ref = np.einsum("xij,rxj->rxi", D[:, 0], x.astype(LD))
    for mu in range(4):
        for d, sign in ((1 + mu, +1), (5 + mu, -1)):
            ref = ref + np.einsum("xij,rxj->rxi", D[:, d], x.astype(LD)[:, lat.coarse_neighbor(mu, sign)])
    e = norm(out.cpu().numpy().reshape(ref.shape) - ref) / norm(ref)
    bar = 1.15 * float(np.hypot(chain(nc), chain(10)))
    print(f"coarse apply n={n}: {e:.2e}, bar {bar:.2e}", flush=True)
    assert e < bar
    mg.destroy()
    g.destroy()
