"""The orthonormalised test vectors at every number of them (whole and partial groups
of four), aggregates of 16 to 256 sites, FP64 and FP32 working vectors, and nearly
dependent vectors: Q^H Q = 1, Q^H T upper triangular with a positive diagonal,
T = Q Q^H T.  Sums of K = 6 Bv products over n vectors, u = 2^-53: bar n K u (relative
to the vectors' norms).  Dependent vectors are refused with their aggregate."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BLOCKS = {16: ((4, 4, 4, 4), (2, 2, 2, 2)), 32: ((8, 4, 4, 8), (2, 2, 2, 4)), 128: ((8, 8, 4, 8), (4, 4, 2, 4)),
          256: ((8, 8, 8, 8), (4, 4, 4, 4))}


@pytest.fixture(scope="module")
def ctx():
    from paper_1811_00355_amd import Context
    c = Context(0)
    yield c
    c.close()


def _mg(ctx, bv, n, inner, store, near=(), dep=()):
    from paper_1811_00355_amd import Gauge, MG, default_params
    from oracle.lattice import Lattice
    from workloads import gauss_vectors, su3_field
    L, blk = BLOCKS[bv]
    lat = Lattice(L, blk)
    tv = gauss_vectors(n, lat.V, 5).reshape(n, lat.V, 4, 3)
    for i, j, eps in near:   # vector i: vector j and a small part of its own
        tv[i] = tv[j] + eps * tv[i]
    for i, j, k in dep:
        tv[i] = tv[j] - 0.5j * tv[k]
    if inner:
        tv = tv.astype(np.complex64).astype(np.complex128)
    g = Gauge(ctx, L, blk, su3_field(L, 0.2, 9), -0.1, 1.0)
    print(f"Gram-Schmidt Bv={bv} n={n} inner={inner} store={store} near={near} dep={dep}", flush=True)
    try:
        mg = MG(g, default_params(block=blk, n_vec=n, inner_dtype=inner, store_dtype=store, init_sap_apps=0,
                                  setup_iters=0), tv_host=tv)
    except Exception:
        g.destroy()
        raise
    return lat, tv, g, mg


@pytest.mark.parametrize("bv,n,inner,store,near", [
    (16, 6, 0, 0, ()), (32, 8, 0, 0, ()), (128, 12, 1, 3, ()), (256, 16, 1, 2, ()), (256, 20, 1, 1, ()),
    (256, 24, 0, 0, ()), (16, 12, 0, 0, ((1, 0, 1e-9), (4, 1, 1e-6), (11, 7, 1e-10))),
    (256, 24, 0, 0, ((3, 2, 1e-10), (9, 0, 1e-10), (23, 12, 1e-8)))])
def test_orthonormal_and_triangular(ctx, bv, n, inner, store, near):
    from oracle import amg
    lat, tv, g, mg = _mg(ctx, bv, n, inner, store, near)
    Q = np.moveaxis(amg.to_aggregates(lat, mg.export_vectors()), 0, 2)   # [Vc][2][n][K]
    T = np.moveaxis(amg.to_aggregates(lat, tv), 0, 2)
    bar = n * 6 * lat.Bv * 2.0 ** -53
    gram = np.conj(Q) @ np.swapaxes(Q, -1, -2)
    R = np.conj(Q) @ np.swapaxes(T, -1, -2)              # [n of Q][n of T]
    nT = np.linalg.norm(T, axis=-1)
    low = np.abs(np.tril(R, -1)) / nT[..., None, :]
    dg = np.diagonal(R, axis1=-2, axis2=-1)
    back = np.swapaxes(T, -1, -2) - np.swapaxes(Q, -1, -2) @ R
    errs = [np.abs(gram - np.eye(n)).max(), low.max(), (np.abs(dg.imag) / nT).max(),
            (np.linalg.norm(back, axis=-2) / nT).max()]
    print("  " + " ".join(f"{e:.2e}" for e in errs) + f" bar {bar:.2e}", flush=True)
    assert max(errs) < bar
    assert np.all(dg.real > 0)
    mg.destroy()
    g.destroy()


@pytest.mark.parametrize("bv,n,dep", [(16, 6, (1, 0, 0)), (256, 20, (3, 1, 0)), (256, 24, (22, 1, 9))])
def test_dependent_vectors_are_refused(ctx, bv, n, dep):
    with pytest.raises(Exception, match="rank deficient"):
        _mg(ctx, bv, n, 0, 0, dep=(dep,))
