"""The coarse GMRES step at the edges of its forms: restart lengths of one and two,
the last step of a cycle, cycles of 64 (the reductions ride on the step's other
launches) and 65 (launches of their own), one and two Gram-Schmidt passes, a zero
right-hand side beside ordinary ones.  Against the oracle with a fixed iteration
count in FP64: 1e-10 of the largest entry, the repository's bar for this solve."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1811_00355_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("name,iters,restart,passes", [
    ("c1", 1, 1, 1), ("c1", 5, 1, 1), ("asym", 7, 2, 1), ("asym", 6, 3, 1), ("b4", 9, 9, 1), ("b4", 9, 4, 2),
    ("b4", 66, 64, 1), ("b4", 67, 65, 1)])
def test_coarse_gmres_step(ctx, name, iters, restart, passes):
    import _gpu
    from test_gpu_mg import _build, _close, _coarse_roundtrip
    from oracle import amg
    from workloads import gauss_vectors
    kw = dict(coarse_fixed_iters=iters, coarse_restart=restart, coarse_cgs_passes=passes)
    d = _build(ctx, name, **kw)
    lat, mg, n = d["lat"], d["mg"], d["n"]
    Pb = amg.gram_schmidt(lat, d["tv0"])
    ceo = amg.CoarseEO(lat, amg.coarse_operator(d["W"], Pb))
    b = gauss_vectors(3, lat.Vc, 43, ncomp=2 * n)
    b[1] = 0
    got = _coarse_roundtrip(mg, 0, 3, b, lambda i, o: mg.dd_coarse_solve(0, 3, i, o))
    assert np.all(got[1] == 0)
    for r in (0, 2):
        err = _gpu.max_rel(got[r], ceo.solve(b[r], amg.MGParams(n_vec=n, **kw)))
        print(f"  rhs {r}: {err:.2e}", flush=True)
        assert err < 1e-10
    _close(d)
