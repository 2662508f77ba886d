"""The stored clover inverse where the elimination has to exchange rows (m0 = -3.5:
off-diagonal entries of the clover term exceed the diagonal) and where there is no
clover term.  Bar on the entries: the first-order forward bound of Gauss-Jordan
elimination with partial pivoting, n^3 u cond(A) max|A^-1| with n = 6, u = 2^-53."""
import numpy as np
import pytest

L, BLK, SEED = (8, 4, 4, 8), (2, 2, 2, 4), 5
CASES = [(-3.5, 1.0), (-3.9, 2.0), (-0.3, 0.0)]


def _blocks(m0, c_sw):
    from oracle.dirac import clover_matrix, chiral_blocks
    from oracle.lattice import Lattice
    from workloads import su3_field
    U = su3_field(L, 0.3, SEED)
    return U, chiral_blocks(clover_matrix(U, Lattice(L, BLK), m0, c_sw))


def test_cases_need_row_exchanges():
    for m0, c_sw in CASES[:2]:
        _, a = _blocks(m0, c_sw)
        first = np.abs(a[..., :, 0])
        assert np.mean(np.argmax(first, axis=-1) != 0) > 0.01


@pytest.mark.gpu
@pytest.mark.parametrize("m0,c_sw", CASES)
def test_inverse_of_every_block(m0, c_sw):
    from oracle.dirac import unpack_hermitian6
    from paper_1811_00355_amd import Context, Gauge
    U, a = _blocks(m0, c_sw)
    ctx = Context(0)
    g = Gauge(ctx, L, BLK, U, m0, c_sw)
    got, inv = (unpack_hermitian6(p) for p in g.export_clover())
    assert np.abs(got - a).max() <= 1e-13
    ref = np.linalg.inv(got)
    bound = 216 * 2.0 ** -53 * np.linalg.cond(got) * np.abs(ref).max(axis=(-1, -2))
    err = np.abs(inv - ref).max(axis=(-1, -2))
    print(f"m0={m0} c_sw={c_sw}: worst error / bound {np.max(err / bound):.2e}", flush=True)
    assert np.all(err <= bound)
    g.destroy()
    ctx.close()
