"""dd_footprint_bytes: the scratch of a setup counts the Galerkin build's scratch vectors only
where the build takes them (blocks other than 4^4); the figures suffice as a budget."""
import os

import pytest

from paper_1811_00355_amd import binding as B

BLOCKS = [((4, 4, 4, 4), (8, 8, 8, 16)), ((4, 4, 4, 2), (8, 8, 8, 8))]


def _scratch(L, blk, store, n=20):
    inner = B.DD_F64 if store == B.DD_F64 else B.DD_F32
    p = B.default_params(block=blk, n_vec=n, inner_dtype=inner, store_dtype=store)
    return B.footprint(L, blk, p, 1)


@pytest.mark.skipif(not os.path.exists(B.LIB_PATH), reason="libdd.so not built")
@pytest.mark.parametrize("store", [0, 1, 2, 3])
def test_scratch_is_what_the_build_takes(store):
    L, n = (32, 32, 32, 64), 20
    V, pair = 32 ** 3 * 64, 16 if store == 0 else 8
    vectors = 2 * 12 * V * n * pair              # the V-cycle's fine vectors for the n test vectors
    direct = _scratch(L, (4, 4, 4, 4), store)["scratch"]
    assert vectors < direct < 1.5 * vectors
    # 4 GiB hold 10 of the FP64 fine vectors
    Vc2 = V // 128
    other = _scratch(L, (4, 4, 4, 2), store)["scratch"]
    coarse = (8 if store else 16) * Vc2 * 2 * n * n * 70
    assert vectors + 10 * 12 * V * 16 < other < vectors + coarse + 10 * 12 * V * 16 + (1 << 30)


@pytest.mark.gpu
@pytest.mark.parametrize("blk,L", BLOCKS)
@pytest.mark.parametrize("store", [0, 1, 3])
def test_setup_runs_within_the_figures(blk, L, store):
    from paper_1811_00355_amd import Context, Gauge, MG
    from workloads import su3_field
    fp = _scratch(L, blk, store)
    ctx = Context(0, hbm_budget_bytes=fp["gauge"] + fp["setup"] + fp["scratch"])
    g = Gauge(ctx, L, blk, su3_field(L, 0.2, 6201), -0.15, 1.0)
    inner = B.DD_F64 if store == B.DD_F64 else B.DD_F32
    print(f"setup block={blk} store={store}: {fp}", flush=True)
    mg = MG(g, B.default_params(block=blk, n_vec=20, setup_iters=1, inner_dtype=inner, store_dtype=store, seed=7))
    assert ctx.bytes_in_use() == fp["gauge"] + fp["setup"]
    mg.dd_setup_update_mass(-0.1)
    mg.destroy()
    g.destroy()
    assert ctx.bytes_in_use() == 0
    ctx.close()
