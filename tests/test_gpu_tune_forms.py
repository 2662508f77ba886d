"""The autotuner times only choices that a launch of the setup reads: the others keep the
caller's values (they were picked by noise between runs of one kernel) and have no line
in the report."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blk,store,half,timed", [
    ((4, 4, 4, 4), 1, 0, dict(sap_wpe=2, sap_dom_rhs=2)),          # one FP32 domain form, once launched and once persistent
    ((4, 4, 4, 4), 3, 0, dict(sap_wpe=2, sap_dom_rhs=3)),
    ((4, 4, 4, 4), 3, 1, dict(sap_wpe=2, sap_dom_rhs=3, coarse_spw=3)),
    ((2, 2, 2, 2), 1, 0, dict(dirac_threads=3)),                   # small domains have one form of their own
    ((2, 2, 2, 2), 2, 1, dict(dirac_threads=3, coarse_spw=3))])
def test_only_choices_that_are_read(blk, store, half, timed):
    from paper_1811_00355_amd import Context, Gauge, MG, default_params
    from workloads import su3_field
    L = (8, 8, 8, 8)
    ctx = Context(0)
    g = Gauge(ctx, L, blk, su3_field(L, 0.2, 23), -0.1, 1.0)
    mg = MG(g, default_params(block=blk, n_vec=8, inner_dtype=1, store_dtype=store, init_sap_apps=1, setup_iters=0))
    before = dict(sap_wpe=3, dirac_threads=128, coarse_spw=8, coarse_half=half, coarse_basis_half=0,
                  coarse_mfma_half=half, sap_dom_rhs=2, sap_persist=0)
    g.dd_gauge_set_tuning(**before)
    rep = mg.dd_autotune(2)
    print(rep, flush=True)
    lines = [l for l in rep.splitlines() if " ms" in l]
    for k in ("sap_wpe", "sap_dom_rhs", "dirac_threads", "coarse_spw"):
        n = sum(f" {k}=" in l for l in lines)
        # the persistent form is timed only where a domain form won
        assert n == timed.get(k, 0) or (k == "sap_dom_rhs" and n == timed.get(k, 0) - 1), k
        if k not in timed:
            assert g.dd_gauge_get_tuning()[k] == before[k], k
    mg.destroy()
    g.destroy()
    ctx.close()
