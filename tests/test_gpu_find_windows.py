"""A window of many bins is scanned together with those of its seed's other
candidates; a narrower one by the owner's queue.  The bin grid alone decides
which of the two a window takes, and no result may depend on it: every hit is
tested against the window itself, and equal children rank by their hit's index.
So the same events on a grid of 64 bins a layer (never the first) and on grids
of 4096 and 16384 (low-pT seeds' windows: the whole circle) must agree in every
bit, for every number of candidates kept."""
import numpy as np
import pytest

import eventgen as E

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_cands,width,prec", [(1, 256, "MIXED"), (2, 64, "MIXED"), (3, 256, "FP32"),
                                                  (5, 128, "MIXED"), (6, 256, "MIXED"), (6, 32, "MIXED"),
                                                  (7, 64, "FP32"), (8, 256, "MIXED"), (8, 32, "FP32")])
@pytest.mark.parametrize("disks", [False, True])
def test_results_do_not_depend_on_the_bin_grid(max_cands, width, prec, disks):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1906_02253_amd as K
    from paper_1906_02253_amd import pipeline
    rng = np.random.default_rng(71)
    geom = E.geometry.barrel10_disks14() if disks else E.geometry.barrel10(x0=0.02)
    evs = [E.make_event(rng, geom, 13, E.pt_uniform(0.5, 0.6), 0.4, 40_000),
           E.make_event(rng, geom, 60, E.pt_power2(0.4, 5.0), 2.0, 5_000)]
    inp = E.find_inputs(evs)
    assert inp["seed_hits"].shape[0] >= 50
    ref = None
    for nphi, n2 in ((8, 8), (128, 32), (512, 32)):
        grid = [dict(L, nbin_phi=nphi, nbin_2=n2) for L in geom]
        ctx = K.Context(grid, max_cands=max_cands)
        ctx.set_find_config(width, True)
        fp = pipeline.FindProblem(ctx, inp, prec=getattr(K, "PREC_" + prec))
        fp.run(getattr(K, "PREC_" + prec))
        torch.cuda.synchronize()
        r = fp.results()
        ref = r if ref is None else ref
        for k in ("hits", "par", "cov", "chi2", "ndf", "status"):
            assert np.array_equal(r[k], ref[k], equal_nan=r[k].dtype.kind == "f"), (nphi, n2, k)
    assert (ref["hits"] >= 0).sum(1).max() >= 8
