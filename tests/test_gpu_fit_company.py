"""A fitted track does not depend on the tracks that share its wave: copies of
the same tracks at other places, so that waves of barrels alone, of disks alone
and of both are formed anew, come out the same in every bit."""
import numpy as np
import pytest

import eventgen as E
from tests import common as CM

pytestmark = pytest.mark.gpu
BASE = 300


@pytest.mark.parametrize("prec", ["MIXED", "FP32", "FP64"])
@pytest.mark.parametrize("per_layer", [False, True])
@pytest.mark.parametrize("n", [301, 5000])
def test_a_track_fits_the_same_in_any_company(prec, per_layer, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1906_02253_amd as K
    rng = np.random.default_rng(87)
    geom = E.geometry.barrel10_disks14()
    ev = E.make_event(rng, geom, BASE, E.pt_power2(0.4, 20.0), 2.4, 0)
    flag = getattr(K, "PREC_" + prec)
    hits = K.Hits.from_event(ev)

    def fit(pick):
        ld = CM.ld_of(len(pick))
        up = lambda a: torch.as_tensor(CM.soa_int(np.ascontiguousarray(np.asarray(a)[pick]), ld), device="cuda")
        ctx = K.Context(geom)
        t = K.Tracks(len(pick), ld, flag)
        ctx.seed(hits, up(np.asarray(ev.seq_hit)[:, :3]), t, flag)
        ctx.fit(t, hits, up(ev.seq_layer), up(ev.seq_hit), ev.seq_layer.shape[1],
                flag | (K.PER_LAYER if per_layer else 0))
        torch.cuda.synchronize()
        return t.numpy()

    ref = fit(np.arange(BASE))
    pick = rng.integers(0, BASE, n)
    got = fit(pick)
    for k in ("par", "cov", "chi2", "ndf", "status"):
        assert np.array_equal(got[k], ref[k][pick], equal_nan=True), k
    assert (ref["status"] == 0).sum() > BASE // 2
