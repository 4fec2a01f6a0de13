"""Many small events through the two levels of the binning.  A chunk of 4096
hits keeps its events' boundaries in LDS up to 64 events and its counters up to
2048 segments (an event's layer each); with more, it searches the boundaries
and counts in global memory.  An event's tracks may not depend on which."""
import numpy as np
import pytest

import eventgen as E

pytestmark = pytest.mark.gpu
BASE = 24
KEYS = ("par", "cov", "chi2", "ndf", "status")


def _run(K, geom, inp):
    import torch
    from paper_1906_02253_amd import pipeline
    fp = pipeline.FindProblem(K.Context(geom), inp, prec=K.PREC_MIXED)
    fp.run(K.PREC_MIXED)
    torch.cuda.synchronize()
    return fp.results()


@pytest.mark.parametrize("events,tracks,noise,lo,hi", [
    (3600, 3, 2, 0, 64),           # boundaries and counters in LDS
    (5400, 3, 1, 64, 85),          # counters alone
    (7200, 2, 1, 86, 4096),        # neither
])
def test_events_do_not_depend_on_their_company(events, tracks, noise, lo, hi):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1906_02253_amd as K
    rng = np.random.default_rng(89)
    geom = [dict(L, nbin_phi=16, nbin_2=8) for L in E.geometry.barrel10_disks14()]
    few = E.find_inputs([E.make_event(rng, geom, tracks, E.pt_power2(0.5, 20.0), 1.5, noise) for _ in range(BASE)])
    n, ns, copies = len(few["x"]), len(few["seed_hits"]), events // BASE
    assert ns > BASE // 2 and n * copies > 262_144
    assert lo <= 4096 * BASE / n < hi
    many = {k: np.tile(np.asarray(few[k]), copies) for k in ("x", "y", "z", "su", "sv", "layer")}
    many["event_off"] = np.append((np.arange(copies)[:, None] * n + np.asarray(few["event_off"])[None, :-1]).ravel(),
                                  n * copies)
    shift = np.repeat(np.arange(copies), ns)
    sh = np.tile(np.asarray(few["seed_hits"]), (copies, 1))
    many["seed_hits"] = np.where(sh >= 0, sh + (shift * n)[:, None], -1).astype(np.int32)
    many["seed_layers"] = np.tile(np.asarray(few["seed_layers"]), (copies, 1))
    many["seed_event"] = (np.tile(np.asarray(few["seed_event"]), copies) + shift * BASE).astype(np.int32)
    want, got = _run(K, geom, few), _run(K, geom, many)
    for k in KEYS:
        for c in range(copies):
            assert np.array_equal(got[k][c * ns:(c + 1) * ns], want[k]), (k, c)
    hits = np.where(got["hits"] >= 0, got["hits"] - (shift * n)[:, None], -1).reshape(copies, ns, -1)
    assert (hits == want["hits"][None]).all()
