"""Event offsets that decrease or lie outside the hits.  Every hit still has
one event at most, the one a binary search for its index ends at, so that such
a call finds what the same hits find sorted by that event under rising offsets,
on every run, whether one launch bins them or two levels of counting sort."""
import numpy as np
import pytest

import eventgen as E

pytestmark = pytest.mark.gpu
N_EVENTS = 6


def _event_of(off, i):
    lo, hi = 0, len(off) - 1
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if off[mid] <= i:
            lo = mid
        else:
            hi = mid
    return lo


@pytest.fixture(scope="module")
def events():
    rng = np.random.default_rng(83)
    geom = E.geometry.barrel10(x0=0.02)
    # under 4096 hits in all
    evs = [E.make_event(rng, geom, 14, E.pt_power2(0.5, 50.0), 1.0, 40) for _ in range(N_EVENTS)]
    return geom, E.find_inputs(evs)


def _run(geom, inp):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1906_02253_amd as K
    from paper_1906_02253_amd import pipeline
    fp = pipeline.FindProblem(K.Context(geom), inp, prec=K.PREC_MIXED)
    fp.run(K.PREC_MIXED)
    torch.cuda.synchronize()
    r = fp.results()
    fp.run(K.PREC_MIXED)
    torch.cuda.synchronize()
    again = fp.results()
    for k in ("hits", "par", "cov", "chi2", "ndf", "status"):
        assert np.array_equal(r[k], again[k]), k
    return r


def _offsets(kind, off):
    n, o = int(off[-1]), np.array(off, np.int64)
    if kind == "dip":                        # event 2's range overlaps event 1's
        o[2] = o[1] - (o[1] - o[0]) // 2
    elif kind == "peak":                     # event 1 ends inside event 3
        o[2] = o[3] + (o[4] - o[3]) // 2
    elif kind == "reversed":
        o[1:-1] = o[1:-1][::-1]
    elif kind == "outside":                  # before the first hit and after the last
        o[0], o[-1] = -50, n + 1000
    elif kind == "wild":
        o[1:-1] = np.random.default_rng(3).integers(-n, 2 * n, N_EVENTS - 1)
    return o


@pytest.mark.parametrize("kind", ["rising", "dip", "peak", "reversed", "outside", "wild"])
def test_every_hit_has_one_event(events, kind):
    geom, inp = events
    n = len(inp["x"])
    assert n <= 4096
    off = _offsets(kind, inp["event_off"])
    ev = np.array([_event_of(off, i) if off[0] <= i < off[-1] else -1 for i in range(n)])
    got = _run(geom, dict(inp, event_off=off))
    # the same hits in order of their event, hits of none last
    order = np.argsort(np.where(ev < 0, N_EVENTS, ev), kind="stable")
    new = np.empty(n, np.int64)
    new[order] = np.arange(n)
    plain = dict(inp, event_off=np.searchsorted(ev[order][ev[order] >= 0], np.arange(N_EVENTS + 1)))
    for k in ("x", "y", "z", "su", "sv", "layer"):
        plain[k] = np.asarray(inp[k])[order]
    sh = np.asarray(inp["seed_hits"])
    plain["seed_hits"] = np.where(sh >= 0, new[sh], -1).astype(sh.dtype)
    want = _run(geom, plain)
    assert np.array_equal(np.where(got["hits"] >= 0, new[got["hits"]], -1), want["hits"])
    for k in ("par", "cov", "chi2", "ndf", "status"):
        assert np.array_equal(got[k], want[k]), k
