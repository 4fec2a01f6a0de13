"""Few hits are binned by one launch, many through two levels of counting
sort, and a layer with more hits than a workgroup's LDS holds by a path of its
own in each.  The order of the hits inside a bin is free, and no result may
depend on it or on the route: an event by itself (one launch) and the same
event beside a large one (two levels) must give the same tracks in every bit.
Hits of no layer and hits outside the events are left out by both."""
import numpy as np
import pytest

import eventgen as E

pytestmark = pytest.mark.gpu
KEYS = ("par", "cov", "chi2", "ndf", "status")


def _run(K, geom, inp):
    import torch
    from paper_1906_02253_amd import pipeline
    fp = pipeline.FindProblem(K.Context(geom), inp, prec=K.PREC_MIXED)
    fp.run(K.PREC_MIXED)
    torch.cuda.synchronize()
    return fp.results()


def _with_strays(inp, n_layers, rng):
    """The same hits among strays: of layers that do not exist inside the
    events, of layer 0 before the first event and after the last."""
    n, off = len(inp["x"]), np.asarray(inp["event_off"])
    m = 500 + n // 3
    at = np.sort(rng.integers(0, n + 1, m))
    at[:7], at[-7:] = 0, n
    where = np.zeros(n + m, bool)
    where[at + np.arange(m)] = True
    new = np.flatnonzero(~where)                        # place of each old hit
    out = dict(inp)
    for k in ("x", "y", "z", "su", "sv", "layer"):
        old = np.asarray(inp[k])
        v = np.empty(n + m, old.dtype)
        v[new] = old
        v[where] = rng.choice([-1, n_layers, 1000], m) if k == "layer" else rng.normal(0, 30, m)
        out[k] = v
    o = np.append(new, n + m)[off]
    o[0], o[-1] = 7, n + m - 7
    out["layer"][:7] = out["layer"][-7:] = 0
    out["event_off"] = o.astype(np.asarray(inp["event_off"]).dtype)
    sh = np.asarray(inp["seed_hits"])
    out["seed_hits"] = np.where(sh >= 0, new[sh], -1).astype(sh.dtype)
    return out, new


@pytest.mark.parametrize("layers,grid,sizes", [
    (10, (128, 32), [(40, 3_000), (1, 0), (60, 30_000)]),       # one workgroup or several a layer
    (24, (512, 32), [(40, 3_000), (80, 50_000)]),               # the largest grid
    (4, (7, 3), [(30, 62_000), (5, 0), (2, 900)]),              # a layer of more than 15,360 hits
    (4, (1, 1), [(10, 1_100), (3, 40)]),                        # one bin, one row to share
])
def test_results_do_not_depend_on_the_route(layers, grid, sizes):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1906_02253_amd as K
    rng = np.random.default_rng(73)
    geom = E.geometry.barrel10_disks14() if layers > 10 else E.geometry.barrel10(x0=0.02)[:layers]
    geom = [dict(L, nbin_phi=grid[0], nbin_2=grid[1]) for L in geom]
    evs = [E.make_event(rng, geom, n, E.pt_power2(0.5, 50.0), 1.0, m // layers) for n, m in sizes]
    big = E.make_event(rng, geom, 20, E.pt_power2(0.5, 50.0), 1.0, 120_000 // layers)
    inp = E.find_inputs(evs + [big])
    both = _run(K, geom, inp)
    strays, new = _with_strays(inp, layers, rng)
    r = _run(K, geom, strays)
    for k in KEYS:
        assert np.array_equal(r[k], both[k]), k
    assert np.array_equal(r["hits"], np.where(both["hits"] >= 0, new[both["hits"]], -1))
    off, se = np.asarray(inp["event_off"]), np.asarray(inp["seed_event"])
    for e, ev in enumerate(evs):
        one = E.find_inputs([ev])
        if one["seed_hits"].shape[0] == 0:
            continue
        assert len(one["x"]) <= 65_536 < len(inp["x"])
        mine = se == e
        for with_strays in (False, True):
            new = np.arange(len(one["x"]))
            if with_strays:
                one, new = _with_strays(one, layers, rng)
            r = _run(K, geom, one)
            for k in KEYS:
                assert np.array_equal(r[k], both[k][..., mine] if both[k].shape[-1] == len(se) else both[k][mine]), (e, k)
            want = both["hits"][mine]
            assert np.array_equal(r["hits"], np.where(want >= 0, new[want - off[e]], -1)), e
