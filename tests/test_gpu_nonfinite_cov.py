"""A covariance with an entry that is not finite.  A seed or a track that is
not moved keeps its covariance bit for bit (a frozen seed in finding, a track
whose first surface cannot be reached in a fit or a propagation); one that is
moved gets the full product F P F^T, in which the rows of F for q/pT and theta
are unit rows; and its neighbours' results do not change in any bit."""
import numpy as np
import pytest

import eventgen as E
from tests import common as CM

pytestmark = pytest.mark.gpu
PK = {(i, j): k for k, (i, j) in enumerate(zip(*np.triu_indices(6)))}


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1906_02253_amd as K
    return K


def _fit_setup(K, prec):
    import torch
    geom, ev = E.fit_sample(n_tracks=96, seed=17)
    ld = CM.ld_of(ev.n_tracks)
    up = lambda a: torch.as_tensor(CM.soa_int(np.ascontiguousarray(a), ld), device="cuda")
    ctx = K.Context(geom)
    hits = K.Hits.from_event(ev)
    t = K.Tracks(ev.n_tracks, ld, prec)
    ctx.seed(hits, up(ev.seq_hit[:, :3]), t, prec)
    return geom, ev, ctx, hits, t, up, ld


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("prec", ["MIXED", "FP32"])
def test_frozen_seed_keeps_its_covariance(K, prec, value):
    import torch
    from paper_1906_02253_amd import pipeline
    flag = getattr(K, "PREC_" + prec)
    geom = E.geometry.barrel10(x0=0.02)
    ev = E.make_event(np.random.default_rng(5), geom, 60, E.pt_power2(0.5, 50.0), 1.0, 300)
    fp = pipeline.FindProblem(K.Context(geom), E.find_inputs([ev]), prec=flag)
    fp.seed_fit(flag)
    frozen = [0, 7, 20]
    for s in frozen:
        fp.seeds.status[s] = K.ST_NOCONV
    fp.find(flag)
    torch.cuda.synchronize()
    want = fp.results()
    entries = [PK[1, 2], PK[3, 3], PK[5, 5]]
    for s, k in zip(frozen, entries):
        fp.seeds.cov[k, s] = float(value)
    fp.find(flag)
    torch.cuda.synchronize()
    got = fp.results()
    seeds = fp.seeds.numpy()
    for s in frozen:
        assert np.array_equal(got["cov"][s], seeds["cov"][s], equal_nan=True), s
    others = np.setdiff1d(np.arange(fp.n_seeds), frozen)
    for k in ("hits", "par", "cov", "chi2", "ndf", "status"):
        assert np.array_equal(got[k][others], want[k][others]), k


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("prec", ["MIXED", "FP32", "FP64"])
@pytest.mark.parametrize("per_layer", [False, True])
def test_unreachable_first_surface_keeps_the_covariance(K, prec, value, per_layer):
    import torch
    flag = getattr(K, "PREC_" + prec)
    geom, ev, ctx, hits, t, up, ld = _fit_setup(K, flag)
    lay, hit = np.array(ev.seq_layer), np.array(ev.seq_hit)
    stuck = [3, 64, 90]
    t.par[3, stuck] = 50.0                      # a circle of 2 cm radius
    lay[stuck, 0] = 9                           # never gets to 100 cm
    lay[stuck, 1:] = -1
    want = None
    for v in (0.0, float(value)):
        s = K.Tracks(t.n, t.ld, flag)
        for a in ("par", "cov", "chi2", "ndf", "status"):
            getattr(s, a).copy_(getattr(t, a))
        s.cov[PK[3, 4], stuck] = v
        before = s.numpy()
        ctx.fit(s, hits, up(lay), up(hit), lay.shape[1], flag | (K.PER_LAYER if per_layer else 0))
        torch.cuda.synchronize()
        got = s.numpy()
        assert (got["status"][stuck] & K.ST_UNREACHABLE).all()
        assert np.array_equal(got["cov"][stuck], before["cov"][stuck], equal_nan=True)
        want = got if want is None else want
    others = np.setdiff1d(np.arange(t.n), stuck)
    for k in want:
        assert np.array_equal(got[k][others], want[k][others]), k


@pytest.mark.parametrize("prec", ["MIXED", "FP32", "FP64"])
@pytest.mark.parametrize("layer", [3, 11])
def test_moved_covariance_is_the_full_product(K, prec, layer):
    import torch
    flag = getattr(K, "PREC_" + prec)
    geom = [dict(L, x0=0.0) for L in E.geometry.barrel10_disks14()]
    n, ld = 64, 64
    rng = np.random.default_rng(9)
    R = geom[0]["r_or_z"]
    phi = rng.uniform(-3, 3, n)
    theta = rng.uniform(1.2, 1.9, n) if layer < 10 else rng.uniform(0.2, 0.4, n)
    if geom[layer]["kind"] == 1 and geom[layer]["r_or_z"] < 0:
        theta = np.pi - theta
    par = np.stack([R * np.cos(phi), R * np.sin(phi), np.zeros(n), rng.uniform(-1, 1, n), phi, theta], 1)
    cov = np.tile(np.diag([1e-4, 1e-4, 1e-3, 1e-4, 1e-5, 1e-5])[np.triu_indices(6)], (n, 1))
    cov[:, PK[3, 5]] = 2e-6
    out = []
    target = torch.full((ld,), layer, dtype=torch.int32, device="cuda")
    for v in (0.0, np.inf):
        c = cov.copy()
        if v:
            c[[5, 40], PK[4, 4]] = v
        t = K.Tracks.from_numpy(par, c, flag, ld=ld)
        K.Context(geom).propagate(t, target, flags=flag)
        torch.cuda.synchronize()
        out.append(t.numpy())
    a, b = out
    assert (a["status"] == 0).all()
    others = np.setdiff1d(np.arange(n), [5, 40])
    for k in a:
        assert np.array_equal(a[k][others], b[k][others]), k
    for s in (5, 40):
        # phi's variance enters every entry but those of q/pT and theta alone
        for ij in ((3, 3), (3, 5), (5, 5)):
            assert b["cov"][s, PK[ij]] == a["cov"][s, PK[ij]], (s, ij)
        assert not np.isfinite(b["cov"][s, PK[4, 4]])
        assert np.array_equal(b["par"][s], a["par"][s])
