"""Tracks that want no guess stay as they are: with an empty layer sequence for
every track, or for all but a few of each wave, a learned fit leaves their
seeds' states as it found them, bit for bit."""
import numpy as np
import pytest

import eventgen as E
from tests import common as CM

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wanted", [0, 1, 17])
def test_unwanted_tracks_stay(wanted):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1906_02253_amd as K
    geom, ev = E.fit_sample(n_tracks=320, seed=5)
    lay, hit = np.array(ev.seq_layer), np.array(ev.seq_hit)
    n, ld = len(lay), CM.ld_of(len(lay))
    rng = np.random.default_rng(wanted)
    keep = np.concatenate([rng.permutation(64) < wanted for _ in range(-(-n // 64))])[:n]
    lay[~keep], hit[~keep] = -1, -1
    up = lambda a: torch.as_tensor(CM.soa_int(np.ascontiguousarray(a), ld), device="cuda")
    ctx = K.Context(geom)
    ctx.mlp_load(E.mlp_init(5))
    hits = K.Hits.from_event(ev)
    t = K.Tracks(n, ld)
    ctx.seed(hits, up(np.asarray(ev.seq_hit)[:, :3]), t)
    torch.cuda.synchronize()
    seeds = t.numpy()
    ctx.fit(t, hits, up(lay), up(hit), lay.shape[1], K.INIT_MLP)
    torch.cuda.synchronize()
    r = t.numpy()
    for k in ("par", "cov", "status"):
        assert np.array_equal(r[k][~keep], seeds[k][~keep]), k
    assert (r["ndf"][~keep] == -5).all() and (r["chi2"][~keep] == 0).all()
    if wanted:
        assert not np.array_equal(r["par"][keep], seeds["par"][keep])
