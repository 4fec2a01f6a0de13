"""The network's forward pass takes only the lanes that want a guess, packed
into as few 16-row tiles as hold them.  A row's guess does not depend on the
tile or the row it is computed in: a track fitted with the learned start must
come out the same in every bit whatever tracks share its wave, and whether they
want guesses or not (a track whose layer sequence is empty wants none)."""
import numpy as np
import pytest

import eventgen as E
from tests import common as CM

pytestmark = pytest.mark.gpu


def _fit(K, geom, hits, w, sh, lay, hit):
    import torch
    ctx = K.Context(geom)
    ctx.mlp_load(w)
    n = sh.shape[0]
    ld = CM.ld_of(n)
    up = lambda a: torch.as_tensor(CM.soa_int(np.ascontiguousarray(a), ld), device="cuda")
    t = K.Tracks(n, ld)
    ctx.seed(hits, up(sh), t)
    ctx.fit(t, hits, up(lay), up(hit), lay.shape[1], K.INIT_MLP)
    torch.cuda.synchronize()
    return t.numpy()


@pytest.mark.parametrize("wanted", [0, 1, 15, 16, 17, 31, 33, 48, 49, 63, 64])
def test_a_guess_does_not_depend_on_its_row(wanted):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1906_02253_amd as K
    geom, ev = E.fit_sample(n_tracks=320, seed=5)
    w = E.mlp_init(5)
    hits = K.Hits.from_event(ev)
    lay, hit = np.asarray(ev.seq_layer), np.asarray(ev.seq_hit)
    ref = _fit(K, geom, hits, w, hit[:, :3], lay, hit)
    # of every 64 tracks, `wanted` keep their sequence, at random places
    rng = np.random.default_rng(wanted)
    keep = np.concatenate([rng.permutation(64) < wanted for _ in range(-(-len(lay) // 64))])[:len(lay)]
    l2, h2 = lay.copy(), hit.copy()
    l2[~keep], h2[~keep] = -1, -1
    r = _fit(K, geom, hits, w, hit[:, :3], l2, h2)
    for k in ("par", "cov", "chi2", "ndf", "status"):
        a, b = (v if v.shape[0] == len(lay) else v.T for v in (r[k], ref[k]))
        assert np.array_equal(a[keep], b[keep]), k
