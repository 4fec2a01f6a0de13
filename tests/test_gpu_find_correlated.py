"""Windows whose two residuals are strongly correlated (thin tilted ellipses):
in 32 bits the chi2 of a hit carries the rounding of S00 S11 - S01^2, which may
put it below its larger residual's own share.  Which hit a candidate takes is
decided by that computed chi2 alone, so the scan of a long window (a fine bin
grid) and the queue of a short one (a coarse grid) must choose the same hits
and give the same tracks in every bit, whatever the correlation."""
import numpy as np
import pytest

import eventgen as E
from tests import common as CM

pytestmark = pytest.mark.gpu
N_SEEDS, N_HITS, START, TARGET = 96, 384, 4, 5


def _seeds(geom, rho, rng):
    """States on barrel START flying outwards, sigma(phi) and sigma(theta) of
    0.4 rad, correlated by rho."""
    phi = rng.uniform(-np.pi, np.pi, N_SEEDS)
    R = geom[START]["r_or_z"]
    par = np.stack([R * np.cos(phi), R * np.sin(phi), rng.uniform(-3, 3, N_SEEDS),
                    rng.uniform(-0.3, 0.3, N_SEEDS), phi, np.pi / 2 + rng.uniform(-0.1, 0.1, N_SEEDS)], 1)
    P = np.diag([1e-6, 1e-6, 1e-6, 1e-6, 0.16, 0.16])
    P[4, 5] = P[5, 4] = 0.16 * rho
    cov = np.tile(P[np.triu_indices(6)], (N_SEEDS, 1))
    return par, cov


def _hits_on_axis(geom, pred, pcov, rng):
    """Hits on barrel TARGET at 1 to 1.05 of the ellipse along its long axis:
    the larger residual alone accounts for the whole chi2."""
    R = geom[TARGET]["r_or_z"]
    out = []
    for p, c in zip(pred, pcov):
        P = np.zeros((6, 6))
        P[np.triu_indices(6)] = c
        P = P + P.T - np.diag(np.diag(P))
        want = np.sqrt(rng.uniform(1.0, 1.05, N_HITS)) * rng.choice([-1, 1], N_HITS)
        az0 = np.arctan2(p[1], p[0])
        az = az0 + want * np.sqrt(P[0, 0] + P[1, 1]) / R
        for _ in range(20):                      # the hit azimuth whose ru / sqrt(S00) is `want`
            s, k = np.sin(az), np.cos(az)
            x, y = R * k, R * s
            ru = -s * (x - p[0]) + k * (y - p[1])
            S00 = s * s * P[0, 0] - 2 * s * k * P[0, 1] + k * k * P[1, 1] + 1e-6
            az = az + np.clip(want - ru / np.sqrt(S00), -0.3, 0.3) * np.sqrt(S00) / R
        S01 = -s * P[0, 2] + k * P[1, 2]
        out.append(np.stack([x, y, p[2] + S01 / S00 * ru], 1))
    return np.array(out)


@pytest.mark.parametrize("prec", ["FP32", "MIXED"])
@pytest.mark.parametrize("rho", [0.99, 0.999, 0.9999, 0.99999])
def test_hits_do_not_depend_on_the_bin_grid(prec, rho):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1906_02253_amd as K
    flag = getattr(K, "PREC_" + prec)
    rng = np.random.default_rng(79)
    geom = E.geometry.barrel10(x0=0.0)
    par, cov = _seeds(geom, rho, rng)
    ld = CM.ld_of(N_SEEDS)
    t = K.Tracks.from_numpy(par, cov, ld=ld)
    K.Context(geom).propagate(t, torch.full((ld,), TARGET, dtype=torch.int32, device="cuda"), flags=flag)
    g = t.numpy()
    assert (g["status"] == 0).all()
    xyz = _hits_on_axis(geom, g["par"], g["cov"], rng).reshape(-1, 3)
    n = len(xyz)
    hits = K.Hits(xyz[:, 0], xyz[:, 1], xyz[:, 2], np.full(n, 1e-3), np.full(n, 1e-3),
                  np.full(n, TARGET))
    off = torch.arange(N_SEEDS + 1, dtype=torch.int32, device="cuda") * N_HITS
    ev = torch.zeros(ld, dtype=torch.int32, device="cuda")
    ev[:N_SEEDS] = torch.arange(N_SEEDS, device="cuda")
    none = torch.full((3, ld), -1, dtype=torch.int32, device="cuda")
    for mc in (1, 2, 6, 8):
        ref = None
        for grid in ((8, 8), (512, 32)):         # below and above the length of a long window
            ctx = K.Context([dict(L, nbin_phi=grid[0], nbin_2=grid[1]) for L in geom], max_cands=mc)
            s = K.Tracks.from_numpy(par, cov, ld=ld)
            out = K.Tracks(N_SEEDS, ld)
            oh = torch.full((N_SEEDS, len(geom)), -1, dtype=torch.int32, device="cuda")
            ctx.find(hits, off, s, ev, none, oh, out, flags=flag)
            torch.cuda.synchronize()
            r = dict(out.numpy(), hits=oh.cpu().numpy())
            ref = r if ref is None else ref
            assert (r["hits"][:, TARGET] >= 0).all()
            for k in r:
                assert np.array_equal(r[k], ref[k]), (mc, k, int((r["hits"] != ref["hits"]).any(1).sum()))
