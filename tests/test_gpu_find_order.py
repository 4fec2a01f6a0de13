"""A few seeds are put into tile order by one workgroup, more by the counting
sort over cells.  The order decides only which wave a seed runs in: a seed's
track must be the same in every bit, wherever it stands and however many
others there are.  So copies of an event's seeds, at and around the sizes
where the sort changes, must find what the seeds find by themselves."""
import numpy as np
import pytest

import eventgen as E

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def base():
    rng = np.random.default_rng(74)
    geom = E.geometry.barrel10(x0=0.02)
    evs = [E.make_event(rng, geom, n, E.pt_power2(0.5, 50.0), 1.0, m) for n, m in ((90, 300), (7, 0), (40, 500))]
    return geom, E.find_inputs(evs)


def _run(geom, inp, largest_first):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1906_02253_amd as K
    from paper_1906_02253_amd import pipeline
    ctx = K.Context(geom)
    ctx.set_find_config(256, largest_first)
    fp = pipeline.FindProblem(ctx, inp, prec=K.PREC_MIXED)
    fp.run(K.PREC_MIXED)
    torch.cuda.synchronize()
    return fp.results()


@pytest.mark.parametrize("largest_first", [False, True])
@pytest.mark.parametrize("n,events", [(1, 3), (64, 3), (1023, 3), (1024, 256), (1025, 3), (2048, 257), (2049, 256),
                                      (4096, 3), (4096, 256), (4097, 3)])
def test_seeds_find_the_same_in_any_company(base, n, events, largest_first):
    geom, inp = base
    ref = _run(geom, inp, largest_first)
    n0 = inp["seed_hits"].shape[0]
    rng = np.random.default_rng(n)
    pick = rng.integers(0, n0, n)
    many = dict(inp)
    for k in ("seed_hits", "seed_layers", "seed_event"):
        many[k] = np.ascontiguousarray(np.asarray(inp[k])[pick])
    off = np.asarray(inp["event_off"])
    many["event_off"] = np.append(off, np.full(events - (len(off) - 1), off[-1])).astype(off.dtype)
    r = _run(geom, many, largest_first)
    assert np.array_equal(r["hits"], ref["hits"][pick])
    for k in ("par", "cov", "chi2", "ndf", "status"):
        want = ref[k][..., pick] if ref[k].shape[-1] == n0 else ref[k][pick]
        assert np.array_equal(r[k], want), k
