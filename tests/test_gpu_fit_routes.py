"""A fit takes one of several kernels by its precision, its number of tracks
and whether a launch does one step or all.  The arithmetic is the same in all.
Where registers and memory hold the state in the same precision (mixed fits
round it between launches), a track must come out the same in every bit by one
launch and by one launch a layer; and in 64 bits among as many tracks as one
wave a SIMD holds and among one more."""
import numpy as np
import pytest

import eventgen as E
from tests import common as CM

pytestmark = pytest.mark.gpu
BASE = 300
KEYS = ("par", "cov", "chi2", "ndf", "status")


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1906_02253_amd as K
    return K


def _fit(K, ev, geom, n, flags, learned=False, field=0.0):
    """Fits n tracks, copies of the event's, in order."""
    import torch
    ctx = K.Context(geom, field_z0=field)
    if learned:
        ctx.mlp_load(E.mlp_init(5))
        flags |= K.INIT_MLP
    pick = np.arange(n) % ev.n_tracks
    ld = CM.ld_of(n)
    up = lambda a: torch.as_tensor(CM.soa_int(np.ascontiguousarray(np.asarray(a)[pick]), ld), device="cuda")
    hits = K.Hits.from_event(ev)
    t = K.Tracks(n, ld, flags & 3)
    ctx.seed(hits, up(np.asarray(ev.seq_hit)[:, :3]), t, flags & 3)
    ctx.fit(t, hits, up(ev.seq_layer), up(ev.seq_hit), ev.seq_layer.shape[1], flags)
    torch.cuda.synchronize()
    return t.numpy()


def _event(disks):
    rng = np.random.default_rng(87)
    geom = E.geometry.barrel10_disks14() if disks else E.geometry.barrel10(x0=0.01)
    return geom, E.make_event(rng, geom, BASE, E.pt_power2(0.4, 20.0), 2.4 if disks else 1.0, 0)


@pytest.mark.parametrize("prec", ["FP32", "FP64"])
@pytest.mark.parametrize("kind", ["barrel", "disks", "learned", "field"])
def test_one_launch_and_one_a_layer(K, prec, kind):
    geom, ev = _event(kind == "disks")
    flag = getattr(K, "PREC_" + prec)
    kw = dict(learned=kind == "learned", field=300.0 if kind == "field" else 0.0)
    a = _fit(K, ev, geom, BASE, flag, **kw)
    b = _fit(K, ev, geom, BASE, flag | K.PER_LAYER, **kw)
    for k in KEYS:
        assert np.array_equal(a[k], b[k]), k
    assert ((a["status"] & ~K.ST_FALLBACK) == 0).sum() > BASE // 2


@pytest.mark.parametrize("kind", ["barrel", "disks", "learned", "field"])
@pytest.mark.parametrize("extra", [0, 1])
def test_64_bits_around_one_wave_a_simd(K, kind, extra):
    import torch
    geom, ev = _event(kind == "disks")
    kw = dict(learned=kind == "learned", field=300.0 if kind == "field" else 0.0)
    few = _fit(K, ev, geom, BASE, K.PREC_FP64, **kw)
    n = 256 * torch.cuda.get_device_properties(0).multi_processor_count + extra
    many = _fit(K, ev, geom, n, K.PREC_FP64, **kw)
    pick = np.arange(n) % BASE
    for k in KEYS:
        assert np.array_equal(many[k], few[k][pick]), k
