"""The anchor integrals of very many targets in one call."""
import numpy as np
import pytest

from paper_1811_04156_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rj():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_04156_amd import rjpath
    rjpath.load()
    return rjpath


@pytest.mark.parametrize("targets", [16_384, 16_385, 262_143, 262_145, 1 << 20])
def test_anchor_of_many_targets(rj, targets):
    """A launch has fewer than 2^32 threads, so the blocks per target go down
    from 16 to 1 as the targets grow (between 2^14 and 2^18).  Targets of both
    sectors here and there give what a call of eight gives (the same nodes,
    summed in another order: 1e-12); the others have no anchor sector."""
    w = W.layered_pairs(seed=12, pairs=8, chains=8, cap=8, n_layers=9, dz=4.0, dmin=4.0, dmax=25.0)
    w["t_n0"] = np.array([3, 3, 3, 3, 3, 3, 2, 2], np.int32)
    w["t_emit_kind"] = np.where(w["t_n0"] == 2, W.EMIT_ISO, w["t_emit_kind"]).astype(np.int32)
    few = rj.Sampler(w, precision="f32").anchor()
    assert np.all(few > 0)
    at = np.unique(np.concatenate([np.arange(8), targets // 2 + np.arange(8), targets - 8 + np.arange(8)]))
    big = dict(w)
    for k in list(w):
        if k.startswith("t_"):
            big[k] = np.asarray(w[k])[np.arange(targets) % 8]
    n0 = np.zeros(targets, np.int32)
    n0[at] = big["t_n0"][at]
    big["t_n0"] = n0
    an = rj.Sampler(big, precision="f32").anchor()
    rest = np.ones(targets, bool)
    rest[at] = False
    assert np.all(np.isnan(an[rest]))
    assert np.allclose(an[at], few[at % 8], rtol=1e-12, atol=0)


@pytest.mark.parametrize("targets", [1, 7, 300])
def test_anchor_of_mixed_sectors(rj, targets):
    """Direct sectors, one-scatter sectors of both cap forms and targets
    without an anchor sector side by side, each by the kernel of its own: what
    a call with the one target gives (its sum over as many blocks as a call of
    all has: 1e-12), the same bits in a second call, and the device call's
    (rjpath_intensity_noalloc's anchors: 1e-12)."""
    w = W.layered_pairs(seed=13, pairs=8, chains=8, cap=8, n_layers=9, dz=4.0, dmin=4.0, dmax=25.0)
    w["t_n0"] = np.array([2, 3, 3, 0, 2, 3, 7, 3], np.int32)
    w["t_emit_kind"] = np.where(w["t_n0"] == 2, W.EMIT_ISO, w["t_emit_kind"]).astype(np.int32)
    w["t_det_kind"] = np.array([0, 1, 0, 0, 1, 0, 0, 1], np.int32)
    w["t_det_dir"] = np.tile([0.0, -1.0, 0.0], (8, 1))

    def pick(ix):
        v = dict(w)
        for k in w:
            if k.startswith("t_"):
                v[k] = np.asarray(w[k])[ix]
        v["c_target"] = np.zeros(64, np.int32)
        return v

    one = np.array([rj.Sampler(pick(np.array([t])), precision="f32").anchor()[0] for t in range(8)])
    none = ~np.isin(w["t_n0"], (2, 3))
    assert np.array_equal(np.isnan(one), none)
    ix = (np.arange(targets) * 3 + 1) % 8
    s = rj.Sampler(pick(ix), precision="f32")
    an = s.anchor()
    assert np.allclose(an, one[ix], rtol=1e-12, atol=0, equal_nan=True)
    assert np.array_equal(s.anchor(refresh=True), an, equal_nan=True)
    s.run(200, run=dict(burn_in=0))
    I = [s.intensity_noalloc(anchor=x)["I"].cpu().numpy() for x in (None, torch.as_tensor(an, device=s.dev))]
    assert np.allclose(I[0], I[1], rtol=1e-12, atol=0, equal_nan=True)
