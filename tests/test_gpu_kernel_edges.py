"""Kernel branches at the sizes and shapes where they change over, against
the FP64 oracle or the kernels' own general forms."""
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


def _cone_targets(edges, f_sl, det, sensor_z, copies=1):
    """Cone sources (20 degrees about x) at z = 5 whose sensor (radius 0.165 m,
    about 55 degrees off the axis, 8 m away) is centred at height sensor_z."""
    L = len(edges) - 1
    rng = np.random.default_rng(L)
    media = W._layered_medium(rng.uniform(8, 30, L), rng.uniform(30, 90, L), np.full(L, 0.9), 0.0, 1.0)
    media["edges"] = np.asarray(edges, np.float64)
    media["f_sl"] = np.full(L, f_sl)
    src = np.tile([0.0, 0.0, 5.0], (copies, 1))
    sen = np.array([[4.6, 6.5, sensor_z]] * copies) + np.arange(copies)[:, None] * [0.3, 0.0, 0.0]
    r, ax, half = np.full(copies, 0.165), np.tile([1.0, 0.0, 0.0], (copies, 1)), np.full(copies, np.deg2rad(20.0))
    n, init = W._cone_start(src, sen, r, ax, half)
    tg = W._targets(np.zeros(copies), src, sen, r, np.full(copies, W.EMIT_CONE), ax, half, n, init,
                    np.full(copies, det), np.tile([0.0, -1.0, 0.0], (copies, 1)))
    w = dict(name="cone", cap=16, **media, **tg, c_target=np.arange(copies, dtype=np.int32))
    w.update(W.DEFAULT_RUN)
    return w


@pytest.mark.parametrize("case", ["one layer", "inside", "astride an edge", "over several edges", "mixture", "paper"])
@pytest.mark.parametrize("copies", [1, 3])
def test_one_scatter_anchor_branches(rj, case, copies):
    """I_3 at the device's resolution against the oracle's same rule, for each
    form of the cap integral: the sensor inside one layer, astride one edge
    and over several edges (the general form, as for the simplified-Liu
    mixture and the paper's angular response).  The same nodes summed in FP64:
    rounding only, held to 1e-9 as for the layered batch's targets."""
    from oracle import oracle as O
    edges = {"one layer": [0.0, 100.0], "over several edges": [0.0, 3.0, 6.95, 7.0, 7.05, 12.0]}.get(
        case, [0.0, 3.0, 7.0, 12.0])
    z = 7.0 if case in ("astride an edge", "over several edges") else 5.8
    w = _cone_targets(edges, 0.45 if case == "mixture" else 0.0, 1 if case == "paper" else 0, z, copies)
    assert np.all(w["t_n0"] == 3)
    an = rj.Sampler(w, precision="f32").anchor()
    orc = O.Oracle(w)
    for t in range(copies):
        ref = orc.anchor_I3(t, 32, 32, 32, 8, 8)
        print(case, t, an[t] / ref - 1)
        assert an[t] == pytest.approx(ref, rel=1e-9), t


def _with_spare_medium(w):
    """The same workload with one more, homogeneous medium that no target
    uses: the launch then takes the kernels without the even-layers facts."""
    w = dict(w)
    L = len(w["lam_s"])
    w["m_axis"] = np.concatenate([w["m_axis"], [[0.0, 0.0, 1.0]]])
    w["m_layer_off"] = np.append(w["m_layer_off"], L).astype(np.int32)
    w["m_layer_cnt"] = np.append(w["m_layer_cnt"], 1).astype(np.int32)
    w["edges"] = np.concatenate([w["edges"], [0.0, 1.0]])
    for k, v in (("lam_s", 20.0), ("lam_a", 80.0), ("g", 0.9), ("f_sl", 0.0)):
        w[k] = np.append(w[k], v)
    return w


@pytest.mark.parametrize("f_sl", [0.0, 0.45])
@pytest.mark.parametrize("sampler", [0, 1, 2, 3])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_even_layer_kernels_take_the_general_kernels_steps(rj, prec, sampler, f_sl):
    """Evenly layered media run kernels of their own; the general ones do the
    same arithmetic, so the paths agree bit for bit (257 chains: a ragged last
    wave; 5 slots per chain, so that paths leave them)."""
    w = W.layered_pairs(seed=4, pairs=7, chains=257, cap=40, n_layers=9, dz=4.0, dmin=4.0, dmax=25.0)
    w["f_sl"] = np.where(np.arange(9) % 2 == 0, f_sl, 0.0)
    w.update(sampler=sampler, mala_h=0.02 if sampler == 1 else 0.2, sigma=2.0, burn_in=0)
    out = []
    for ww in (w, _with_spare_medium(w)):
        s = rj.Sampler(ww, precision=prec)
        s.run(300, block=64, v_lds=5)
        torch.cuda.synchronize()
        n, v = s.get_state()
        used = np.arange(s.cap)[None, :] < n[:, None]
        out.append((n, np.where(used[..., None], v, 0.0), s.logp.cpu().numpy(), s.stats.cpu().numpy()))
    for x, y in zip(*out):
        assert np.array_equal(x, y)
    assert out[0][0].max() > 6


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("slots", [1, 7, 8, 9, 15, 16, 17])
def test_slot_count_around_the_scan_leaves_the_paths_alone(rj, prec, slots):
    """A birth's segment scan reads a fixed number of LDS slots and continues
    in HBM; path lengths on both sides of the slot count and of the scan give
    the same paths bit for bit, whatever the slots (sampling also starts in
    the middle of the launch, so that the statistics fold a partial run)."""
    w = W.single_target(1.5, 0.165, 0.3, 50.0, 0.9, chains=130, cap=64, burn_in=150, seed=53)
    out = []
    for v in (40, slots):
        s = rj.Sampler(w, precision=prec)
        for k in range(3):
            s.run(200, block=64, v_lds=v)
        torch.cuda.synchronize()
        n, x = s.get_state()
        used = np.arange(s.cap)[None, :] < n[:, None]
        out.append((n, np.where(used[..., None], x, 0.0), s.logp.cpu().numpy(), s.stats.cpu().numpy()))
    for x, y in zip(*out):
        assert np.array_equal(x, y)
    assert out[0][0].max() > 17 and out[0][3][:, 0].min() == 450


@pytest.mark.parametrize("chains", [49_152, 51_201])
def test_default_launch_with_staged_tables(rj, chains):
    """The default launch gives up slots so that four blocks with 100-layer
    tables share a CU (from 49,153 chains on 256 CUs): the same paths as with
    an explicit launch."""
    w = W.layered_pairs(seed=6, pairs=50, chains=chains, cap=48)
    w["burn_in"] = 0
    out = []
    for kw in (dict(), dict(block=128, v_lds=11)):
        s = rj.Sampler(w, precision="f32")
        s.run(60, **kw)
        torch.cuda.synchronize()
        out.append((s.n.clone(), s.logp.clone(), s.stats.clone()))
    for x, y in zip(*out):
        assert torch.equal(x, y)
