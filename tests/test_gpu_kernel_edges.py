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
    w = W.single_target(1.5, 0.165, 0.05, 50.0, 0.9, chains=130, cap=64, burn_in=150, seed=53)
    out = []
    for v in (40, slots):
        s = rj.Sampler(w, precision=prec)
        for k in range(3):
            s.run(800, block=64, v_lds=v)
        torch.cuda.synchronize()
        n, x = s.get_state()
        used = np.arange(s.cap)[None, :] < n[:, None]
        out.append((n, np.where(used[..., None], x, 0.0), s.logp.cpu().numpy(), s.stats.cpu().numpy()))
    for x, y in zip(*out):
        assert np.array_equal(x, y)
    assert out[0][0].max() > 17 and out[0][3][:, 0].min() == 2250


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


@pytest.mark.parametrize("medium", ["homogeneous", "even", "uneven"])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_score_pass_whatever_the_order_of_the_chains(rj, prec, medium):
    """A wave of the score pass shares the segments of its 64 chains, target by
    target, from a strip that long paths overflow.  The same paths with their
    chains grouped by target, and dealt out so that every wave holds many
    targets (and a ragged last wave), give the same log p and vertex gradients
    bit for bit and the same score sums up to the order of FP64 additions
    (about 1e3 of them: 1e-12)."""
    T, C, cap = 9, 333, 48
    if medium == "homogeneous":
        w = W.homogeneous_groups(seed=2, groups=T, per_group=C // T, cap=cap)
    else:
        w = W.layered_pairs(seed=2, pairs=T, chains=C, cap=cap, n_layers=8, dz=5.0, dmin=4.0, dmax=30.0)
        if medium == "uneven":
            w["edges"] = w["edges"] + np.where(np.arange(9) % 2 == 1, 0.7, 0.0)
    w["lam_s"] = 0.1 * w["lam_s"]  # long paths
    w.update(burn_in=0, sigma=2.0)
    s = rj.Sampler(w, precision=prec)
    s.run(2000)
    torch.cuda.synchronize()
    n, v = s.get_state()
    assert n.max() > 12
    out = []
    for order in (np.arange(C), np.argsort(np.arange(C) % 37, kind="stable")):
        wp = dict(w)
        wp["c_target"] = w["c_target"][order]
        p = rj.Sampler(wp, precision=prec, logw=np.tile(0.1 * np.arange(cap + 1), (T, 1)))
        p.set_state(n[order], v[order])
        lp, g, sc = p.grad(logp=True, dv=True, score=True)
        lp2, _, sc2 = p.grad(logp=True, score=True)
        sl = p.score_length()
        back = np.argsort(order, kind="stable")
        assert torch.equal(torch.isfinite(lp), torch.isfinite(lp2))
        out.append((lp.cpu().numpy()[back], g.cpu().numpy()[:, back], lp2.cpu().numpy()[back],
                    sc.cpu().numpy(), sc2.cpu().numpy(), sl.cpu().numpy()))
    a, b = out
    for i in (0, 2):
        assert np.allclose(a[i], b[i], rtol=1e-13, atol=1e-13)
    assert np.allclose(a[0], a[2], rtol=1e-12 if prec == "f64" else 1e-6)
    assert np.array_equal(a[1], b[1])
    for i in (3, 4, 5):
        assert np.allclose(a[i], b[i], rtol=1e-12, atol=1e-12 * np.abs(a[i]).max())
    assert np.allclose(a[3], a[4], rtol=1e-9, atol=1e-12 * np.abs(a[3]).max())


def test_tree_moves_shared_by_any_number_of_chains(rj):
    """A wave of the tree sampler owns 64 chains of a large launch and 8 of a
    small one; the draws belong to the chain, so the first chains of a
    140,001-chain launch (64 per wave, a ragged last one) take the paths that
    they take as a launch of their own (8 per wave).  The FP64 sums of log A
    may differ in the order of their terms, which a decision has not been
    seen to feel; the statistics' sums differ by their rounding (1e-12)."""
    w = W.layered_pairs(seed=8, pairs=60, chains=140_001, cap=40, n_layers=12, dz=4.0, dmin=4.0, dmax=25.0)
    w.update(sampler=3, mala_h=0.3, burn_in=0, sigma=2.0)
    few = W.subset_chains(w, 5003)
    out = []
    for ww in (w, few):
        s = rj.Sampler(ww, precision="f32")
        s.run(100)
        torch.cuda.synchronize()
        k = 5003
        used = torch.arange(s.cap, device=s.dev)[:, None] < s.n[:k]
        out.append((s.n[:k].cpu().numpy(), torch.where(used[..., None], s.verts[:, :k, :3], 0.0).cpu().numpy(),
                    s.stats[:k].cpu().numpy()))
    a, b = out
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    assert np.allclose(a[2], b[2], rtol=1e-12)
    assert a[2][:, 14].sum() > 1000  # tree moves were accepted


@pytest.mark.parametrize("run", [1, 11])
def test_joint_moves_shared_by_any_number_of_chains(rj, run):
    """A wave of the joint Langevin sampler owns 64 chains of a large launch
    and 8 of a small one, whose lanes without a chain help its targets.  The
    first 5003 chains of a 262,201-chain launch take the paths that they take
    as a launch of their own, with ``run`` neighbouring chains per target
    (waves of up to 64 targets; of one or two of them).  The statistics' sums
    differ by their rounding (1e-12)."""
    w = W.layered_pairs(seed=8, pairs=70, chains=262_201, cap=40, n_layers=12, dz=4.0, dmin=4.0, dmax=25.0)
    w.update(sampler=1, mala_h=0.01, burn_in=0, sigma=2.0)
    w["c_target"] = (np.arange(262_201) // run % 70).astype(np.int32)
    out = []
    for ww in (w, W.subset_chains(w, 5003)):
        s = rj.Sampler(ww, precision="f32")
        s.run(100)
        torch.cuda.synchronize()
        k = 5003
        used = torch.arange(s.cap, device=s.dev)[:, None] < s.n[:k]
        out.append((s.n[:k].cpu().numpy(), torch.where(used[..., None], s.verts[:, :k, :3], 0.0).cpu().numpy(),
                    s.stats[:k].cpu().numpy()))
    a, b = out
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    assert np.allclose(a[2], b[2], rtol=1e-12)
    assert a[2][:, 14].sum() > 1000  # joint moves were accepted


@pytest.mark.parametrize("prec,sampler,chains", [("f32", 0, 140_001), ("f32", 2, 140_001), ("f64", 0, 140_001),
                                                 ("f32", 1, 60_001)])
def test_ordered_launch_leaves_no_trace(rj, prec, sampler, chains):
    """A launch of more blocks than the chip holds takes its waves in the
    order of their vertices, kept in the status words meanwhile.  Every chain
    takes the same path as in launches of fewer steps than the order is made
    for, malformed chains (the first and last among them) are flagged and
    untouched, and the status words hold 0 and 1 alone."""
    w = W.layered_pairs(seed=9, pairs=90, chains=chains, cap=40, n_layers=12, dz=4.0, dmin=4.0, dmax=25.0)
    w.update(sampler=sampler, mala_h=0.05 if sampler == 2 else 0.01, burn_in=0, sigma=2.0)
    out = []
    for parts in ((32,), (8, 8, 8, 8)):
        s = rj.Sampler(w, precision=prec)
        bad = torch.tensor([0, 1, 63, 64, 2186, 2187, 2188, 30_000, chains - 1], device=s.dev)
        s.n[bad] = torch.tensor([0, 1, -3, 41, 1000, 1, 0, 1, 41], dtype=s.n.dtype, device=s.dev)
        s.status.fill_(0x7F7F7F)
        for k in parts:
            s.run(k)
        torch.cuda.synchronize()
        flagged = torch.zeros(chains, dtype=s.status.dtype, device=s.dev)
        flagged[bad] = 1
        assert torch.equal(s.status, flagged)
        used = torch.arange(s.cap, device=s.dev)[:, None] < s.n
        out.append((s.n.clone(), torch.where(used[..., None], s.verts[..., :3], 0.0).clone()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("sampler,h", [(1, 0.01), (3, 0.3)])
def test_far_vertices_of_shared_waves(rj, prec, sampler, h):
    """The whole-path samplers keep the vertices beyond the LDS slots in the
    work buffer and use the chains' own rows meanwhile.  Whatever the slots
    (1: all but one vertex; 40: none; the last wave has 3 chains) and however
    often the launches end, the paths are the same bit for bit, and a
    malformed chain beside them keeps every row it has."""
    w = W.single_target(1.5, 0.165, 0.05, 50.0, 0.9, chains=131, cap=40, burn_in=0, seed=54)
    w.update(sampler=sampler, mala_h=h)
    out = []
    for v, parts in ((40, 1), (16, 1), (3, 4), (1, 2)):
        s = rj.Sampler(w, precision=prec)
        bad = torch.tensor([5, 64, 129], device=s.dev)
        s.n[bad] = torch.tensor([0, 1, 41], dtype=s.n.dtype, device=s.dev)
        marks = torch.arange(40 * 3 * 4, device=s.dev, dtype=s.verts.dtype).reshape(40, 3, 4) + 0.5
        s.verts[:, bad] = marks
        for _ in range(parts):
            s.run(1200 // parts, block=64, v_lds=v)
        torch.cuda.synchronize()
        assert torch.equal(s.verts[:, bad], marks) and s.status[bad].tolist() == [1, 1, 1]
        used = torch.arange(s.cap, device=s.dev)[:, None] < s.n
        used[:, bad] = False
        out.append((s.n.clone(), torch.where(used[..., None], s.verts[..., :3], 0.0).clone()))
    assert out[0][0].max() > 17
    for n, x in out[1:]:
        assert torch.equal(n, out[0][0]) and torch.equal(x, out[0][1])


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("sampler,h", [(1, 0.01), (3, 0.3)])
def test_few_chains_of_shared_moves(rj, prec, sampler, h):
    """Small launches of the whole-path samplers give each chain, or 2, 4 or 8,
    a wave.  The first chains of a 70,001-chain launch (32 per wave) take the
    paths that they take as launches of 1, 63, 1300, 3001 and 9001 chains."""
    w = W.layered_pairs(seed=10, pairs=50, chains=70_001, cap=40, n_layers=12, dz=4.0, dmin=4.0, dmax=25.0)
    w.update(sampler=sampler, mala_h=h, burn_in=0, sigma=2.0)
    w["c_target"] = (np.arange(70_001) % 50).astype(np.int32)
    state = []
    for k in (70_001, 1, 63, 1300, 3001, 9001):
        s = rj.Sampler(W.subset_chains(w, k), precision=prec)
        s.run(100)
        torch.cuda.synchronize()
        used = torch.arange(s.cap, device=s.dev)[:, None] < s.n
        state.append((s.n.clone(), torch.where(used[..., None], s.verts[..., :3], 0.0).clone(), s.stats.clone()))
    n, x, st = state[0]
    for a, b, c in state[1:]:
        k = len(a)
        assert torch.equal(a, n[:k]) and torch.equal(b, x[:, :k])
        assert torch.allclose(c, st[:k], rtol=1e-12)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_bridge_whatever_the_order_and_number_of_chains(rj, prec):
    """The bridge's waves share the vertices of 8 chains in a small launch and
    of 64 in a large one, target by target: the same paths grouped by target,
    dealt out over the targets, and repeated to 131,200 chains give the same
    log r per chain (sums of about 60 FP64 terms of magnitude up to 1e2 in
    another order: 1e-11)."""
    from paper_1811_04156_amd.table1 import replicate
    w = replicate(W.two_region(b1=0.3, scale=0.1, chains_per_sensor=1, cap=64), 3, 55)
    w.update(burn_in=0, sampler=3, mala_h=0.3)
    s = rj.Sampler(w, precision=prec)
    s.run(400)
    torch.cuda.synchronize()
    n, v = s.get_state()
    C = len(n)
    out = []
    orders = [np.arange(C), np.argsort(np.arange(C) % 41, kind="stable")]
    if prec == "f32":
        orders.append(np.tile(np.arange(C), 131_200 // C + 1))
    for order in orders:
        wp = dict(w)
        wp["c_target"] = w["c_target"][order]
        p = rj.Sampler(wp, precision=prec)
        p.set_state(n[order], v[order][:, : n.max()])
        acc, lr = p.yield_accumulate(p.yield_pairs([(0, 1), (2, 3), (4, 5)]), groups=4, logr=True)
        lr = lr.cpu().numpy()
        assert acc[..., 1].sum().item() == np.sum(np.isfinite(lr) | np.isneginf(lr))
        first = np.zeros(C)
        first[order[:C]] = lr[:C]
        out.append(first)
        if len(order) > C:
            assert np.allclose(lr, first[order], rtol=1e-11, atol=1e-11, equal_nan=True)
    for x in out[1:]:
        assert np.allclose(out[0], x, rtol=1e-11, atol=1e-11, equal_nan=True)
    assert np.isfinite(out[0]).sum() > C // 2


@pytest.mark.parametrize("chains", [1, 130, 131_073, 262_145])
def test_length_hist_whatever_the_lanes_per_chain(rj, chains):
    """Four lanes sum a chain's segments up to 131,072 chains, two up to
    262,144, one beyond.  The bins equal a histogram of the state's own lengths
    (a length within 1e-9 of an edge could fall on either side of it: none
    does)."""
    w = W.single_target(1.5, 0.165, 0.05, 50.0, 0.9, chains=chains, cap=24, burn_in=0, seed=55)
    s = rj.Sampler(w, precision="f32")
    s.run(300)
    torch.cuda.synchronize()
    h = s.length_hist(30, 1.0, 0.1).cpu().numpy().ravel()
    used = torch.arange(1, s.cap, device=s.dev)[:, None] < s.n
    x = s.verts[..., :3].double()
    L = torch.where(used, (x[1:] - x[:-1]).norm(dim=-1), 0.0).sum(0).cpu().numpy()
    at = (L - 1.0) / 0.1
    assert np.abs(at - np.round(at)).min() > 1e-9
    want = np.bincount(np.floor(at[(at >= 0) & (at < 30)]).astype(int), minlength=30)
    assert np.array_equal(h[:30], want) and h[30] == chains
