"""Kernels whose waves either share their chains' items or give each lane its
own chain: both forms on the same paths."""
import numpy as np
import pytest

from gpu_helpers import mixed_workload, random_paths
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


def _workload(medium, chains, cap):
    if medium == "homogeneous":
        return W.homogeneous_groups(seed=2, groups=4, per_group=chains // 4, cap=cap)
    if medium == "mixture":
        return mixed_workload(cap=cap, chains=chains)  # 12 layers
    w = W.layered_pairs(seed=2, pairs=4, chains=chains, cap=cap, n_layers=20, dz=2.0, dmin=4.0, dmax=15.0)
    if medium == "uneven":
        w["edges"] = w["edges"] + np.where(np.arange(21) % 2 == 1, 0.3, 0.0)
    return w


@pytest.mark.parametrize("medium", ["homogeneous", "even", "uneven", "mixture"])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_score_pass_by_items_and_by_lanes(rj, prec, medium):
    """The same paths with every wave's lengths alike (a lane per chain; up to
    20 vertices, which the wave's LDS strip does not hold) and with long ones
    beside short ones (shared), for one, two and 64 targets per wave: the same
    vertex gradients bit for bit, log p up to the order of its FP64 terms
    (1e-13 relative), the score sums likewise (1e-12)."""
    from oracle import oracle as O
    C, cap = 512, 24
    w = _workload(medium, C, cap)
    T = len(w["t_src"])
    w["c_target"] = np.zeros(C, np.int32)
    orc = O.Oracle(w)
    rng = np.random.default_rng(11)
    n, V = random_paths(orc, w, rng, 20)
    lw = np.tile(0.05 * np.arange(cap + 1), (T, 1))
    alike, ragged = np.argsort(n, kind="stable"), np.argsort(rng.permutation(C), kind="stable")
    out = []
    for order in (alike, ragged):
        s = rj.Sampler(w, precision=prec, logw=lw)
        s.set_state(n[order], V[order])
        lp, g, _ = s.grad(logp=True, dv=True)
        lp2, _, sc = s.grad(logp=True, score=True)
        lp3, g3, sc3 = s.grad(logp=True, dv=True, score=True)
        lp4, _, _ = s.grad(logp=True)
        back = np.argsort(order, kind="stable")
        out.append(([x.cpu().numpy()[back] for x in (lp, lp2, lp3, lp4)], [x.cpu().numpy()[:, back] for x in (g, g3)],
                    [x.cpu().numpy() for x in (sc, sc3, s.score_length())]))
    a, b = out
    for x, y in zip(a[0], b[0]):
        assert np.allclose(x, y, rtol=1e-13, atol=1e-13)
    assert np.all(np.isfinite(a[0][0])) and np.array_equal(a[1][0], b[1][0]) and np.array_equal(a[1][1], b[1][1])
    for x, y in zip(a[2], b[2]):
        assert np.allclose(x, y, rtol=1e-12, atol=1e-12 * np.abs(x).max())
    for c in range(0, C, 37):
        ref = orc.logp(0, V[c, : n[c]])
        assert abs(a[0][0][c] - ref) < (1e-9 if prec == "f64" else 2e-3), (c, a[0][0][c], ref)
    # targets dealt out: a score table per block no more, sums of few layers by lanes
    for run in (1, 64):
        wd = dict(w)
        wd["c_target"] = (np.arange(C) // run % T).astype(np.int32)
        n2, V2 = random_paths(O.Oracle(wd), wd, np.random.default_rng(12), 20)
        res = []
        for order in (np.arange(C), np.argsort(wd["c_target"], kind="stable")):
            wo = dict(wd)
            wo["c_target"] = wd["c_target"][order]
            s = rj.Sampler(wo, precision=prec, logw=lw)
            s.set_state(n2[order], V2[order])
            lp, g, sc = s.grad(logp=True, dv=True, score=True)
            back = np.argsort(order, kind="stable")
            res.append((lp.cpu().numpy()[back], g.cpu().numpy()[:, back], sc.cpu().numpy()))
        assert np.allclose(res[0][0], res[1][0], rtol=1e-13, atol=1e-13) and np.array_equal(res[0][1], res[1][1])
        assert np.allclose(res[0][2], res[1][2], rtol=1e-12, atol=1e-12 * np.abs(res[0][2]).max())


@pytest.mark.parametrize("medium", ["homogeneous", "even", "uneven", "mixture"])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_score_pass_of_long_paths(rj, prec, medium):
    """Ragged paths of up to 80 vertices, all in two waves (more than four of a
    wave's LDS strips) and spread over eight among paths of up to 4: the same
    vertex gradients bit for bit, log p up to the order of its FP64 terms (1e-13
    relative), the score sums likewise (1e-12).  Against the oracle the bound of 20
    vertices (2e-3 in FP32) times four."""
    from oracle import oracle as O
    C, cap = 512, 80
    w = _workload(medium, C, cap)
    w["c_target"] = np.zeros(C, np.int32)
    orc = O.Oracle(w)
    rng = np.random.default_rng(13)
    n, V = random_paths(orc, w, rng, 80)
    short, Vs = random_paths(orc, w, rng, 4)
    n[128:], V[128:] = short[128:], Vs[128:]
    assert all(n[c : c + 64].sum() > 4 * 7 * 64 for c in (0, 64))
    out = []
    for order in (np.arange(C), np.argsort(np.arange(C) % 128, kind="stable")):
        s = rj.Sampler(w, precision=prec)
        s.set_state(n[order], V[order])
        lp, g, _ = s.grad(logp=True, dv=True)
        lp2, _, sc = s.grad(logp=True, score=True)
        lp3, g3, sc3 = s.grad(logp=True, dv=True, score=True)
        lp4, _, _ = s.grad(logp=True)
        back = np.argsort(order, kind="stable")
        out.append(([x.cpu().numpy()[back] for x in (lp, lp2, lp3, lp4)], [x.cpu().numpy()[:, back] for x in (g, g3)],
                    [x.cpu().numpy() for x in (sc, sc3)]))
    a, b = out
    for x, y in zip(a[0], b[0]):
        assert np.all(np.isfinite(x)) and np.allclose(x, y, rtol=1e-13, atol=1e-13)
    assert np.array_equal(a[1][0], b[1][0]) and np.array_equal(a[1][1], b[1][1])
    for x, y in zip(a[2], b[2]):
        assert np.allclose(x, y, rtol=1e-12, atol=1e-12 * np.abs(x).max())
    for c in range(0, 128, 7):
        ref = orc.logp(0, V[c, : n[c]])
        assert abs(a[0][0][c] - ref) < (1e-9 if prec == "f64" else 8e-3), (c, a[0][0][c], ref)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_bridge_by_vertices_and_by_lanes(rj, prec):
    """The bridge's waves share their chains' vertices or give each lane its
    own chain's, by their lengths and targets.  The same paths grouped by
    target with every wave's lengths alike, mixed, and dealt out over six
    targets give the same log r (FP64 sums of about 60 terms of magnitude up to
    1e2 in another order: 1e-11), NaN for the pair whose second sensor lies on
    the emission axis (no map), and the same sums.  FP64: the oracle's log r to
    1e-8."""
    from oracle import oracle as O
    from paper_1811_04156_amd.table1 import replicate
    w = replicate(W.two_region(b1=0.3, scale=0.1, radius=(0.15, 0.3), chains_per_sensor=1, cap=24), 3, 256)
    C = len(w["c_target"])
    orc = O.Oracle(w)
    n, V = random_paths(orc, w, np.random.default_rng(5), 20)
    t = np.asarray(w["c_target"])
    orders = [np.lexsort((n, t)), np.lexsort((np.arange(C) * 7919 % C, t)), np.arange(C) % 6 * 256 + np.arange(C) // 6]
    out = []
    for order in orders:
        wo = dict(w)
        wo["c_target"] = t[order]
        s = rj.Sampler(wo, precision=prec)
        s.set_state(n[order], V[order])
        acc, lr = s.yield_accumulate(s.yield_pairs([(0, 1), (2, 3), (5, 4)]), groups=2, logr=True)
        out.append((lr.cpu().numpy()[np.argsort(order, kind="stable")], acc.cpu().numpy().sum(2)))
    a, sums = out[0]
    assert np.all(np.isnan(a[t >= 4])) and np.all(sums[2] == 0)
    assert np.isfinite(a[t < 4]).sum() > 400
    for b, other in out[1:]:
        assert np.allclose(a, b, rtol=1e-11, atol=1e-11, equal_nan=True)
        assert np.allclose(sums, other, rtol=1e-10)
    if prec == "f64":
        for c in range(0, 4 * 256, 29):
            ref = orc.yield_log_ratio(t[c] // 2 * 2, t[c] // 2 * 2 + 1, t[c] % 2, V[c, : n[c]])
            assert (a[c] == -np.inf and not np.isfinite(ref)) or abs(a[c] - ref) < 1e-8, (c, a[c], ref)


@pytest.mark.parametrize("chains", [65_537, 131_072, 131_073])
def test_length_hist_at_its_lines(rj, chains):
    """Four lanes sum a chain's segments up to 65,536 chains (256 CUs), two up
    to 131,072, one beyond: every chain is counted once, in the bin of its own
    length (none lies within 1e-9 of an edge)."""
    w = W.single_target(1.5, 0.165, 0.05, 50.0, 0.9, chains=chains, cap=24, burn_in=0, seed=56)
    s = rj.Sampler(w, precision="f32")
    s.run(200)
    torch.cuda.synchronize()
    h = s.length_hist(30, 1.0, 0.1).cpu().numpy().ravel()
    used = torch.arange(1, s.cap, device=s.dev)[:, None] < s.n
    x = s.verts[..., :3].double()
    L = torch.where(used, (x[1:] - x[:-1]).norm(dim=-1), 0.0).sum(0).cpu().numpy()
    at = (L - 1.0) / 0.1
    assert np.abs(at - np.round(at)).min() > 1e-9
    want = np.bincount(np.floor(at[(at >= 0) & (at < 30)]).astype(int), minlength=30)
    assert np.array_equal(h[:30], want) and h[30] == chains


@pytest.mark.parametrize("sampler,h,chains", [(3, 0.3, 131_072), (1, 0.01, 131_073)])
def test_launches_of_few_steps(rj, sampler, h, chains):
    """Launches of fewer than 4 and 16 steps of the whole-path samplers take
    more chains per wave (tree moves 64 instead of 32, joint Langevin moves 64
    at 1 step, 32 at 4): the same paths however the steps are cut, by calls and
    by the chunks of one."""
    w = W.layered_pairs(seed=14, pairs=60, chains=chains, cap=40, n_layers=12, dz=4.0, dmin=4.0, dmax=25.0)
    w.update(sampler=sampler, mala_h=h, burn_in=0, sigma=2.0)
    out = []
    for parts, chunk in (((24,), 0), ((1, 3, 4, 15, 1), 0), ((24,), 3)):
        s = rj.Sampler(w, precision="f32")
        for k in parts:
            s.run(k, chunk=chunk)
        torch.cuda.synchronize()
        used = torch.arange(s.cap, device=s.dev)[:, None] < s.n
        out.append((s.n.clone(), torch.where(used[..., None], s.verts[..., :3], 0.0).clone(), s.status.clone()))
    for x in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(x, out[0]))
    assert out[0][0].max() > 4 and out[0][2].sum() == 0


def test_order_at_its_largest_launch(rj):
    """A launch of 16,384 waves is ordered, one of a wave more is not: the same
    paths, and status words of 0 and 1 alone.  The order is kept beside the
    status in its words, so a chain that was flagged before the launch and one
    with other bits set end as flagged or not by this launch."""
    chains = 64 * 16_384 + 1
    w = W.layered_pairs(seed=15, pairs=90, chains=chains, cap=12, n_layers=12, dz=4.0, dmin=4.0, dmax=25.0)
    w.update(burn_in=0, sigma=2.0)
    out = []
    for k in (chains, chains - 1):
        s = rj.Sampler(W.subset_chains(w, k), precision="f32")
        s.n[5] = 13
        s.status.fill_(1)
        s.status[::3] = 0x01020304
        s.run(20)
        torch.cuda.synchronize()
        flagged = torch.zeros(k, dtype=s.status.dtype, device=s.dev)
        flagged[5] = 1
        assert torch.equal(s.status, flagged)
        used = torch.arange(s.cap, device=s.dev)[:, None] < s.n
        used[:, 5] = False
        out.append((s.n[: chains - 1].clone(), torch.where(used[..., None], s.verts[..., :3], 0.0)[:, : chains - 1].clone()))
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("per", [8, 16, 32, 64])
@pytest.mark.parametrize("prec,sampler,h", [("f32", 1, 0.01), ("f64", 1, 0.01), ("f32", 3, 0.3), ("f64", 3, 0.3)])
def test_far_vertices_of_waves_of_many_chains(rj, prec, sampler, h, per):
    """Waves of 8 to 64 chains whose paths and proposals leave the LDS slots:
    the paths are the same bit for bit whatever the slots (40: nothing leaves
    them), malformed chains beside healthy ones in a wave keep every row they
    have, and the proposals do lie in other chains' rows (a run without jumps,
    where a chain of its own wave would write rows below its own n alone)."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    lines = {3: {8: 40, 16: 100, 32: 300, 64: 520}, 1: {8: 100, 16: 200, 32: 600, 64: 1030}}
    chains = lines[sampler][per] * cus + 3
    cap = 40
    w = W.single_target(1.5, 0.165, 0.05, 50.0, 0.9, chains=chains, cap=cap, burn_in=0, seed=57)
    w.update(sampler=sampler, mala_h=h)
    bad = torch.tensor([5, per - 1, per, 3 * per + 2, 3 * per + 3, chains - 2])
    out = []
    for v in (cap, 3, 1):
        s = rj.Sampler(w, precision=prec)
        bad = bad.to(s.dev)
        s.n[bad] = torch.tensor([0, 1, cap + 1, -7, 2**30, 1], dtype=s.n.dtype, device=s.dev)
        marks = torch.arange(cap * 6 * 4, device=s.dev, dtype=s.verts.dtype).reshape(cap, 6, 4) + 0.5
        s.verts[:, bad] = marks
        for k in (100, 60):
            s.run(k, block=64, v_lds=v)
        torch.cuda.synchronize()
        assert torch.equal(s.verts[:, bad], marks) and s.status[bad].tolist() == [1] * 6
        assert s.status.sum() == 6
        used = torch.arange(cap, device=s.dev)[:, None] < s.n
        used[:, bad] = False
        out.append((s.n.clone(), torch.where(used[..., None], s.verts[..., :3], 0.0).clone()))
    assert out[0][0][out[0][0] < 41].max() > 8
    for n, x in out[1:]:
        assert torch.equal(n, out[0][0]) and torch.equal(x, out[0][1])
    # (s: one slot) no jumps: n stays, rows from n on are written by others
    rest = ~used
    rest[:, bad] = False
    s.verts[rest] = 0.0
    s.run(20, run=dict(n_perturb=int(w["cycle_len"])), block=64, v_lds=1)
    torch.cuda.synchronize()
    assert torch.equal(s.n, out[0][0]) and torch.equal(s.verts[:, bad], marks)
    assert (s.verts[..., :3].abs().sum(-1)[rest] > 0).sum() > chains // per
