// rj_tree.h -- the tree-coordinate move of the step kernel (included by
// rj_step.h, whose path storage and density factors it uses).
#pragma once

#include "rj_paths.h"

namespace rj {

// ---------------------------------------------------------------------------
// Tree-coordinate move of the whole path (App. "Path space coordinate
// system"; Sec. "Path proposal distribution").  Interval (k, l), l - k >= 2,
// places vertex m = (k + l) / 2 by bi-spherical coordinates (zeta, t, phi)
// about the foci f_k, f_l (cos s = tanh zeta), then splits into (k, m) and
// (m, l); the root is (0, n - 1).  The azimuth is measured in a frame handed
// down the tree: the root's is the orthonormal completion of its axis, a
// child's has e3 = the unit normal of the plane of its parent's foci and
// vertex (the parent's frame turned about the parent's axis to the parent
// vertex's azimuth, then rotated onto the child's axis) and e2 = e3 x e1.
// The move draws a von Mises-Fisher step of the end point on the sensor
// (words 4, 5, as the end-point perturbation) and Gaussian steps of variance
// mala_h / n for every (zeta, t, phi) (vertex m: one Philox block with
// counter word 3 = 2 + m), builds the proposal level by level (each vertex's
// foci and frame come from vertices of the levels above), and accepts with
//   log A = log p(y) - log p(x) + sum_m [log J_m(y) - log J_m(x)],
//   J_m = gamma^3 sech^2(zeta) / (cosh t - tanh zeta)^3.
// The coordinates are formed from unit vectors: with uA, uB the unit vectors
// from f_m to its foci, 1 + cos s = |uA + uB|^2 / 2, 1 - cos s = |uA - uB|^2 / 2
// and sin s = |uA + uB| |uA - uB| / 2, which keep their precision for nearly
// straight (s ~ pi) and nearly folded paths.
//
// Work split.  The vertex counts of a wave's chains differ (mean 6.6 and
// longest about 40 on the ragged layered batch), so a lane that walks its own
// chain's nodes and segments leaves the others waiting: 262,144 chains took
// 266 us per tree step that way.  Here the wave shares the work of its chains
// instead: at level d of the trees the items are (chain, node), 2^d per chain
// that reaches the level, 64 at a time; then the items are (chain, segment)
// over both walks of log p, and over the accepted proposals' copy-back.  The
// terms of log A are summed per chain in FP64 in the tile's leading padding
// slot, which nothing else keeps.  The walks need a chain's target, so the lanes
// of one target share theirs (share_lanes).  Where waves of 64 chains would leave
// the chip waves short, a wave owns fewer (cpw, by shared_cpw in rj_api.hip).  The
// same step takes 79 us.
// ---------------------------------------------------------------------------
// frame (e2, e3) of interval (k, l) of a path: root (uniform over the wave) ->
// onb of the axis; otherwise from the parent interval (kp, lp) and its vertex fp.
template <class R> struct Frame2 {
    V3<R> e2, e3;
};

template <class R>
__device__ __forceinline__ Frame2<R> tree_frame(bool root, V3<R> e1, V3<R> fkp, V3<R> flp, V3<R> fp) {
    Frame2<R> f;
    if (root) {
        onb(e1, f.e2, f.e3);
    } else {
        const V3<R> ep = unit_dir(fkp, flp);
        const V3<R> g = fp - fkp;
        const V3<R> c = {ep.y * g.z - ep.z * g.y, ep.z * g.x - ep.x * g.z, ep.x * g.y - ep.y * g.x};
        f.e3 = Mth<R>::rsqrt(dot(c, c)) * c;
        f.e2 = {f.e3.y * e1.z - f.e3.z * e1.y, f.e3.z * e1.x - f.e3.x * e1.z, f.e3.x * e1.y - f.e3.y * e1.x};
    }
    return f;
}

// Node m of an interval of chain c whose parent interval is (kp, lp) (the
// interval itself at the root) and lies right or left of its vertex: the
// coordinates of x_m, the proposed ones, y_m, and log J(y) - log J(x).
template <class R>
__device__ __forceinline__ void tree_node(const WaveChain<R>& c, const StepCtx& sc, uint64_t step, R sig, bool root,
                                          bool right, int kp, int lp, int m) {
    const int pm = (kp + lp) >> 1;
    V3<R> xv[4], yv[3];
    {
        const int vx[4] = {kp, lp, pm, m}, vy[3] = {kp, lp, pm};
        c.xs(vx, xv);
        c.ys(vy, yv);
    }
    const V3<R> xkp = xv[0], xlp = xv[1], xpm = xv[2], xm = xv[3];
    const V3<R> ykp = yv[0], ylp = yv[1], ypm = yv[2]; // (the root's own vertex, not placed yet, is not used)
    // the foci: the parent's vertex and one of its foci
    auto pick3 = [](bool s, V3<R> a, V3<R> b) __attribute__((always_inline)) {
        return V3<R>{s ? a.x : b.x, s ? a.y : b.y, s ? a.z : b.z};
    };
    const V3<R> xk = pick3(!root && right, xpm, xkp), xl = pick3(root || right, xlp, xpm);
    const V3<R> yk = pick3(!root && right, ypm, ykp), yl = pick3(root || right, ylp, ypm);
    double lj = 0.0;
    // current coordinates of x_m
    const V3<R> rx = xl - xk;
    const R gx = (R)0.5 * Mth<R>::sqrt(dot(rx, rx));
    const V3<R> e1x = ((R)0.5 * Mth<R>::rcp(gx)) * rx;
    const Frame2<R> fx = tree_frame(root, e1x, xkp, xlp, xpm);
    const V3<R> e2x = fx.e2, e3x = fx.e3;
    const V3<R> va = xk - xm, vb = xl - xm;
    const R dA = Mth<R>::sqrt(dot(va, va)), dB = Mth<R>::sqrt(dot(vb, vb));
    const V3<R> ua = Mth<R>::rcp(dA) * va, ub = Mth<R>::rcp(dB) * vb;
    const V3<R> sp = ua + ub, sm = ua - ub;
    const R np2 = dot(sp, sp), nm2 = dot(sm, sm);
    const R zeta = (R)0.5 * Mth<R>::log(np2 * Mth<R>::rcp(nm2));
    const R tt = Mth<R>::log(dA * Mth<R>::rcp(dB));
    const V3<R> q = xm - (R)0.5 * (xk + xl);
    const R phi = atan2(dot(q, e3x), dot(q, e2x));
    // log J(x): sech zeta = sin s, cosh t - tanh zeta = (dA - dB)^2 / (2 dA dB) + (1 - cos s)
    const R dd = dA - dB;
    const R denx = dd * dd * Mth<R>::rcp((R)2 * dA * dB) + (R)0.5 * nm2;
    lj -= (double)((R)3 * Mth<R>::log(gx) + Mth<R>::log((R)0.25 * np2 * nm2) - (R)3 * Mth<R>::log(denx));
    // proposed coordinates
    uint32_t qd[4] = {c.W.chain0 + (uint32_t)c.q, (uint32_t)step, (uint32_t)(step >> 32), 2u + (uint32_t)m};
    philox4x32_10(qd, sc.k0, sc.k1);
    V3<R> xi;
    box_muller3<R>(qd[0], qd[1], qd[2], qd[3], xi);
    const R z2 = zeta + sig * xi.x, t2 = tt + sig * xi.y, p2 = phi + sig * xi.z;
    // y_m from its (already placed) foci and frame
    const V3<R> ry = yl - yk;
    const R gy = (R)0.5 * Mth<R>::sqrt(dot(ry, ry));
    const V3<R> e1y = ((R)0.5 * Mth<R>::rcp(gy)) * ry;
    const Frame2<R> fy = tree_frame(root, e1y, ykp, ylp, ypm);
    const V3<R> e2y = fy.e2, e3y = fy.e3;
    // tanh and sech of zeta and cosh t - tanh zeta without cancellation
    const R az = fabs(z2);
    const R ez = Mth<R>::exp((R)-2 * az);
    const R th = copysign(((R)1 - ez) * Mth<R>::rcp((R)1 + ez), z2);
    const R sh = (R)2 * Mth<R>::sqrt(ez) * Mth<R>::rcp((R)1 + ez);
    const R et = Mth<R>::exp(t2), iet = Mth<R>::rcp(et);
    const R sht = (R)0.5 * (et - iet);
    const R s2h = sht * sht * Mth<R>::rcp((R)0.5 * (et + iet) + (R)1); // cosh t - 1 = sinh^2 t / (cosh t + 1)
    const R omt = z2 > (R)0 ? (R)2 * ez * Mth<R>::rcp((R)1 + ez) : (R)1 - th; // 1 - tanh zeta
    const R deny = s2h + omt;
    const V3<R> dir = sht * e1y + sh * (Mth<R>::cos2pi(p2 * (R)0.15915494309189534) * e2y +
                                        Mth<R>::sin2pi(p2 * (R)0.15915494309189534) * e3y);
    const V3<R> ym = (R)0.5 * (yk + yl) + (gy * Mth<R>::rcp(deny)) * dir;
    lj += (double)((R)3 * Mth<R>::log(gy) + (R)2 * Mth<R>::log(sh) - (R)3 * Mth<R>::log(deny));
    c.W.sty(c.at + m, Vtx<R>{ym.x, ym.y, ym.z, (R)0});
    c.W.add(c.q, lj);
}

// The move of every chain of the wave (all 64 lanes call it together).
template <class R>
__device__ __forceinline__ void tree_move(const Tgt<R>& T, const PathRef<R, false>& ps, const WavePaths<R>& W,
                                          Lane<R>& ln, const StepCtx& sc, uint64_t step, const uint32_t r[8], R logu,
                                          int& accepted, R& logA) {
    const int n = ln.n, lane = W.lane;
    const bool act = ln.live;
    const V3<R> x0 = ps.p(0), xe = ps.p(n - 1);
    const WavePlaces P = wave_places<R>(W, act ? n : 0);
    const int at = P.at, all = P.all;
    // end point: von Mises-Fisher step about the current sensor normal
    V3<R> yend;
    {
        const R u4 = unif<R>(r[4]), u5 = unif<R>(r[5]);
        const R lg = Mth<R>::log(u4 + ((R)1 - u4) * (R)sc.e2k);
        const V3<R> dd = from_eta(T, xe);
        const V3<R> nu = Mth<R>::rsqrt(dot(dd, dd)) * dd;
        V3<R> e2, e3;
        onb(nu, e2, e3);
        const R omw = -lg * (R)sc.ikappa;
        const R sw = Mth<R>::sqrt(fmax(omw * ((R)2 - omw), (R)0));
        const V3<R> nn = ((R)1 - omw) * nu + sw * (Mth<R>::cos2pi(u5) * e2 + Mth<R>::sin2pi(u5) * e3);
        yend = T.eta + (T.eta_lo + T.rad * nn);
    }
    if (act) {
        *W.sum(lane) = 0.0;
        W.sty(at, Vtx<R>{x0.x, x0.y, x0.z, (R)0});
        W.sty(at + n - 1, Vtx<R>{yend.x, yend.y, yend.z, (R)0});
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    const R sig = Mth<R>::sqrt((R)sc.mala_h / (R)n);
    const int N = act ? n - 1 : 0; // segments
    // levels: a chain reaches level d if N > 2^d (it then has nodes there)
    for (int d = 0;; ++d) {
        const bool on = N > 0 && ((N - 1) >> d) != 0;
        const uint64_t mask = __ballot(on);
        if (mask == 0) break;
        const int cnt = __popcll(mask);
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
        // lane r: the lane of the r-th such chain
        const int nth = __builtin_amdgcn_ds_permute(4 * (on ? rank : cnt + lane - rank), lane);
        const int total = cnt << d;
        for (int base = 0; base < total; base += WAVE) {
            const int i = base + lane;
            const int q = __shfl(nth, (i >> d) & (WAVE - 1), WAVE);
            const WaveChain<R> cq{W, q, __shfl(at, q, WAVE)};
            const int nq = __shfl(n, q, WAVE);
            const R sq = __shfl(sig, q, WAVE);
            // interval of node i mod 2^d: left or right halves from the root, by its bits
            int k = 0, l = nq - 1, kp = 0, lp = nq - 1;
            bool right = false;
            for (int e = d - 1; e >= 0; --e) {
                const int mid = (k + l) >> 1;
                kp = k;
                lp = l;
                right = ((i >> e) & 1) != 0;
                k = right ? mid : k;
                l = right ? l : mid;
            }
            if (i < total && l - k >= 2) tree_node<R>(cq, sc, step, sq, d == 0, right, kp, lp, (k + l) >> 1);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    }
    // log p(y) - log p(x): the segments, by the lanes of the same target
    WaveItems it;
    it.init(lane, N, W.run);
    while (it.more()) {
        int q, k;
        const bool has = it.next(q, k);
        const WaveChain<R> cq{W, q, __shfl(at, q, WAVE)};
        const int nq = __shfl(n, q, WAVE);
        if (has) {
            const int v[3] = {k, k + 1, k + 2 < nq ? k + 2 : k + 1};
            V3<R> x[3], y[3];
            cq.xs(v, x);
            cq.ys(v, y);
            R tx, ty;
            const double a = walk_term<R, false>(T, nq, k, x[0], x[1], x[2], tx);
            const double b = walk_term<R, false>(T, nq, k, y[0], y[1], y[2], ty);
            W.styw(cq.at + k, ty);
            W.add(q, b - a);
        }
    }
    settle_shared<R>(W, P, ln, act, logu, accepted, logA);
}

} // namespace rj
