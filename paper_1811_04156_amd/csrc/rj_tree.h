// rj_tree.h -- the tree-coordinate move of the step kernel (included by
// rj_step.h, whose path storage and density factors it uses).
#pragma once

#include "rj_wave.h"

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
// slot, which nothing else keeps.  The walks use the
// lane's own target, so a wave with several targets walks its chains lane by
// lane.  With fewer chains than two waves per SIMD a wave owns fewer than 64
// chains (cpw), so that more waves share the work.
//
// Storage.  Neighbouring lanes work on neighbouring vertices of one chain, so
// the proposals are kept chain after chain without gaps (a wave's chains need
// the sum of their n, not 64 times the longest), the first My vertices in LDS
// and the rest in the wave's part of the work buffer; the vertices of the paths
// beyond their LDS slots, which lie 16 n_chains bytes apart, are copied behind
// them in the same order first.  (Read in place, one cache line per vertex
// and read, the two-region test's 80-vertex paths kept the waves waiting for
// 75% of their cycles.)
// ---------------------------------------------------------------------------
template <class R> struct WavePaths {
    LdsPtr<R> x, y;    // paths: slot 0 of column 0 of the wave's tile (stride WAVE); proposals: LDS vertex 0
    Vtx<R>* gx;        // vertex 0 of the wave's first chain
    Vtx<R>* part;      // the wave's part of the work buffer (cap vertices per chain)
    int V, My, ymask;  // LDS vertex i of the proposals is y[i + (i & ymask)]
    int cpw;           // chains of the wave (a power of two; the last wave may have fewer)
    int room;          // vertices of the wave's part
    size_t C;
    uint32_t chain0;   // the wave's first chain
    int lane;

    __device__ __forceinline__ Vtx<R> ldy(int i) const {
        if (i < My) return lds_ld<R>(y + (i + (i & ymask)));
        return part[i];
    }
    __device__ __forceinline__ void sty(int i, const Vtx<R>& p) const {
        if (i < My) lds_st<R>(y + (i + (i & ymask)), p);
        else part[i] = p;
    }
    __device__ __forceinline__ void styw(int i, R w) const {
        if (i < My) ((LdsScalar<R>)(y + (i + (i & ymask))))[3] = w;
        else part[i].w = w;
    }
    // the chain's FP64 sums (padding slot -1 holds two)
    __device__ __forceinline__ LdsScalar<double> sum(int q) const { return (LdsScalar<double>)(x - WAVE + q); }
    __device__ __forceinline__ void add(int q, double v, int k = 0) const {
        __hip_atomic_fetch_add(sum(q) + k, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};

// Chain q of the wave during a move: its first vertex's place `at` among the
// wave's proposals, and the offset of the copied paths (0: not copied).
template <class R> struct WaveChain {
    const WavePaths<R>& W;
    int q, at, copy;
    __device__ __forceinline__ V3<R> x(int v) const {
        if (v < W.V) return pos(lds_ld<R>(W.x + v * WAVE + q));
        return far_x(v);
    }
    __device__ __forceinline__ V3<R> far_x(int v) const {
        const Vtx<R>* const p = copy ? W.part + (copy + at + v) : W.gx + ((size_t)v * W.C + q);
        const L4<R> g = *(const L4<R>*)p;
        return {g.x, g.y, g.z};
    }
    __device__ __forceinline__ V3<R> y(int v) const { return pos(W.ldy(at + v)); }
    // Several vertices at once: LDS reads for all (the ones that lie elsewhere
    // read some slot), then one branch that fetches those together.
    template <int K> __device__ __forceinline__ void xs(const int (&v)[K], V3<R> (&o)[K]) const {
        int hi = v[0];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            o[i] = pos(lds_ld<R>(W.x + (v[i] < W.V ? v[i] : W.V) * WAVE + q));
            hi = max(hi, v[i]);
        }
        if (hi >= W.V) {
            V3<R> g[K];
#pragma unroll
            for (int i = 0; i < K; ++i) g[i] = far_x(v[i]);
#pragma unroll
            for (int i = 0; i < K; ++i)
                if (v[i] >= W.V) o[i] = g[i];
        }
    }
    template <int K> __device__ __forceinline__ void ys(const int (&v)[K], V3<R> (&o)[K]) const {
        int hi = v[0];
#pragma unroll
        for (int i = 0; i < K; ++i) hi = max(hi, v[i]);
        if (W.My > 0) { // (uniform)
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const int j = min(at + v[i], W.My - 1);
                o[i] = pos(lds_ld<R>(W.y + (j + (j & W.ymask))));
            }
        }
        if (at + hi >= W.My) {
            V3<R> g[K];
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const L4<R> p = *(const L4<R>*)(W.part + (at + v[i]));
                g[i] = {p.x, p.y, p.z};
            }
#pragma unroll
            for (int i = 0; i < K; ++i)
                if (at + v[i] >= W.My) o[i] = g[i];
        }
    }
};

// One chain's path or proposal as the log p walk of a single lane reads it.
template <class R, bool Y> struct LanePath {
    WaveChain<R> c;
    __device__ __forceinline__ V3<R> p(int v) const { return Y ? c.y(v) : c.x(v); }
    __device__ __forceinline__ void stw(int v, R t) const {
        if (Y) c.W.styw(c.at + v, t);
    }
};

// frame (e2, e3) of interval (k, l) of a path: root -> onb of the axis;
// otherwise from the parent interval (kp, lp) and its vertex fp.  Both are
// formed and one is selected by value (a choice between output references
// would become a dynamically indexed stack slot).
template <class R> struct Frame2 {
    V3<R> e2, e3;
};

template <class R>
__device__ __forceinline__ Frame2<R> tree_frame(bool root, V3<R> e1, V3<R> fkp, V3<R> flp, V3<R> fp) {
    V3<R> r2, r3;
    onb(e1, r2, r3);
    const V3<R> ep = unit_dir(fkp, flp);
    const V3<R> g = fp - fkp;
    const V3<R> c = {ep.y * g.z - ep.z * g.y, ep.z * g.x - ep.x * g.z, ep.x * g.y - ep.y * g.x};
    const V3<R> c3 = Mth<R>::rsqrt(dot(c, c)) * c;
    const V3<R> c2 = {c3.y * e1.z - c3.z * e1.y, c3.z * e1.x - c3.x * e1.z, c3.x * e1.y - c3.y * e1.x};
    Frame2<R> f;
    f.e2 = {root ? r2.x : c2.x, root ? r2.y : c2.y, root ? r2.z : c2.z};
    f.e3 = {root ? r3.x : c3.x, root ? r3.y : c3.y, root ? r3.z : c3.z};
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
                                          bool one_target, int& accepted, R& logA) {
    const int n = ln.n, lane = W.lane;
    const bool act = ln.live;
    accepted = 0;
    logA = Mth<R>::ninf();
    // (the chains' own lanes wrote the vertices beyond the LDS slots)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    const V3<R> x0 = ps.p(0), xe = ps.p(n - 1);
    // the chains' places among the wave's vertices, and the paths' copy
    const int mine = act ? n : 0;
    const int upto = wave_prefix(mine), at = upto - mine;
    const int all = __builtin_amdgcn_readlane(upto, WAVE - 1);
    const int copy = 2 * all <= W.room && __any(mine > W.V) ? all : 0;
    if (copy) {
        // row by row, lanes over the wave's chains (whole cache lines), four rows in flight
        const int q = lane & (W.cpw - 1), rows = WAVE / W.cpw;
        const int nq = __shfl(mine, q, WAVE), to = copy + __shfl(at, q, WAVE);
        for (int v = W.V + lane / W.cpw; __any(v < nq); v += 4 * rows) {
            L4<R> g[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (v + i * rows < nq) g[i] = *(const L4<R>*)(W.gx + ((size_t)(v + i * rows) * W.C + q));
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (v + i * rows < nq) *(L4<R>*)(W.part + (to + v + i * rows)) = g[i];
        }
    }
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
            const WaveChain<R> cq{W, q, __shfl(at, q, WAVE), copy};
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
    // log p(y) - log p(x)
    if (one_target) {
        // items: the segments of all chains in order
        WaveItems it;
        it.init(lane, N);
        while (it.more()) {
            int q, k;
            const bool has = it.next(q, k);
            const WaveChain<R> cq{W, q, __shfl(at, q, WAVE), copy};
            const int nq = __shfl(n, q, WAVE);
            if (has) {
                const int v[3] = {k, k + 1, k + 2 < nq ? k + 2 : k + 1};
                V3<R> x[3], y[3];
                cq.xs(v, x);
                cq.ys(v, y);
                R tx, ty;
                const double a = walk_term(T, nq, k, x[0], x[1], x[2], tx);
                const double b = walk_term(T, nq, k, y[0], y[1], y[2], ty);
                W.styw(cq.at + k, ty);
                W.add(q, b - a);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    } else if (act) {
        double L;
        const WaveChain<R> c{W, lane, at, copy};
        const double lpx = full_logp(T, LanePath<R, false>{c}, n, L);
        const double lpy = full_logp(T, LanePath<R, true>{c}, n, L);
        *W.sum(lane) += lpy - lpx;
    }
    if (act) {
        const double la = *W.sum(lane);
        logA = isfinite(la) ? (R)la : Mth<R>::ninf();
        accepted = logu < logA ? 1 : 0;
        // (the sums of the accepted proposal's length and depths next)
        W.sum(lane)[0] = 0.0;
        W.sum(lane)[1] = 0.0;
    }
    // the accepted proposals, with the depths their walk left
    WaveItems it;
    it.init(lane, accepted ? n : 0);
    while (it.more()) {
        int q, k;
        const bool has = it.next(q, k);
        const int aq = __shfl(at, q, WAVE), nq = __shfl(n, q, WAVE);
        if (has) {
            Vtx<R> f = W.ldy(aq + k);
            if (k < nq - 1) {
                const V3<R> d = pos(W.ldy(aq + k + 1)) - pos(f);
                const R l2 = dot(d, d);
                const R len = l2 * Mth<R>::rsqrt(l2);
                W.add(q, (double)len, 0);
                W.add(q, (double)f.w, 1);
            } else {
                f.w = (R)0;
            }
            if (k < W.V) lds_st<R>(W.x + k * WAVE + q, f);
            else W.gx[(size_t)k * W.C + q] = f;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    if (accepted) {
        ln.L = W.sum(lane)[0];
        ln.S = W.sum(lane)[1];
    }
}

} // namespace rj
