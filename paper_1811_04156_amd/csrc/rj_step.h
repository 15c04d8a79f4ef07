// rj_step.h -- the fused reversible-jump step kernel for gfx950 (templates;
// instantiated per precision and sampler in the rj_run_*.hip units).
//
// One chain per lane.  A block owns a tile of chains for every step of the
// launch.  The first V vertices of each chain live in LDS in a vertex-major,
// lane-minor layout ([slot][lane]: per-lane random slots stay conflict-free),
// the rest stay in the caller's HBM array (same [v][C] layout, read and
// written coalesced at launch start and end; the samplers of whole-path moves keep
// them chain after chain in the work buffer meanwhile, rj_paths.h).  When every lane of a wave fits
// its LDS slots (a wave vote per step) the step runs a branch-free LDS-only
// instantiation.  Layered media are staged in LDS once per block; a
// homogeneous medium lives in registers.
//
// Every step of a launch is the same move class for all lanes (the move
// schedule depends only on the global step index), so waves diverge only
// inside a class: interior and end-point perturbations share one
// local-density evaluator, births and deaths share one jump evaluator.
//
// Method references: path density (App. "Path probability distribution"),
// jump proposal and bi-spherical map (App. "Jump proposal", "Dimension
// matching transformation"), acceptance (eq. acceptFact read in Green's
// form), end-point move on the sensor and proposal mix (Sec. "Path proposal
// distribution"); the Langevin move follows the Discussion's suggestion of
// gradient-informed moves.
#pragma once

#include <hip/hip_runtime.h>

#include "rj_device.h"
#include "rj_kernels.h"

namespace rj {

enum { MV_INTERIOR = 0, MV_END = 1, MV_BIRTH = 2, MV_DEATH = 3, MV_MALA = 4, MV_NULL = 5, MV_LMALA = 6, MV_TREE = 7 };

// Interior-vertex move of the sampler (RJPATH_PLAIN / _MALA / _LMALA / _TREE).
enum { SAMP_PLAIN = 0, SAMP_JOINT = 1, SAMP_LOCAL = 2, SAMP_TREE = 3 };

// Lane-private path storage: slots below V in LDS, the rest in HBM.  LO: the
// whole path is known to be in LDS.  The LDS side is addressed through an
// address-space-3 pointer to a 4-vector, so that every access is one ds_*
// instruction (never a generic flat access).
template <class R> using L4 = R __attribute__((ext_vector_type(4)));
template <class R> using LdsPtr = __attribute__((address_space(3))) L4<R>*;
template <class R> using LdsScalar = __attribute__((address_space(3))) R*;

template <class R> __device__ __forceinline__ Vtx<R> lds_ld(LdsPtr<R> p) {
    const L4<R> q = *p;
    return Vtx<R>{q.x, q.y, q.z, q.w};
}
template <class R> __device__ __forceinline__ void lds_st(LdsPtr<R> p, const Vtx<R>& x) { *p = L4<R>{x.x, x.y, x.z, x.w}; }

// LDS layout: each wave owns a tile of V + 2 slots of 64 lanes, slot -1 and
// slot V being padding, so that a slot stride is a constant (64 vertices) and
// the LDS-only step can read the neighbours of a vertex (slots -1 .. n + 1,
// n < V) without clamping their indices: the padding or stale slots it then
// reads are only ever discarded.
constexpr int WAVE = 64;
constexpr int SLOT_PAD = 2;

template <class R, bool LO> struct PathRef {
    LdsPtr<R> lds; // this lane's slot 0, stride WAVE
    Vtx<R>* glb;   // this chain's vertex 0, stride C
    int V;
    size_t C;
    __device__ __forceinline__ Vtx<R> ld(int v) const {
        if (LO || v < V) return lds_ld<R>(lds + v * WAVE);
        return glb[(size_t)v * C];
    }
    __device__ __forceinline__ void st(int v, const Vtx<R>& x) const {
        if (LO || v < V) lds_st<R>(lds + v * WAVE, x);
        else glb[(size_t)v * C] = x;
    }
    __device__ __forceinline__ V3<R> p(int v) const { return pos(ld(v)); }
    __device__ __forceinline__ R w(int v) const {
        if (LO || v < V) return ((LdsScalar<R>)(lds + v * WAVE))[3];
        return glb[(size_t)v * C].w;
    }
    __device__ __forceinline__ R lds_w(int v) const { return ((LdsScalar<R>)(lds + v * WAVE))[3]; }
    __device__ __forceinline__ void stw(int v, R x) const {
        if (LO || v < V) ((LdsScalar<R>)(lds + v * WAVE))[3] = x;
        else glb[(size_t)v * C].w = x;
    }
    // Five vertices at once.  LDS-only: five reads.  Otherwise five LDS
    // reads (the indices that lie in HBM read the padding slot V instead)
    // and, for the lanes whose five reach HBM, one branch that reads all five
    // from HBM and keeps those (no branch per vertex on the address space).
    __device__ __forceinline__ void ld5(int i0, int i1, int i2, int i3, int i4, Vtx<R>& o0, Vtx<R>& o1, Vtx<R>& o2,
                                        Vtx<R>& o3, Vtx<R>& o4) const {
        const int c0 = LO || i0 < V ? i0 : V, c1 = LO || i1 < V ? i1 : V, c2 = LO || i2 < V ? i2 : V;
        const int c3 = LO || i3 < V ? i3 : V, c4 = LO || i4 < V ? i4 : V;
        o0 = lds_ld<R>(lds + c0 * WAVE);
        o1 = lds_ld<R>(lds + c1 * WAVE);
        o2 = lds_ld<R>(lds + c2 * WAVE);
        o3 = lds_ld<R>(lds + c3 * WAVE);
        o4 = lds_ld<R>(lds + c4 * WAVE);
        if (LO) return;
        const int hi = max(max(max(i0, i1), max(i2, i3)), i4);
        if (hi >= V) {
            const L4<R>* const g = (const L4<R>*)glb;
            const L4<R> g0 = g[(size_t)i0 * C], g1 = g[(size_t)i1 * C], g2 = g[(size_t)i2 * C];
            const L4<R> g3 = g[(size_t)i3 * C], g4 = g[(size_t)i4 * C];
            if (i0 >= V) o0 = Vtx<R>{g0.x, g0.y, g0.z, g0.w};
            if (i1 >= V) o1 = Vtx<R>{g1.x, g1.y, g1.z, g1.w};
            if (i2 >= V) o2 = Vtx<R>{g2.x, g2.y, g2.z, g2.w};
            if (i3 >= V) o3 = Vtx<R>{g3.x, g3.y, g3.z, g3.w};
            if (i4 >= V) o4 = Vtx<R>{g4.x, g4.y, g4.z, g4.w};
        }
    }
    // The vertex shift of an accepted jump: slots lo..hi move one up (from the
    // top), or slots lo+1..hi+1 one down (from the bottom).  In LDS births and
    // deaths share one loop, which reads SHIFT vertices before it writes them
    // and past the last one moves that one again: the wave waits once per
    // SHIFT vertices of its longest shift.  (A loop for each, four vertices at
    // a time and then one at a time: a jump step of 65,536 homogeneous chains
    // took 3.55 us and takes 3.05.)
    static constexpr int SHIFT = 6;
    __device__ __forceinline__ void shift(bool up, int lo, int hi) const {
        if (!LO && up) far_up(lo, hi);
        const int top = LO || hi < V - 2 ? hi : V - 2; // the moves that stay in LDS
        const int dir = up ? -1 : 1;
        for (int left = top - lo, v = up ? top : lo + 1; left >= 0; left -= SHIFT, v += dir * SHIFT) {
            L4<R> x[SHIFT];
            LdsPtr<R> at[SHIFT];
#pragma unroll
            for (int i = 0; i < SHIFT; ++i) at[i] = lds + (v + dir * (i < left ? i : left)) * WAVE;
#pragma unroll
            for (int i = 0; i < SHIFT; ++i) x[i] = *at[i];
#pragma unroll
            for (int i = 0; i < SHIFT; ++i) at[i][-dir * WAVE] = x[i];
        }
        if (!LO && !up) far_down(lo, hi);
    }
    // The moves to and beyond slot V, one way each (in one loop for both, with
    // the LDS ones, a jump step of the two-region test took 76 us instead of 65).
    __device__ __forceinline__ void far_up(int lo, int hi) const {
        int v = hi;
        L4<R>* const g = (L4<R>*)glb;
        for (; v - 3 >= lo && v - 3 >= V; v -= 4) {
            const L4<R> a = g[(size_t)v * C], b = g[(size_t)(v - 1) * C], c = g[(size_t)(v - 2) * C],
                        d = g[(size_t)(v - 3) * C];
            g[(size_t)(v + 1) * C] = a;
            g[(size_t)v * C] = b;
            g[(size_t)(v - 1) * C] = c;
            g[(size_t)(v - 2) * C] = d;
        }
        for (; v >= lo && v >= V; --v) g[(size_t)(v + 1) * C] = g[(size_t)v * C];
        if (v >= lo && v == V - 1) g[(size_t)V * C] = lds[v * WAVE];
    }
    __device__ __forceinline__ void far_down(int lo, int hi) const {
        int v = lo > V - 1 ? lo : V - 1;
        L4<R>* const g = (L4<R>*)glb;
        if (v <= hi && v == V - 1) {
            lds[v * WAVE] = g[(size_t)V * C];
            ++v;
        }
        for (; v + 3 <= hi; v += 4) {
            const L4<R> a = g[(size_t)(v + 1) * C], b = g[(size_t)(v + 2) * C], c = g[(size_t)(v + 3) * C],
                        d = g[(size_t)(v + 4) * C];
            g[(size_t)v * C] = a;
            g[(size_t)(v + 1) * C] = b;
            g[(size_t)(v + 2) * C] = c;
            g[(size_t)(v + 3) * C] = d;
        }
        for (; v <= hi; ++v) g[(size_t)v * C] = g[(size_t)(v + 1) * C];
    }
};

// Full log p of the path (FP64 sum of the factors), refreshing the cached
// segment scattering depths; also returns the path length L and, where Sb is
// given, the FP64 sum of the refreshed depths in path order.
template <class R, class P>
__device__ __forceinline__ double full_logp(const Tgt<R>& T, const P& ps, int n, double& L, double* Sb = nullptr) {
    V3<R> f0 = ps.p(0), f1 = ps.p(1);
    LPt<R> lc = lpt(T, f1);
    Seg<R> s = make_seg_lp(T, f0, f1, lpt(T, f0), lc);
    bool zero = !(s.len > (R)0);
    double lp = (double)emit_term(T, s.u) + (double)seg_term(s);
    L = (double)s.len;
    double sb = (double)s.tb;
    ps.stw(0, s.tb);
    V3<R> fc = f1;
    for (int k = 1; k <= n - 2; ++k) {
        V3<R> fn = ps.p(k + 1);
        const LPt<R> lnx = lpt(T, fn);
        Seg<R> s2 = make_seg_lp(T, fc, fn, lc, lnx);
        zero |= !(s2.len > (R)0);
        const LayV<R> ly = lay_at(T, lc.l);
        lp += (double)(ly.logb + turn_term(ly, s.u, s2.u)) + (double)seg_term(s2);
        L += (double)s2.len;
        sb += (double)s2.tb;
        ps.stw(k, s2.tb);
        s = s2;
        fc = fn;
        lc = lnx;
    }
    lp += (double)end_term(T, s.u, fc);
    if (zero) lp = -__builtin_inf();
    if (Sb) *Sb = sb;
    return lp;
}

// The factors of log p that belong to segment k of a path of n vertices (the
// segment, the emission at k = 0, the turn or the end at vertex k + 1), as
// full_logp forms them; -inf where the segment or the next one, whose direction
// the turn needs, has no length, so that the sum over a path with such a segment
// is -inf, as full_logp's, and never NaN.  (NEXT false: NaN there; for a proposal,
// which is rejected either way, 1% of a tree step.)
template <class R, bool NEXT = true>
__device__ __forceinline__ double walk_term(const Tgt<R>& T, int n, int k, V3<R> f0, V3<R> f1, V3<R> f2, R& tb) {
    const LPt<R> l0 = lpt(T, f0), l1 = lpt(T, f1);
    const Seg<R> s = make_seg_lp(T, f0, f1, l0, l1);
    tb = s.tb;
    double t = (double)seg_term(s);
    if (k == 0) t += (double)emit_term(T, s.u);
    bool length = s.len > (R)0;
    if (k <= n - 3) {
        const LayV<R> ly = lay_at(T, l1.l);
        const V3<R> r = f2 - f1;
        const R l2 = dot(r, r), il = Mth<R>::rsqrt(l2);
        t += (double)(ly.logb + turn_term(ly, s.u, il * r));
        if (NEXT) length &= l2 * il > (R)0;
    } else {
        t += (double)end_term(T, s.u, f1);
    }
    return length ? t : -__builtin_inf();
}

// q(s) of the bi-spherical proposal with concentration beta, in the two
// forms the jump needs: E = e^{-2 beta}, the normaliser
// log((1 - E) / beta) = log(2 sinh(beta) / beta) - beta, and the inverse CDF
// of cos s written as w = 1 + cos s = -log(u' + (1 - u') E) / beta with
// u' = 1 - u.  For beta >= 1/4 the direct forms lose nothing (1 - E > 0.39);
// below that the expm1 / log1p forms are used.
template <class R> struct QS {
    R beta, E, ibeta, lnorm;
    bool small;
};

template <class R> __device__ __forceinline__ QS<R> make_qs(R beta) {
    QS<R> q;
    q.beta = beta;
    R ab = beta < (R)0 ? -beta : beta;
    q.small = ab < (R)0.25;
    q.E = Mth<R>::exp((R)-2 * beta);
    q.ibeta = Mth<R>::rcp(beta);
    if (!q.small) {
        q.lnorm = Mth<R>::log(((R)1 - q.E) * q.ibeta);
    } else if (ab < (R)1e-6) {
        q.lnorm = (R)0.69314718055994530942 - beta;
    } else {
        q.lnorm = Mth<R>::log(-Mth<R>::expm1((R)-2 * beta) * q.ibeta);
    }
    return q;
}

// 1 + cos s from the uniform u (inverse CDF of q(s))
template <class R> __device__ __forceinline__ R qs_sample(const QS<R>& q, R u) {
    R up = (R)1 - u;
    if (!q.small) return -Mth<R>::log(u + up * q.E) * q.ibeta;
    R ab = q.beta < (R)0 ? -q.beta : q.beta;
    if (ab < (R)1e-6) return (R)2 * up;
    return -Mth<R>::log1p(up * Mth<R>::expm1((R)-2 * q.beta)) * q.ibeta;
}

template <class R>
__device__ __forceinline__ void box_muller3(uint32_t a, uint32_t b, uint32_t c, uint32_t d, V3<R>& xi) {
    R u0 = unif<R>(a), u1 = unif<R>(b), u2 = unif<R>(c), u3 = unif<R>(d);
    R rho1 = Mth<R>::sqrt((R)-2 * Mth<R>::log(u0));
    R rho2 = Mth<R>::sqrt((R)-2 * Mth<R>::log(u2));
    xi = {rho1 * Mth<R>::cos2pi(u1), rho1 * Mth<R>::sin2pi(u1), rho2 * Mth<R>::cos2pi(u3)};
}

// d tau_c / d P and d tau_c / d Q of a segment with the endpoints' layer
// points known: the mean coefficient along the segment, plus the change of
// the layers' shares where it crosses edges.
template <class R>
__device__ __forceinline__ void seg_depth_grad_lp(const Tgt<R>& T, LPt<R> P, LPt<R> Q, const Seg<R>& s, V3<R>& dP,
                                                  V3<R>& dQ) {
    R F = s.tc * Mth<R>::rcp(s.len); // mean total coefficient along the segment
    dP = (-F) * s.u;
    dQ = F * s.u;
    if (!T.hom && P.l != Q.l) {
        double cP = (double)T.lay[P.l * LY_NW + LY_C], cQ = (double)T.lay[Q.l * LY_NW + LY_C];
        const double du = (double)Q.u - (double)P.u;
        const double inv = du != 0.0 ? 1.0 / du : 0.0;
        R gP = (R)((double)s.len * ((double)F - cP) * inv);
        R gQ = (R)((double)s.len * (cQ - (double)F) * inv);
        const V3<R> ax = T.axr;
        dP = dP + gP * ax;
        dQ = dQ + gQ * ax;
    }
}

// d log sigma / d mu at a turn, q = |ua - ub|^2
template <class R> __device__ __forceinline__ R dturn_dmu(const LayV<R>& ly, R q) {
    R den = ly.hg1 + ly.g * q;
    R dhg = (R)3 * ly.g * Mth<R>::rcp(den);
    if (ly.fsl == (R)0) return dhg;
    R hg = ly.hgn - (R)1.5 * Mth<R>::log(den);
    R v = (R)1 - (R)0.25 * q; // (1 + mu) / 2
    R sl = ly.sln + ly.sla * Mth<R>::log(v);
    R dsl = ly.sla * Mth<R>::rcp((R)2 * v);
    R m = sl > hg ? sl : hg;
    R es = ly.fsl * Mth<R>::exp(sl - m), eh = ((R)1 - ly.fsl) * Mth<R>::exp(hg - m);
    return (es * dsl + eh * dhg) * Mth<R>::rcp(es + eh);
}

template <class R> __device__ __forceinline__ V3<R> dunit(V3<R> u, R len, V3<R> c) {
    // d (u . c) / d r for u = r / |r|
    R il = Mth<R>::rcp(len);
    return il * (c - dot(u, c) * u);
}

// Role of a vertex in a local density factor (see vtx_term).
enum { VK_EMIT = 0, VK_TURN = 1, VK_END = 2, VK_NONE = 3 };

// d log p / d f_j of an interior vertex j from its five-vertex window, the
// terms the single-vertex evaluator reads: the segments A = f_{j-1} -> f_j and
// B = f_j -> f_{j+1} (attenuation and inverse square), the turn at j, the turn
// at j-1 (or, for j = 1, the emission factor, which depends on the direction
// only for a von Mises-Fisher source), and the turn at j+1 (or the end factor
// log(-u . nu) when f_{j+1} is the end point).  log b(f_j) is constant within
// a layer and contributes nothing.
template <class R>
__device__ __forceinline__ V3<R> vertex_grad(const Tgt<R>& T, int km1, const LayV<R>& lm1, V3<R> um, LPt<R> pm1,
                                             LPt<R> po, LPt<R> pp1, const Seg<R>& A, const Seg<R>& B,
                                             const LayV<R>& lo, int kp1, V3<R> up, V3<R> nu1, const LayV<R>& lp1) {
    V3<R> dPA, dQA, dPB, dQB;
    seg_depth_grad_lp(T, pm1, po, A, dPA, dQA);
    seg_depth_grad_lp(T, po, pp1, B, dPB, dQB);
    V3<R> g = ((R)2 * Mth<R>::rcp(B.len)) * B.u - ((R)2 * Mth<R>::rcp(A.len)) * A.u - dQA - dPB;
    {
        const V3<R> dd = A.u - B.u;
        const R h = dturn_dmu(lo, dot(dd, dd));
        g = g + h * (dunit(A.u, A.len, B.u) - dunit(B.u, B.len, A.u));
    }
    {
        const V3<R> dd = um - A.u;
        const R ht = dturn_dmu(lm1, dot(dd, dd));
        const R he = T.ek == RJPATH_EMIT_VMF ? T.kappa : (R)0;
        const bool turn = km1 == VK_TURN;
        g = g + (turn ? ht : he) * dunit(A.u, A.len, turn ? um : T.ed);
    }
    {
        const V3<R> dd = B.u - up;
        const R ht = dturn_dmu(lp1, dot(dd, dd));
        const R ce = -dot(B.u, nu1);
        const bool turn = kp1 == VK_TURN;
        g = g + (turn ? -ht : Mth<R>::rcp(ce)) * dunit(B.u, B.len, turn ? up : nu1);
    }
    return g;
}

// log p's factors of segment k of a path of n vertices and the gradient of its
// vertex j = k + 1, with the terms in path order
// f: vertices k - 1 .. k + 3 (any value where the path has none), A: the
// segment.  -inf where walk_term gives it.
template <class R>
__device__ __forceinline__ double segment_grad(const Tgt<R>& T, int n, int k, const V3<R> (&f)[5], V3<R>& grad, Seg<R>& A) {
    const int j = k + 1;
    const V3<R> f0 = f[1], f1 = f[2];
    const LPt<R> p0 = lpt(T, f0), p1 = lpt(T, f1);
    A = make_seg_lp(T, f0, f1, p0, p1);
    double t = (double)seg_term(A);
    V3<R> dP, dQ;
    seg_depth_grad_lp(T, p0, p1, A, dP, dQ);
    const R ilA = (R)2 * Mth<R>::rcp(A.len);
    const V3<R> z = {(R)0, (R)0, (R)0};
    V3<R> g = z - dQ - ilA * A.u;
    bool length = A.len > (R)0;
    if (k == 0) {
        t += (double)emit_term(T, A.u);
        if (T.ek == RJPATH_EMIT_VMF) g = g + T.kappa * dunit(A.u, A.len, T.ed);
    } else {
        const V3<R> um = unit_dir(f[0], f0), dd = um - A.u;
        const R h = dturn_dmu(lay_at(T, p0.l), dot(dd, dd));
        g = g + h * dunit(A.u, A.len, um);
    }
    if (j < n - 1) {
        const V3<R> f2 = f[3];
        const LPt<R> p2 = lpt(T, f2);
        const Seg<R> B = make_seg_lp(T, f1, f2, p1, p2);
        length &= B.len > (R)0;
        seg_depth_grad_lp(T, p1, p2, B, dP, dQ);
        const R ilB = (R)2 * Mth<R>::rcp(B.len);
        g = g - dP + ilB * B.u;
        const LayV<R> ly = lay_at(T, p1.l);
        t += (double)(ly.logb + turn_term(ly, A.u, B.u));
        {
            const V3<R> dd = A.u - B.u;
            const R h = dturn_dmu(ly, dot(dd, dd));
            g = g + h * dunit(A.u, A.len, B.u) - h * dunit(B.u, B.len, A.u);
        }
        if (j < n - 2) {
            const V3<R> uc = unit_dir(f2, f[4]), dd = B.u - uc;
            const R h = dturn_dmu(lay_at(T, p2.l), dot(dd, dd));
            g = g - h * dunit(B.u, B.len, uc);
        } else {
            const V3<R> nu = unit_dir_eta(T, f2);
            const R ic = Mth<R>::rcp(-dot(B.u, nu));
            g = g - ic * ((R)-1 * dunit(B.u, B.len, nu));
        }
    } else {
        t += (double)end_term(T, A.u, f1);
        const V3<R> d = from_eta(T, f1);
        const R dn2 = dot(d, d), idn = Mth<R>::rsqrt(dn2);
        const V3<R> nu = idn * d;
        const R ic = Mth<R>::rcp(-dot(A.u, nu));
        const V3<R> dcr = (R)-1 * dunit(A.u, A.len, nu), dcd = (R)-1 * dunit(nu, dn2 * idn, A.u);
        g = g + ic * dcr + ic * dcd;
        if (T.dk == RJPATH_DET_PAPER) {
            const R cr = dot(nu, T.dd);
            const R th = tanh((R)2 * cr + (R)0.7);
            g = g + ((R)3 - (R)2 * th) * dunit(nu, dn2 * idn, T.dd);
        }
    }
    grad = g;
    return length ? t : -__builtin_inf();
}

// The score of one path by one lane, fed a vertex at a time: step(f_k) takes
// vertex k >= 1 and, with G, gives the gradient of vertex k - 2, finish() adds
// the end term and gives log p and the gradients of vertices n - 2 and n - 1.
// The terms and their order within a vertex are segment_grad's.
template <class R, bool G> struct PathWalk {
    V3<R> gA, gB; // gradients of vertices k - 2 and k - 1 so far
    V3<R> fprev, uprev;
    R lprev;
    LPt<R> pprev;
    double lp = 0.0;
    bool length = true; // every segment so far has one
    int k = 1;

    __device__ __forceinline__ PathWalk(const Tgt<R>& T, V3<R> f0) : fprev(f0), pprev(lpt(T, f0)) {
        gA = gB = uprev = V3<R>{(R)0, (R)0, (R)0};
        lprev = (R)0;
    }
    __device__ __forceinline__ void step(const Tgt<R>& T, V3<R> f, V3<R>& out) {
        const LPt<R> p = lpt(T, f);
        const Seg<R> s = make_seg_lp(T, fprev, f, pprev, p);
        length &= s.len > (R)0;
        lp += (double)seg_term(s);
        V3<R> gC;
        if (G) {
            V3<R> dP, dQ;
            seg_depth_grad_lp(T, pprev, p, s, dP, dQ);
            const R il = (R)2 * Mth<R>::rcp(s.len);
            const V3<R> z = {(R)0, (R)0, (R)0};
            gB = gB - dP + il * s.u;
            gC = z - dQ - il * s.u;
        }
        if (k == 1) {
            lp += (double)emit_term(T, s.u);
            if (G && T.ek == RJPATH_EMIT_VMF) gC = gC + T.kappa * dunit(s.u, s.len, T.ed);
        } else {
            const LayV<R> ly = lay_at(T, pprev.l);
            lp += (double)(ly.logb + turn_term(ly, uprev, s.u));
            if (G) {
                const V3<R> dd = uprev - s.u;
                const R h = dturn_dmu(ly, dot(dd, dd));
                const V3<R> da = dunit(uprev, lprev, s.u), db = dunit(s.u, s.len, uprev);
                gA = gA - h * da;
                gB = gB + h * da - h * db;
                gC = gC + h * db;
            }
        }
        if (G) {
            out = gA;
            gA = gB;
            gB = gC;
        }
        uprev = s.u;
        lprev = s.len;
        fprev = f;
        pprev = p;
        ++k;
    }
    __device__ __forceinline__ double finish(const Tgt<R>& T, V3<R>& g2, V3<R>& g1) {
        lp += (double)end_term(T, uprev, fprev);
        if (G) {
            const V3<R> d = from_eta(T, fprev);
            const R dn2 = dot(d, d), idn = Mth<R>::rsqrt(dn2);
            const V3<R> nu = idn * d;
            const R ic = Mth<R>::rcp(-dot(uprev, nu));
            const V3<R> dcr = (R)-1 * dunit(uprev, lprev, nu), dcd = (R)-1 * dunit(nu, dn2 * idn, uprev);
            g2 = gA - ic * dcr;
            g1 = gB + ic * dcr + ic * dcd;
            if (T.dk == RJPATH_DET_PAPER) {
                const R cr = dot(nu, T.dd);
                const R th = tanh((R)2 * cr + (R)0.7);
                g1 = g1 + ((R)3 - (R)2 * th) * dunit(nu, dn2 * idn, T.dd);
            }
        }
        return length ? lp : -__builtin_inf();
    }
};

// Per-lane constants of the step kernel.
struct StepCtx {
    uint32_t chain, k0, k1;
    int cap;
    uint32_t bthresh;
    double log_pb, log_pd; // log of the birth / death probabilities of a jump step
    double sigma, ikappa, e2k, mala_h;
    int sampler;
    const double* logw;
    uint32_t* hist; // this target's sector histogram (cap + 1 counts) or NULL
};



// log rho(nu) of the paper's angular response (0 for a uniform response)
template <class R> __device__ __forceinline__ R rho_log(const Tgt<R>& T, V3<R> nu) {
    if (T.dk != RJPATH_DET_PAPER) return (R)0;
    R cr = dot(nu, T.dd);
    R z = (R)2 * cr + (R)0.7;
    R az = z < (R)0 ? -z : z;
    // log rho = 3 c - 1 - log cosh(2 c + 0.7), log cosh z = |z| + log1p(e^{-2|z|}) - log 2
    return (R)3 * cr - (R)1 - (az + Mth<R>::log1p(Mth<R>::exp((R)-2 * az)) - (R)0.69314718055994530942);
}

// ---------------------------------------------------------------------------
// One factor of the path density attached to one vertex (App. "Path
// probability distribution"), evaluated branch-free so that lanes of a wave
// whose vertices play different roles do not diverge:
//   VK_EMIT: the source, log eps(ub) of the first direction;
//   VK_TURN: an interior vertex, log b + log sigma_sr(ua . ub);
//   VK_END:  the end point with outward sensor normal nu, log max(0, -ua . nu)
//            (the angular response log rho(nu) is added by the caller where
//            it does not cancel);
//   VK_NONE: no vertex (0).
// CE / CT / CN: whether the kinds END / EMIT / NONE can occur at the call.
// ---------------------------------------------------------------------------
template <class R, bool CE, bool CT, bool CN>
__device__ __forceinline__ R vtx_term(const Tgt<R>& T, int kind, const LayV<R>& ly, V3<R> ua, V3<R> ub, V3<R> nu) {
    V3<R> d = ua - ub;
    const R q = dot(d, d);
    R X = ly.hg1 + ly.g * q; // HG denominator, 1 - mu = |ua - ub|^2 / 2
    R ce = (R)1;
    if (CE) {
        ce = -dot(ua, nu);
        if (kind == VK_END) X = ce;
    }
    const R lx = Mth<R>::log(X);
    R out = ly.logb + ly.hgn - (R)1.5 * lx;
    if (ly.fsl != (R)0) {
        R hg = ly.hgn - (R)1.5 * lx;
        R sl = ly.sln + ly.sla * Mth<R>::log((R)1 - (R)0.25 * q);
        R m = sl > hg ? sl : hg;
        out = ly.logb + m + Mth<R>::log(ly.fsl * Mth<R>::exp(sl - m) + ((R)1 - ly.fsl) * Mth<R>::exp(hg - m));
    }
    if (CE && kind == VK_END) out = ce > (R)0 ? lx : Mth<R>::ninf();
    if (CT && kind == VK_EMIT) out = emit_term(T, ub);
    if (CN && kind == VK_NONE) out = (R)0;
    return out;
}

// The eight random words of one step: Philox4x32-10 blocks 0 and 1 of the
// counter (chain, step).  The products that depend on the chain alone are the
// same at every step and the compiler keeps them in registers; the whole-path
// moves need those registers (their walks spill otherwise) and form them again.
template <int SAMP> __device__ __forceinline__ void draw8(const StepCtx& sc, uint64_t step, uint32_t r[8]) {
    uint32_t chain = sc.chain;
    if constexpr (SAMP == SAMP_JOINT || SAMP == SAMP_TREE) asm volatile("" : "+v"(chain));
    uint32_t q0[4] = {chain, (uint32_t)step, (uint32_t)(step >> 32), 0u};
    uint32_t q1[4] = {chain, (uint32_t)step, (uint32_t)(step >> 32), 1u};
    philox4x32_10(q0, sc.k0, sc.k1);
    philox4x32_10(q1, sc.k0, sc.k1);
    r[0] = q0[0]; r[1] = q0[1]; r[2] = q0[2]; r[3] = q0[3];
    r[4] = q1[0]; r[5] = q1[1]; r[6] = q1[2]; r[7] = q1[3];
}

// ---------------------------------------------------------------------------
// Per-lane sampler state and statistics.  Counts that are the same for every
// lane (the steps of each class) are formed at the end of the launch.
// ---------------------------------------------------------------------------
template <class R> struct Lane {
    int n;
    bool live; // the chain steps (a malformed or zero-density chain keeps its state)
    double L;    // path length (running sum; refreshed at launch start)
    double S;    // sum of the cached segment scattering depths (running sum; refreshed at launch start)
    double lp;   // log p (refreshed at launch start and end)
    double invw; // 1 / w(n) of the sector tilt
    double lwm, lw0, lwp; // log w(n - 1), log w(n), log w(n + 1)
    // statistics of this launch.  The sums that depend on n alone are kept
    // lazily: the steps since `mark`, the step of the launch from which the
    // chain has had its current n, are folded in when n changes and at the
    // end of the launch.
    int mark;
    double a1, a2, sl, sl2;
    uint64_t sn;
    uint32_t cnt, c2, ncap, pb, ap, ab, ad, mp, ma;
    uint32_t ne; // jump proposals rejected without a density evaluation (birth at cap, death at n = 2)
};

// Depths that a birth's segment scan reads at once (16 cover all but rare
// long paths of the batched workloads; the FP64 and Langevin variants keep 8
// so that their registers still allow two resident waves per SIMD where they
// did).
template <class R, int SAMP> __device__ constexpr int scan_slots() {
    return (sizeof(R) == 4 && SAMP == SAMP_PLAIN) ? 16 : 8;
}

// Perturbation steps among the `count` steps from global index s0 on.
__device__ __forceinline__ uint32_t count_perturbs(uint64_t s0, uint32_t count, int cycle, int n_perturb) {
    auto upto = [&](uint64_t x) {
        const uint64_t q = x / (uint64_t)cycle, f = x % (uint64_t)cycle;
        return q * (uint64_t)n_perturb + (f < (uint64_t)n_perturb ? f : (uint64_t)n_perturb);
    };
    return (uint32_t)(upto(s0 + count) - upto(s0));
}

// The wave's place in the launch: step s of the launch (global index
// step0 + s), counted in the statistics from s >= first on.
struct StepLoop {
    uint64_t step0;
    int s, first;
    bool tilt;
    __device__ __forceinline__ bool counted() const { return s >= first; }
};

// 1 / w(n) = e^{-log w(n)} of the sector tilt, a weight of the statistics
// only: FP32 chains take it from the FP32 exponential (relative error
// ~1e-6 at log w = 40, against a 1% target), FP64 chains in FP64.
template <class R> __device__ __forceinline__ double inv_tilt(double lw) {
    if constexpr (sizeof(R) == 4) return (double)Mth<float>::exp(-(float)lw);
    else return exp(-lw);
}

// Adds the steps spent at the current n to the sums (counted steps) and to
// the sector histogram (every step of the launch).
template <class R> __device__ __forceinline__ void fold_run(Lane<R>& ln, int n0, const StepCtx& sc, const StepLoop& lp) {
    const int from = ln.mark > lp.first ? ln.mark : lp.first;
    const uint32_t r = lp.s > from ? (uint32_t)(lp.s - from) : 0u;
    const bool at0 = ln.n == n0;
    ln.cnt += r;
    ln.c2 += at0 ? r : 0u;
    ln.sn += (uint64_t)r * (uint64_t)ln.n;
    ln.ncap += ln.n == sc.cap ? r : 0u;
    if (lp.tilt) {
        const double a = (double)r * ln.invw;
        ln.a1 += a;
        ln.a2 += at0 ? a : 0.0;
    }
    if (sc.hist && lp.s > ln.mark) atomicAdd(sc.hist + ln.n, (uint32_t)(lp.s - ln.mark));
    ln.mark = lp.s;
}

// The per-step sums of a counted step, after the move.
template <class R> __device__ __forceinline__ void count_step(Lane<R>& ln) {
    ln.sl += ln.L;
    ln.sl2 += ln.L * ln.L;
}

template <class R>
__device__ __forceinline__ void put_trace(const KArgs& a, const Lane<R>& ln, int c, int s, int move, int idx, int accepted,
                                          R logA, R logu) {
    if (a.trace && ln.live) {
        double* tr = a.trace + ((size_t)c * a.trace_steps + a.trace_off + s) * RJPATH_TRACE_WORDS;
        tr[0] = move;
        tr[1] = accepted;
        tr[2] = idx;
        tr[3] = (double)logA;
        tr[4] = (double)logu;
    }
}

} // namespace rj

#include "rj_joint.h"
#include "rj_tree.h"

namespace rj {

// A perturbation step: moves interior vertex j or the end point (the joint
// Langevin sampler comes here with lanes that picked the end point).
// n does not change.  Returns the move kind, log A, the vertex and whether it
// was accepted.
template <class R, bool LO, int SAMP>
__device__ __forceinline__ void perturb_move(const Tgt<R>& T, const PathRef<R, LO>& ps, Lane<R>& ln, const StepCtx& sc,
                                             uint64_t step, const uint32_t r[8], R logu, int& move, int& idx,
                                             int& accepted, R& logA) {
    const int n = ln.n;
    idx = -1;
    accepted = 0;
    logA = Mth<R>::ninf();
    const V3<R> ex = {(R)1, (R)0, (R)0};
    const int j = 1 + pick(r[0], (uint32_t)(n - 1));
    idx = j;
    const bool is_end = SAMP == SAMP_JOINT || (j == n - 1);
    // ---------- single-vertex perturbation: the five-vertex window ----------
    const bool hm2 = j >= 2, hp1 = !is_end, hp2 = j <= n - 3;
    // slots j-2 .. j+2 (absent neighbours are replaced by stand-ins below;
    // in LDS their slots are readable as they are, elsewhere the indices
    // are clamped to stay in range)
    Vtx<R> wm2, vm1, vo, wp1, wp2;
    ps.ld5(LO || hm2 ? j - 2 : 0, j - 1, j, LO || hp1 ? j + 1 : 0, LO || hp2 ? j + 2 : 0, wm2, vm1, vo, wp1, wp2);
    const V3<R> gm2 = pos(wm2), fm1 = pos(vm1), fo = pos(vo);
    const V3<R> gp1 = pos(wp1), gp2 = pos(wp2);
    const V3<R> fm2 = hm2 ? gm2 : fm1 - ex;
    const V3<R> fp1 = hp1 ? gp1 : fo + ex;
    const V3<R> fp2 = hp2 ? gp2 : fp1 + ex;
    move = is_end ? MV_END : MV_INTERIOR;
    // layer points of the window vertices, once each; the ones near an
    // edge are settled together with the proposal's (one branch per
    // step), except that the Langevin step needs the old window first
    constexpr bool EARLY = SAMP == SAMP_LOCAL;
    bool q1, q2, q3, q4;
    LPt<R> pm1 = lpt_fast(T, fm1, q1), po = lpt_fast(T, fo, q2), pp1 = lpt_fast(T, fp1, q3);
    if constexpr (EARLY) {
        if (q1 | q2 | q3) {
            lpt_settle(T, fm1, pm1);
            lpt_settle(T, fo, po);
            lpt_settle(T, fp1, pp1);
        }
    }
    Seg<R> Ao, Bo;
    LayV<R> lm1, lo, lp1;
    auto old_window = [&]() __attribute__((always_inline)) {
        Ao = make_seg_lp(T, fm1, fo, pm1, po);
        Bo = make_seg_lp(T, fo, fp1, po, pp1);
        lm1 = lay_at(T, pm1.l);
        lo = lay_at(T, po.l);
        lp1 = lay_at(T, pp1.l);
    };
    if constexpr (EARLY) old_window();
    // the direction past f_{j+1}: of the next segment or, where f_{j+1} is the
    // end point, of the sensor normal there (a turn reads the one, an end
    // factor the other: one normalisation serves both)
    const bool fin = hp1 && !hp2;
    const V3<R> um = unit_dir(fm2, fm1);
    V3<R> up;
    {
        const V3<R> rt = fp2 - fp1, re = from_eta(T, fp1);
        const V3<R> rr = {fin ? re.x : rt.x, fin ? re.y : rt.y, fin ? re.z : rt.z};
        up = Mth<R>::rsqrt(dot(rr, rr)) * rr;
    }
    const int km1 = hm2 ? VK_TURN : VK_EMIT;
    const int kj = is_end ? VK_END : VK_TURN;
    const int kp1 = !hp1 ? VK_NONE : (hp2 ? VK_TURN : VK_END);
    // one log and one sin/cos pair serve both proposals: Box-Muller on
    // words 4..7 for the Gaussian step, and words 4, 5 for the end-point
    // von Mises-Fisher step (inverse CDF of its cosine, uniform azimuth)
    const R u4 = unif<R>(r[4]), u5 = unif<R>(r[5]);
    const R lg = Mth<R>::log(is_end ? u4 + ((R)1 - u4) * (R)sc.e2k : u4);
    const R c5 = Mth<R>::cos2pi(u5), s5 = Mth<R>::sin2pi(u5);
    V3<R> fn, nu, nn;
    R hx = (R)0, half_xi2 = (R)0;
    {
        const R rho1 = Mth<R>::sqrt((R)-2 * lg);
        const R rho2 = Mth<R>::sqrt((R)-2 * Mth<R>::log(unif<R>(r[6])));
        const V3<R> xi = {rho1 * c5, rho1 * s5, rho2 * Mth<R>::cos2pi(unif<R>(r[7]))};
        V3<R> fg;
        if constexpr (SAMP == SAMP_LOCAL) {
            // single-vertex Langevin step with h = mala_h * (shorter adjacent segment)^2
            const V3<R> gx = vertex_grad(T, km1, lm1, um, pm1, po, pp1, Ao, Bo, lo, kp1, up, up, lp1);
            const R m = fmin(Ao.len, Bo.len);
            hx = (R)sc.mala_h * m * m;
            half_xi2 = (R)0.5 * dot(xi, xi);
            fg = fo + ((R)0.5 * hx) * gx + Mth<R>::sqrt(hx) * xi;
        } else {
            fg = fo + (R)sc.sigma * xi;
        }
        V3<R> dd = from_eta(T, fo), e2, e3;
        nu = Mth<R>::rsqrt(dot(dd, dd)) * dd; // sensor normal at the current end point
        onb(nu, e2, e3);
        const R omw = -lg * (R)sc.ikappa; // 1 - cos
        const R wv = (R)1 - omw;
        const R sw = Mth<R>::sqrt(fmax(omw * ((R)2 - omw), (R)0));
        nn = wv * nu + sw * (c5 * e2 + s5 * e3); // sensor normal at the proposed end point
        fn = is_end ? T.eta + (T.eta_lo + T.rad * nn) : fg;
    }
    LPt<R> pn = lpt_fast(T, fn, q4);
    if constexpr (EARLY) {
        if (q4) lpt_settle(T, fn, pn);
    } else {
        if (q1 | q2 | q3 | q4) {
            lpt_settle(T, fm1, pm1);
            lpt_settle(T, fo, po);
            lpt_settle(T, fp1, pp1);
            lpt_settle(T, fn, pn);
        }
        old_window();
    }
    const Seg<R> An = make_seg_lp(T, fm1, fn, pm1, pn), Bn = make_seg_lp(T, fn, fp1, pn, pp1);
    const LayV<R> lnw = lay_at(T, pn.l);
    R d = seg_term(An) - seg_term(Ao);
    d += hp1 ? seg_term(Bn) - seg_term(Bo) : (R)0;
    d += vtx_term<R, false, true, false>(T, km1, lm1, um, An.u, up) -
         vtx_term<R, false, true, false>(T, km1, lm1, um, Ao.u, up);
    d += vtx_term<R, true, false, false>(T, kj, lnw, An.u, Bn.u, nn) -
         vtx_term<R, true, false, false>(T, kj, lo, Ao.u, Bo.u, nu);
    d += vtx_term<R, true, false, true>(T, kp1, lp1, Bn.u, up, up) -
         vtx_term<R, true, false, true>(T, kp1, lp1, Bo.u, up, up);
    if constexpr (SAMP == SAMP_LOCAL) {
        // log q(x | y) - log q(y | x) of the two Gaussian proposals, each
        // with its own step size (so the normalisations h^{-3/2} enter)
        const V3<R> gy = vertex_grad(T, km1, lm1, um, pm1, pn, pp1, An, Bn, lnw, kp1, up, up, lp1);
        const R m = fmin(An.len, Bn.len);
        const R hy = (R)sc.mala_h * m * m;
        const V3<R> b = (fo - fn) - ((R)0.5 * hy) * gy;
        const R lq = (R)1.5 * Mth<R>::log(hx * Mth<R>::rcp(hy)) - dot(b, b) * Mth<R>::rcp((R)2 * hy) + half_xi2;
        d += is_end ? (R)0 : lq;
        move = is_end ? MV_END : MV_LMALA;
    }
    // the angular response changes only when the end point itself moves
    if (T.dk == RJPATH_DET_PAPER && is_end) d += rho_log(T, nn) - rho_log(T, nu);
    logA = d;
    if (logu < logA) {
        accepted = 1;
        ps.st(j, Vtx<R>{fn.x, fn.y, fn.z, hp1 ? Bn.tb : (R)0});
        ps.stw(j - 1, An.tb);
        ln.L += (double)An.len - (double)Ao.len + (hp1 ? (double)Bn.len - (double)Bo.len : 0.0);
        ln.S += ((double)An.tb - (double)vm1.w) + (hp1 ? (double)Bn.tb - (double)vo.w : 0.0);
    }
}

// A jump step: birth or death of an interior vertex through the bi-spherical
// map.  Returns the move kind, log A, the segment or vertex (-1: the proposal
// is invalid) and whether it was accepted.
template <class R, bool LO, int SAMP>
__device__ __forceinline__ void jump_move(const Tgt<R>& T, const PathRef<R, LO>& ps, const WavePaths<R>& W, Lane<R>& ln,
                                          const StepCtx& sc, const StepLoop& lp, const uint32_t r[8], R logu, int& move,
                                          int& idx, int& accepted, R& logA) {
    const int n = ln.n;
    idx = -1;
    accepted = 0;
    const V3<R> ex = {(R)1, (R)0, (R)0};
    const bool birth = r[2] < sc.bthresh;
    move = birth ? MV_BIRTH : MV_DEATH;
    // S = sum of the cached segment depths, kept by the lane as a running sum
    // (summed afresh in path order at every launch start and after whole-path
    // moves).  The segment scan of a birth reads the first depths from their
    // LDS slots at once (scan_slots: depths past the path's end are stale or
    // zero, never negative) and the rest four at a time.
    constexpr int WB = scan_slots<R, SAMP>();
    const double S = ln.S;
    const bool valid = birth ? (n < sc.cap && S > 0.0) : (n > 2);
    int iA = 0, jv = 1;
    if (valid) {
        if (birth) {
            // segment k with probability tau_b(k) / S: the first k whose
            // cumulative depth exceeds U S, i.e. the number of prefixes that
            // do not (the cumulative sums never decrease)
            const double tgt = (double)unif<double>(r[0]) * S;
            R wv[WB];
#pragma unroll
            for (int v = 0; v < WB; ++v) wv[v] = ps.lds_w(v < ps.V ? v : ps.V);
            double cum = 0.0;
            int k = 0;
            // (slots past the path only count once its whole sum does not
            // exceed U S, by rounding; k is then cut to the last segment)
#pragma unroll
            for (int v = 0; v < WB; ++v) {
                cum += (double)wv[v];
                k += cum <= tgt ? 1 : 0;
            }
            k = k < ps.V ? k : ps.V; // (the padding slot read past V holds no depth)
            for (int v = WB < ps.V ? WB : ps.V; v < n - 1 && cum <= tgt; v += 4) {
                R w4[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) w4[i] = ps.w(v + i < n - 1 ? v + i : v);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    cum += v + i < n - 1 ? (double)w4[i] : 0.0;
                    k += cum <= tgt ? 1 : 0;
                }
            }
            k = k < n - 2 ? k : n - 2;
            iA = k;
        } else {
            jv = 1 + pick(r[0], (uint32_t)(n - 2));
            iA = jv - 1;
        }
        idx = birth ? iA : jv;
    }
    const int iB = birth ? iA + 1 : iA + 2;
    const bool hprev = iA >= 1, hnext = iB + 1 <= n - 1;
    V3<R> A, B, gprev, gnext, fj;
    R wA, wj; // cached depths of segments iA and jv (jv's is used by a death)
    if (LO) {
        // slots iA-1 .. iA+3, read as they are (padding makes all readable)
        const Vtx<R> s1 = ps.ld(iA), s2 = ps.ld(iA + 1);
        const V3<R> s0 = ps.p(iA - 1), s3 = ps.p(iA + 2), s4 = ps.p(iA + 3);
        gprev = s0;
        A = pos(s1);
        fj = pos(s2); // jv = iA + 1 for a death (unused by a birth)
        wA = s1.w;
        wj = s2.w;
        B = birth ? pos(s2) : s3;
        gnext = birth ? s3 : s4;
    } else {
        Vtx<R> vA, vj, vB, vp, vn;
        ps.ld5(iA, jv, iB < n ? iB : n - 1, hprev ? iA - 1 : 0, hnext ? iB + 1 : 0, vA, vj, vB, vp, vn);
        A = pos(vA);
        wA = vA.w;
        B = pos(vB);
        gprev = pos(vp);
        gnext = pos(vn);
        fj = pos(vj);
        wj = vj.w;
    }
    const V3<R> fprev = hprev ? gprev : A - ex;
    const V3<R> fnext = hnext ? gnext : B + ex;
    const V3<R> mid = (R)0.5 * (A + B);
    bool q1, q2, q3;
    LPt<R> pA = lpt_fast(T, A, q1), pB = lpt_fast(T, B, q2), pmid = lpt_fast(T, mid, q3);
    if (q1 | q2 | q3) {
        lpt_settle(T, A, pA);
        lpt_settle(T, B, pB);
        lpt_settle(T, mid, pmid);
    }
    const Seg<R> AB = make_seg_lp(T, A, B, pA, pB);
    const LayV<R> lm = lay_at(T, pmid.l);
    const R gam = (R)0.5 * AB.len;
    const R beta = lm.keq + (R)0.5 * (gam * lm.b - (R)1); // centering rule at the midpoint
    const QS<R> qs = make_qs(beta);
    V3<R> fv;
    {
        // the bi-spherical proposal (used by births; deaths take the vertex itself)
        R w = qs_sample(qs, unif<R>(r[4])); // 1 + cos s by the inverse CDF of q(s)
        // t from the logistic q(t): e^t = a/(1-a); sinh t and cosh t - cos s in closed form
        R a5 = unif<R>(r[5]), b5 = (R)1 - a5, ab2 = (R)2 * a5 * b5;
        R ss = Mth<R>::sqrt(fmax(w * ((R)2 - w), (R)0));
        R ph = unif<R>(r[6]);
        V3<R> e2, e3;
        onb(AB.u, e2, e3);
        R sc_ = gam * Mth<R>::rcp((R)1 - ab2 * w);
        V3<R> tr = Mth<R>::cos2pi(ph) * e2 + Mth<R>::sin2pi(ph) * e3;
        const V3<R> fb = mid + sc_ * ((a5 - b5) * AB.u + (ab2 * ss) * tr);
        fv = birth ? fb : fj;
    }
    const LPt<R> pv = lpt(T, fv);
    const Seg<R> sA = make_seg_lp(T, A, fv, pA, pv), sB = make_seg_lp(T, fv, B, pv, pB);
    // the direction past B: of the next segment, or the sensor normal where B is the end point
    const V3<R> up = unit_dir(fprev, A);
    V3<R> un;
    {
        const V3<R> rt = fnext - B, re = from_eta(T, B);
        const V3<R> rr = {hnext ? rt.x : re.x, hnext ? rt.y : re.y, hnext ? rt.z : re.z};
        un = Mth<R>::rsqrt(dot(rr, rr)) * rr;
    }
    const LayV<R> la = lay_at(T, pA.l), lb = lay_at(T, pB.l), lv = lay_at(T, pv.l);
    const int kA = hprev ? VK_TURN : VK_EMIT, kB = hnext ? VK_TURN : VK_END;
    // (an end point B is the same in x and y: its angular response cancels)
    const R tx = vtx_term<R, false, true, false>(T, kA, la, up, AB.u, un) +
                 vtx_term<R, true, false, false>(T, kB, lb, AB.u, un, un);
    const R ty = vtx_term<R, false, true, false>(T, kA, la, up, sA.u, un) +
                 vtx_term<R, true, false, false>(T, kB, lb, sB.u, un, un) +
                 vtx_term<R, false, false, false>(T, VK_TURN, lv, sA.u, sB.u, un);
    V3<R> dq = sA.u - sB.u;
    R q = dot(dq, dq);
    // segment factors of y over x times |J| / q(s) q(t) q(phi): the inverse-square
    // factors of the two new segments cancel against J; 1 + cos s = q / 2
    const R LOG2PI = (R)1.83787706640934548356;
    R jac = -sA.tc - sB.tc + AB.tc + (R)2 * Mth<R>::log(sA.len + sB.len) - AB.loglen + qs.lnorm +
            (R)0.5 * beta * q + LOG2PI;
    const int nx = birth ? n : n - 1;
    const double Sx = birth ? S : S - (double)wA - (double)wj + (double)AB.tb;
    R lpup = (R)sc.log_pb + Mth<R>::log(AB.tb) - Mth<R>::log((R)Sx);
    R lpdn = (R)sc.log_pd - Mth<R>::log((R)(nx - 1));
    // logw[nx + 1] - logw[nx] (both differences formed first: a choice between
    // the loads would become a dynamically indexed stack slot)
    const double dlw_b = ln.lwp - ln.lw0, dlw_d = ln.lw0 - ln.lwm;
    R dlw = (sc.logw && valid) ? (R)(birth ? dlw_b : dlw_d) : (R)0;
    R logAb = (ty - tx) + jac + dlw + lpdn - lpup;
    logA = valid ? (birth ? logAb : -logAb) : Mth<R>::ninf();
    accepted = logu < logA ? 1 : 0;
    constexpr bool TOGETHER = !LO && (SAMP == SAMP_TREE || SAMP == SAMP_JOINT);
    if (TOGETHER) shift_shared<R>(W, birth, birth ? n - 1 : iA + 2, accepted ? n - 2 - iA + (birth ? 1 : 0) : 0);
    if (accepted) {
        fold_run(ln, T.n0, sc, lp); // the steps spent at the old n
        const double dL = (double)sA.len + (double)sB.len - (double)AB.len;
        if (!TOGETHER) ps.shift(birth, iA + 1, birth ? n - 1 : n - 2);
        if (birth) ps.st(iB, Vtx<R>{fv.x, fv.y, fv.z, sB.tb});
        ps.stw(iA, birth ? sA.tb : AB.tb);
        ln.L += birth ? dL : -dL;
        ln.S = birth ? (S - (double)wA) + ((double)sA.tb + (double)sB.tb) : Sx;
        ln.n = birth ? n + 1 : n - 1;
        if (sc.logw) {
            const double lw = sc.logw[!birth ? n - 2 : n + 2 <= sc.cap ? n + 2 : sc.cap];
            const double lw0 = birth ? ln.lwp : ln.lwm;
            ln.lwm = birth ? ln.lw0 : lw;
            ln.lwp = birth ? lw : ln.lw0;
            ln.lw0 = lw0;
        }
        if (sc.logw) ln.invw = inv_tilt<R>(ln.lw0);
    }
}

// One perturbation step of a lane inside the step loop, then the counts.  The
// class of a step is the wave's, so each class has its own loop below and its
// counts are touched only there.
template <class R, bool LO, int SAMP>
__device__ __forceinline__ void perturb_step(const KArgs& a, const Tgt<R>& T, const PathRef<R, LO>& ps,
                                             Lane<R>& ln, const StepCtx& sc, const StepLoop& lp, int c) {
    const uint64_t step = lp.step0 + (uint64_t)lp.s;
    uint32_t r[8];
    draw8<SAMP>(sc, step, r);
    // (a chain that is not live rejects every proposal)
    const R logu = ln.live ? Mth<R>::log(unif<R>(r[1])) : -Mth<R>::ninf();
    int move, idx, accepted;
    R logA;
    perturb_move<R, LO, SAMP>(T, ps, ln, sc, step, r, logu, move, idx, accepted, logA);
    if (lp.counted()) {
        ln.ap += (uint32_t)accepted;
        if constexpr (SAMP == SAMP_LOCAL) {
            const uint32_t im = move == MV_LMALA ? 1u : 0u;
            ln.mp += im;
            ln.ma += im & (uint32_t)accepted;
        }
        count_step(ln);
    }
    put_trace(a, ln, c, lp.s, move, idx, accepted, logA, logu);
}

// A perturbation step of the joint Langevin sampler: the lanes whose pick is an
// interior vertex move all of theirs together, shared by the wave; the others'
// end points are perturbed.
template <class R>
__device__ __forceinline__ void joint_step(const KArgs& a, const Tgt<R>& T, const PathRef<R, false>& ps,
                                           const WavePaths<R>& W, Lane<R>& ln, const StepCtx& sc, const StepLoop& lp,
                                           int c) {
    const uint64_t step = lp.step0 + (uint64_t)lp.s;
    uint32_t r[8];
    draw8<SAMP_JOINT>(sc, step, r);
    const R logu = ln.live ? Mth<R>::log(unif<R>(r[1])) : -Mth<R>::ninf();
    int move = MV_MALA, idx = 1 + pick(r[0], (uint32_t)(ln.n - 1)), accepted = 0;
    R logA = Mth<R>::ninf();
    const bool joint = idx != ln.n - 1;
    if (!joint) perturb_move<R, false, SAMP_JOINT>(T, ps, ln, sc, step, r, logu, move, idx, accepted, logA);
    joint_move<R>(T, ps, W, ln, sc, step, joint && ln.live, logu, accepted, logA);
    if (lp.counted()) {
        ln.ap += (uint32_t)accepted;
        ln.mp += joint ? 1u : 0u;
        ln.ma += joint ? (uint32_t)accepted : 0u;
        count_step(ln);
    }
    put_trace(a, ln, c, lp.s, move, idx, accepted, logA, logu);
}

// The tree sampler's first step of every cycle: a tree-coordinate move of
// every chain of the wave.
template <class R>
__device__ __forceinline__ void tree_step(const KArgs& a, const Tgt<R>& T, const PathRef<R, false>& ps,
                                          const WavePaths<R>& W, Lane<R>& ln, const StepCtx& sc, const StepLoop& lp,
                                          int c) {
    const uint64_t step = lp.step0 + (uint64_t)lp.s;
    uint32_t r[8];
    draw8<SAMP_TREE>(sc, step, r);
    const R logu = ln.live ? Mth<R>::log(unif<R>(r[1])) : -Mth<R>::ninf();
    int accepted;
    R logA;
    tree_move<R>(T, ps, W, ln, sc, step, r, logu, accepted, logA);
    if (lp.counted()) {
        ln.ap += (uint32_t)accepted;
        ln.mp += 1u;
        ln.ma += (uint32_t)accepted;
        count_step(ln);
    }
    put_trace(a, ln, c, lp.s, MV_TREE, -1, accepted, logA, logu);
}

template <class R, bool LO, int SAMP>
__device__ __forceinline__ void jump_step(const KArgs& a, const Tgt<R>& T, const PathRef<R, LO>& ps,
                                          const WavePaths<R>& W, Lane<R>& ln, const StepCtx& sc, const StepLoop& lp,
                                          int c) {
    uint32_t r[8];
    draw8<SAMP>(sc, lp.step0 + (uint64_t)lp.s, r);
    const R logu = ln.live ? Mth<R>::log(unif<R>(r[1])) : -Mth<R>::ninf();
    int move, idx, accepted;
    R logA;
    jump_move<R, LO, SAMP>(T, ps, W, ln, sc, lp, r, logu, move, idx, accepted, logA);
    if (lp.counted()) {
        const uint32_t ib = move == MV_BIRTH ? 1u : 0u, ac = (uint32_t)accepted;
        ln.ne += idx < 0 ? 1u : 0u;
        ln.pb += ib;
        ln.ab += ib & ac;
        ln.ad += ac & ~ib;
        count_step(ln);
    }
    put_trace(a, ln, c, lp.s, move, idx, accepted, logA, logu);
}


// ---------------------------------------------------------------------------
// The step kernel.  MK: MK_HOM (every medium of the launch is homogeneous: the
// layer lookups fold away), MK_LAY (layer tables read from HBM) or MK_LAY_LDS
// (tables staged in LDS).  SL: some layer mixes in the Rayleigh-like term.
// EVEN: every medium of the launch has several evenly spaced layers, so that
// the lookups' tests for one layer and for uneven edges fold: each of the
// four segments and seven layer reads of a step otherwise carries two
// branches of its own (about 700 basic blocks in the kernel, which also keep
// the loads of one segment from being issued with the next one's).
// ---------------------------------------------------------------------------
enum { MK_HOM = 0, MK_LAY = 1, MK_LAY_LDS = 2 };

// The place of this wave's chains: an ordered launch's order stands in bits 8
// and up of the status words, one per wave, and is cleared as it is read; bits
// 0 to 7 are the status of the word's own chain, which another wave may have
// stored already, so both sides store bytes.
__device__ __forceinline__ int take_order(const KArgs& a, int wave) {
    if (!a.ordered) return wave;
    if (wave >= a.ordered) return wave; // (past the last chain)
    int32_t* const word = a.status + wave;
    const int w = *(volatile int32_t*)word >> 8;
    if (threadIdx.x % WAVE == 0) {
        ((volatile uint8_t*)word)[1] = 0;
        ((volatile uint16_t*)word)[1] = 0;
    }
    return __builtin_amdgcn_readfirstlane(w);
}
__device__ __forceinline__ void put_status(const KArgs& a, int c, int v) {
    if (c < a.ordered) *(volatile uint8_t*)(a.status + c) = (uint8_t)v;
    else a.status[c] = v;
}

template <class R, int MK, int SAMP, bool SL, bool EVEN> __device__ __forceinline__ void run_body(const KArgs& a) {
    constexpr bool TAB = MK == MK_LAY_LDS;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, bs = blockDim.x;
    MedTab<R> tab = hbm_tab<R>(a);
    size_t tab_bytes = 0;
    if (TAB) {
        tab = stage_tables<R>(a, smem);
        __syncthreads();
        tab_bytes = a.tab_bytes;
    }
    const size_t C = (size_t)a.C;
    const int lane = tid % WAVE, cap = a.cap;
    // the wave's first chain; a wave of the whole-path samplers owns a.cpw
    // chains (its first lanes') and shares their moves over all 64 lanes
    constexpr bool SHARED = SAMP == SAMP_TREE || SAMP == SAMP_JOINT;
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE); // (uniform: kept in SGPRs)
    const int c0 = take_order(a, (int)blockIdx.x * (bs / WAVE) + wave) * (SHARED ? a.cpw : WAVE);
    int c = c0 + lane;
    const bool own = c < a.C && (!SHARED || lane < a.cpw);
    if (!SHARED && !own) return;
    // this wave's tile, past its leading padding slot
    const LdsPtr<R> tiles = (LdsPtr<R>)((L4<R>*)(smem + tab_bytes));
    const LdsPtr<R> tile = tiles + (size_t)wave * (a.V + SLOT_PAD) * WAVE + WAVE;
    const LdsPtr<R> lslots = tile + lane;
    int t = own ? a.target[c] : -1;
    Lane<R> ln{};
    ln.n = own ? a.n[c] : 0;
    // malformed chains are flagged and never touched
    const bool good = own && t >= 0 && t < a.T && ln.n >= 2 && ln.n <= cap && a.medium[t] >= 0 && a.medium[t] < a.n_media;
    if (own && !good) put_status(a, c, 1);
    LaneRun run = whole_wave();
    if (SHARED) {
        // lanes without a chain stay for the shared moves, as a dead chain of
        // two equal vertices; before share_lanes() on the target of the good
        // lane to their left (so that the lanes of a target stay neighbours),
        // or of the first one
        const uint64_t m = __ballot(good);
        if (m == 0) return;
        const uint64_t left = m & ((1ull << lane) - 1);
        const int from = left ? 63 - __clzll((long long)left) : __ffsll((unsigned long long)m) - 1;
        const int t1 = __shfl(t, from, WAVE);
        if (!good) {
            t = t1;
            c = c0 + from;
            ln.n = 2;
        }
        run = share_lanes(lane, a.cpw, good ? ln.n : 0, t);
    } else if (!good) {
        return;
    }
    Tgt<R> T;
    load_target(a, t, T, tab);
    // compile-time facts of this instantiation (the lookups that test them fold)
    if (MK == MK_HOM) {
        T.mcnt = 1;
        T.hom = true;
    }
    if (EVEN) {
        T.hom = false;
        T.uniform = 1;
    }
    T.sl = SL;
    if (!SL) T.l0.fsl = (R)0;
    // vertices beyond the LDS slots: in place (a chain's lie n_chains apart), or
    // chain after chain in the work buffer (move_in)
    Vtx<R>* const own_verts = (Vtx<R>*)a.verts + c;
    Vtx<R>* const far = SHARED ? (Vtx<R>*)a.work + (size_t)c * cap : own_verts;
    const size_t far_stride = SHARED ? 1 : C;
    PathRef<R, false> ps{lslots, far, a.V, far_stride};
    PathRef<R, true> pl{lslots, far, a.V, far_stride};
    // stage the LDS part of the path
    const int nl0 = ln.n < a.V ? ln.n : a.V;
    if (!SHARED || good) {
        for (int v = 0; v < nl0; ++v) lds_st<R>(ps.lds + v * WAVE, own_verts[(size_t)v * C]);
    } else {
        for (int v = 0; v < nl0; ++v) lds_st<R>(ps.lds + v * WAVE, Vtx<R>{(R)0, (R)0, (R)0, (R)0});
    }
    // the depths a birth's scan reads past the path (slot V is padding): none
    for (int v = nl0; v <= a.V && v < scan_slots<R, SAMP>(); ++v) pl.stw(v, (R)0);
    if (a.V < scan_slots<R, SAMP>()) pl.stw(a.V, (R)0);

    WavePaths<R> W{};
    if constexpr (SHARED) {
        // proposals: the tile's columns from 32 on where the wave owns at most
        // 32 chains, else a.Vy slots' room behind the block's tiles
        const bool half = a.cpw < WAVE;
        W.x = tile;
        W.V = a.V;
        W.y = half ? tile + WAVE / 2
                   : tiles + (size_t)(bs / WAVE) * (a.V + SLOT_PAD) * WAVE + (size_t)wave * a.Vy * WAVE;
        W.My = half ? a.V * (WAVE / 2) : a.Vy * WAVE;
        W.ymask = half ? ~(WAVE / 2 - 1) : 0;
        W.width = a.C - c0 < a.cpw ? a.C - c0 : a.cpw;
        W.per_width = (0x80000000u + (uint32_t)W.width - 1u) / (uint32_t)W.width;
        W.rows = (Vtx<R>*)a.verts + c0;
        W.far = (Vtx<R>*)a.work + (size_t)c0 * cap;
        W.C = C;
        W.cap = cap;
        W.cpw = a.cpw;
        W.chain0 = (uint32_t)c0;
        W.lane = lane;
        W.run = run;
        // (malformed chains keep all their vertices)
        W.move_in(own && !good ? 0 : a.V, good ? ln.n : own ? cap : 0);
    }

    ln.lp = full_logp(T, ps, ln.n, ln.L, &ln.S);
    const bool healthy = good && isfinite(ln.lp);
    if (good) put_status(a, c, healthy ? 0 : 1);
    StepCtx sc;
    sc.chain = (uint32_t)c;
    sc.k0 = (uint32_t)a.seed;
    sc.k1 = (uint32_t)(a.seed >> 32);
    sc.cap = cap;
    sc.bthresh = a.bthresh;
    const double pb = (double)a.bthresh * 0x1p-32;
    sc.log_pb = log(pb);
    sc.log_pd = log1p(-pb);
    sc.sigma = a.sigma;
    sc.ikappa = 1.0 / a.kappa_end;
    sc.e2k = exp(-2.0 * a.kappa_end);
    sc.mala_h = a.mala_h;
    sc.sampler = a.sampler;
    sc.logw = a.logw ? a.logw + (size_t)t * (cap + 1) : nullptr;
    sc.hist = a.hist ? a.hist + (size_t)t * (cap + 1) : nullptr;
    ln.invw = 1.0;
    if (sc.logw) {
        ln.lwm = sc.logw[ln.n - 1];
        ln.lw0 = sc.logw[ln.n];
        ln.lwp = sc.logw[ln.n < cap ? ln.n + 1 : cap];
        ln.invw = inv_tilt<R>(ln.lw0);
    }
    StepLoop lp{};
    lp.step0 = a.step_dev ? *a.step_dev + a.step0 : a.step0; // step0 is the offset then
    lp.tilt = sc.logw != nullptr;
    {
        const int64_t d = a.burn_in - (int64_t)lp.step0;
        lp.first = d < 0 ? 0 : (d < (int64_t)a.steps ? (int)d : a.steps);
    }
    int phase = (int)(lp.step0 % (uint64_t)a.cycle_len);

    ln.live = healthy;
    // Every lane runs every step (a lane that is not live only rejects), so
    // that the step loop is uniform across the wave.  The steps of one class
    // follow each other in a loop of their own.  A wave takes the LDS-only
    // form of a step while all its paths fit their slots (n changes in jump
    // steps alone: one vote per run of perturbation steps) and the general
    // form (slots beyond V in HBM) while some do not.
    while (lp.s < a.steps) {
        const int left = a.steps - lp.s;
        if (phase < a.n_perturb) {
            const int m = a.n_perturb - phase < left ? a.n_perturb - phase : left, end = lp.s + m;
            if constexpr (SHARED) {
                if (SAMP == SAMP_TREE && phase == 0) {
                    tree_step<R>(a, T, ps, W, ln, sc, lp, c);
                    ++lp.s;
                }
            }
            if constexpr (SAMP == SAMP_JOINT) {
                for (; lp.s < end; ++lp.s) joint_step<R>(a, T, ps, W, ln, sc, lp, c);
            } else if (__all(ln.n < a.V)) {
                for (; lp.s < end; ++lp.s) perturb_step<R, true, SAMP>(a, T, pl, ln, sc, lp, c);
            } else {
                for (; lp.s < end; ++lp.s) perturb_step<R, false, SAMP>(a, T, ps, ln, sc, lp, c);
            }
            phase += m;
        } else {
            const int m = a.cycle_len - phase < left ? a.cycle_len - phase : left, end = lp.s + m;
            for (; lp.s < end; ++lp.s) {
                if (__all(ln.n < a.V))
                    jump_step<R, true, SAMP>(a, T, pl, W, ln, sc, lp, c);
                else
                    jump_step<R, false, SAMP>(a, T, ps, W, ln, sc, lp, c);
            }
            phase += m;
        }
        if (phase == a.cycle_len) phase = 0;
    }
    // counted steps of each class (the same for every lane)
    const uint32_t counted = (uint32_t)(a.steps - lp.first);
    const uint32_t perturbs = count_perturbs(lp.step0 + (uint64_t)lp.first, counted, a.cycle_len, a.n_perturb);
    const uint32_t jumps = counted - perturbs;

    if (!healthy) ln.mark = lp.s; // (nothing of it enters the histogram)
    fold_run(ln, T.n0, sc, lp);
    // log p of the final path (refreshed once rather than tracked per step)
    if (healthy) ln.lp = full_logp(T, ps, ln.n, ln.L);
    if constexpr (SHARED) {
        W.move_out(own && !good ? 0 : a.V, good ? ln.n : own ? cap : 0);
        if (!good) return;
        asm volatile("" : "+v"(c)); // (formed again here rather than kept through the steps)
    }
    // write back the LDS part, the vertex count, log p and the statistics
    const int nw = ln.n < a.V ? ln.n : a.V;
    for (int v = 0; v < nw; ++v) ((Vtx<R>*)a.verts + c)[(size_t)v * C] = lds_ld<R>(ps.lds + v * WAVE);
    a.n[c] = ln.n;
    a.logp[c] = ln.lp;
    if (healthy) {
        double* sp = a.stats + (size_t)c * RJPATH_NSTAT;
        sp[0] += ln.cnt;
        // without a sector tilt 1/w = 1 and the two sums are counts
        sp[1] += sc.logw ? ln.a1 : (double)ln.cnt;
        sp[2] += sc.logw ? ln.a2 : (double)ln.c2;
        sp[3] += ln.sl;
        sp[4] += ln.sl2;
        sp[5] += (double)ln.sn;
        sp[6] += perturbs;
        sp[7] += ln.pb;
        sp[8] += jumps - ln.pb;
        sp[9] += ln.ap;
        sp[10] += ln.ab;
        sp[11] += ln.ad;
        sp[12] += ln.ncap;
        sp[13] += ln.mp;
        sp[14] += ln.ma;
        sp[15] += ln.ne;
    }
}

// (FP32: two waves per SIMD, which the joint Langevin variant with the mixture
// and tables in HBM would miss by three registers, and the leaner ones reach
// by themselves; below, the even-layer variants of the whole-path moves and of the
// mixture spill for it: 40 bytes per lane for joint Langevin moves, 16 for tree
// moves, 12 to 88 with the mixture.  Without the bound nothing spills and one wave
// runs: 50,001 chains of joint moves, 200 steps, 5.05 ms instead of 3.1, 262,144 of
// tree moves 7.2 instead of 4.4.)
template <class R, int MK, int SAMP, bool SL>
__global__ void __launch_bounds__(256, sizeof(R) == 4 && SAMP == SAMP_JOINT ? 2 : 1) run_kernel(KArgs a) {
    run_body<R, MK, SAMP, SL, false>(a);
}

template <class R, int MK, int SAMP, bool SL>
__global__ void __launch_bounds__(256, sizeof(R) == 4 ? 2 : 1) run_even_layers_kernel(KArgs a) {
    run_body<R, MK, SAMP, SL, true>(a);
}

} // namespace rj
