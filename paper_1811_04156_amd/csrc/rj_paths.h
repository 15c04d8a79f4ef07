// rj_paths.h -- the paths and proposals of a wave's chains as the whole-path
// moves share them over the lanes (included by rj_step.h, whose path storage it
// uses).
#pragma once

#include "rj_wave.h"

namespace rj {

// Neighbouring lanes work on neighbouring vertices of one chain, so
// the proposals are kept chain after chain without gaps (a wave's chains need
// the sum of their n, not 64 times the longest), the first My vertices in LDS
// and the rest in the wave's part of the work buffer; the vertices of the paths
// beyond their LDS slots, which lie 16 n_chains bytes apart, are copied behind
// them in the same order first.  (Read in place, one cache line per vertex
// and read, the two-region test's 80-vertex paths kept the waves waiting for
// 75% of their cycles.)
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
    LaneRun run;       // the lanes with this lane's target, which share its chains' items

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

// A chain's place among the wave's vertices (n of each chain that takes part),
// their total, and the offset of the paths' copy in the wave's part of the work
// buffer (0: none).
struct WavePlaces {
    int at, all, copy;
};

// Begins a shared move (all 64 lanes): `mine` vertices of this lane's chain.
template <class R, bool LO>
__device__ __forceinline__ WavePlaces wave_places(const WavePaths<R>& W, const PathRef<R, LO>& ps, int mine) {
    // (the chains' own lanes wrote the vertices beyond the LDS slots)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    WavePlaces P;
    const int upto = wave_prefix(mine);
    P.at = upto - mine;
    P.all = __builtin_amdgcn_readlane(upto, WAVE - 1);
    P.copy = !LO && 2 * P.all <= W.room && __any(mine > W.V) ? P.all : 0;
    if (P.copy) {
        // row by row, lanes over the wave's chains (whole cache lines), four rows in flight
        const int q = W.lane & (W.cpw - 1), rows = WAVE / W.cpw;
        const int nq = __shfl(mine, q, WAVE), to = P.copy + __shfl(P.at, q, WAVE);
        for (int v = W.V + W.lane / W.cpw; __any(v < nq); v += 4 * rows) {
            L4<R> g[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (v + i * rows < nq) g[i] = *(const L4<R>*)(W.gx + ((size_t)(v + i * rows) * W.C + q));
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (v + i * rows < nq) *(L4<R>*)(W.part + (to + v + i * rows)) = g[i];
        }
    }
    if (mine > 0) *W.sum(W.lane) = 0.0;
    return P;
}

// Ends it (a lane that is not `act` keeps its results): log A is the chain's sum; the accepted proposals, with the segment
// depths kept beside their vertices, replace the paths.
template <class R>
__device__ __forceinline__ void settle_shared(const WavePaths<R>& W, const WavePlaces& P, Lane<R>& ln, bool act, R logu,
                                              int& accepted, R& logA) {
    const int n = ln.n, lane = W.lane;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    int taken = 0;
    if (act) {
        const double la = *W.sum(lane);
        logA = isfinite(la) ? (R)la : Mth<R>::ninf();
        accepted = taken = logu < logA ? 1 : 0;
        // (the sums of the accepted proposal's length and depths next)
        W.sum(lane)[0] = 0.0;
        W.sum(lane)[1] = 0.0;
    }
    WaveItems it;
    it.init(lane, taken ? n : 0);
    while (it.more()) {
        int q, k;
        const bool has = it.next(q, k);
        const int aq = __shfl(P.at, q, WAVE), nq = __shfl(n, q, WAVE);
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
    if (taken) {
        ln.L = W.sum(lane)[0];
        ln.S = W.sum(lane)[1];
    }
}

} // namespace rj
