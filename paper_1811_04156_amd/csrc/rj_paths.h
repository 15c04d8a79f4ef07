// rj_paths.h -- the paths and proposals of a wave's chains as the whole-path
// moves share them over the lanes (included by rj_step.h, whose path storage it
// uses).
#pragma once

#include "rj_wave.h"

namespace rj {

// Neighbouring lanes work on neighbouring vertices of one chain, and a jump
// moves all vertices behind its own, so vertices beyond the LDS slots are kept
// chain after chain while the kernel runs: the paths' in the work buffer (cap
// vertices per chain), the proposals', without gaps (a wave's chains need the
// sum of their n, not 64 times the longest), first in LDS and then in the
// wave's columns of the chains' vertices, whose contents are in LDS and in the
// work buffer meanwhile.  Where they lie between the launches one cache line
// holds one vertex of a chain.  (65,536 chains of the two-region test, per
// step: a tree move, for which the paths were copied into this order each time,
// took 468 us and takes 379 (368 since the root's frame has a branch of its own), a
// perturbation 80 and takes 33; move_in and
// move_out are about 50 us of a launch.)
template <class R> struct WavePaths {
    LdsPtr<R> x, y;    // paths: slot 0 of column 0 of the wave's tile (stride WAVE); proposals: LDS vertex 0
    Vtx<R>* rows;      // vertex 0 of the wave's first chain (rows of n_chains, `width` of them the wave's)
    Vtx<R>* far;       // the wave's part of the work buffer
    int V, My, ymask;  // LDS vertex i of the proposals is y[i + (i & ymask)]
    int cpw, cap;      // chains per wave (a power of two); vertices per chain
    int width;         // chains of this wave (the last one may have fewer)
    uint32_t per_width; // ceil(2^31 / width)
    size_t C;
    uint32_t chain0;   // the wave's first chain
    int lane;
    LaneRun run;       // the lanes with this lane's target, which share its chains' items

    // vertex i (< width cap <= 2^18) of the proposals beyond LDS, row by row
    __device__ __forceinline__ Vtx<R>* spare(int i) const {
        const int row = (int)__umulhi(2u * (uint32_t)i, per_width);
        return rows + ((size_t)row * C + (uint32_t)(i - row * width));
    }
    __device__ __forceinline__ Vtx<R> ldy(int i) const {
        if (i < My) return lds_ld<R>(y + (i + (i & ymask)));
        return *spare(i);
    }
    __device__ __forceinline__ void sty(int i, const Vtx<R>& p) const {
        if (i < My) lds_st<R>(y + (i + (i & ymask)), p);
        else *spare(i) = p;
    }
    __device__ __forceinline__ void styw(int i, R w) const {
        if (i < My) ((LdsScalar<R>)(y + (i + (i & ymask))))[3] = w;
        else spare(i)->w = w;
    }
    // vertices lo .. hi - 1 of this lane's chain from their rows to the work
    // buffer, or back (all 64 lanes): row by row, lanes over the wave's chains
    // (whole cache lines), four rows in flight
    template <bool IN> __device__ __forceinline__ void move(int lo, int hi) const {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        const int q = lane & (cpw - 1), step = WAVE / cpw;
        const int first = __shfl(lo, q, WAVE), end = __shfl(hi, q, WAVE);
        Vtx<R>* const row = rows + q;
        Vtx<R>* const mine = far + (size_t)q * cap;
        for (int v = first + lane / cpw; __any(v < end); v += 4 * step) {
            L4<R> g[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (v + i * step < end)
                    g[i] = *(const L4<R>*)(IN ? row + (size_t)(v + i * step) * C : mine + (v + i * step));
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (v + i * step < end) *(L4<R>*)(IN ? mine + (v + i * step) : row + (size_t)(v + i * step) * C) = g[i];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    }
    __device__ __forceinline__ void move_in(int lo, int hi) const { move<true>(lo, hi); }
    __device__ __forceinline__ void move_out(int lo, int hi) const { move<false>(lo, hi); }
    // the chain's FP64 sums (padding slot -1 holds two)
    __device__ __forceinline__ LdsScalar<double> sum(int q) const { return (LdsScalar<double>)(x - WAVE + q); }
    __device__ __forceinline__ void add(int q, double v, int k = 0) const {
        __hip_atomic_fetch_add(sum(q) + k, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};

// Between a window's loads and its stores, where lanes write what others read:
// the fence keeps the wave's memory operations on their sides of it, the
// barrier the lanes together, so that no branch of the loads runs after a
// branch of the stores.
__device__ __forceinline__ void window_loaded() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The vertex shift of the wave's accepted jumps (all 64 lanes call it): `cnt`
// vertices of this lane's chain (0: none) move one slot up, from slot `from`
// downwards, or one down, from slot `from` upwards.  The items are (chain,
// vertex) in that order, so every window reads vertices that no earlier one
// has written over; within a window the lanes write vertices that others read,
// so all its loads come before its first store (window_loaded).  (Each lane its
// own chain's: a jump step of the two-region test, 65,536 chains, took 60 us
// and takes 42.)
template <class R> __device__ __forceinline__ void shift_shared(const WavePaths<R>& W, bool up, int from, int cnt) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    WaveItems it;
    it.init(W.lane, cnt);
    const int code = up ? ~from : from;
    while (it.more()) {
        int q, k;
        const bool has = it.next(q, k);
        const int cq = __shfl(code, q, WAVE);
        const int src = cq < 0 ? ~cq - k : cq + k, dst = cq < 0 ? src + 1 : src - 1;
        Vtx<R>* const path = W.far + (size_t)q * W.cap;
        L4<R> v;
        if (has) {
            if (src < W.V) v = W.x[src * WAVE + q];
            else v = *(const L4<R>*)(path + src);
        }
        window_loaded();
        if (has) {
            if (dst < W.V) W.x[dst * WAVE + q] = v;
            else *(L4<R>*)(path + dst) = v;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
}

// Chain q of the wave during a move: its first vertex's place `at` among the
// wave's proposals.
template <class R> struct WaveChain {
    const WavePaths<R>& W;
    int q, at;
    __device__ __forceinline__ V3<R> x(int v) const {
        if (v < W.V) return pos(lds_ld<R>(W.x + v * WAVE + q));
        return far_x(v);
    }
    __device__ __forceinline__ V3<R> far_x(int v) const {
        const L4<R> g = *(const L4<R>*)(W.far + ((size_t)q * W.cap + v));
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
                const L4<R> p = *(const L4<R>*)W.spare(at + v[i]);
                g[i] = {p.x, p.y, p.z};
            }
#pragma unroll
            for (int i = 0; i < K; ++i)
                if (at + v[i] >= W.My) o[i] = g[i];
        }
    }
};

// A chain's place among the wave's vertices (n of each chain that takes part)
// and their total.
struct WavePlaces {
    int at, all;
};

// Begins a shared move (all 64 lanes): `mine` vertices of this lane's chain.
template <class R> __device__ __forceinline__ WavePlaces wave_places(const WavePaths<R>& W, int mine) {
    // (the chains' own lanes wrote the vertices beyond the LDS slots)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    WavePlaces P;
    const int upto = wave_prefix(mine);
    P.at = upto - mine;
    P.all = __builtin_amdgcn_readlane(upto, WAVE - 1);
    if (mine > 0) *W.sum(W.lane) = 0.0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); // (other lanes add to it)
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
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
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
            else W.far[(size_t)q * W.cap + k] = f;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    if (taken) {
        ln.L = W.sum(lane)[0];
        ln.S = W.sum(lane)[1];
    }
}

} // namespace rj
