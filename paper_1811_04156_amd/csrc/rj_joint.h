// rj_joint.h -- the joint Langevin move of the step kernel as the wave shares it
// (included by rj_step.h).
#pragma once

#include "rj_paths.h"

namespace rj {

// Langevin move of all interior vertices of the chains with `act` (all 64 lanes
// call it together): y = x + (h / 2) grad log p(x) +
// sqrt(h) xi, accepted with
//   log A = log p(y) - log p(x) + |xi|^2 / 2 - |x - y - (h / 2) grad log p(y)|^2 / (2 h).
// The items are (chain, segment): first over the paths, where an item forms its
// vertex's gradient from the five vertices around it and the proposal of that
// vertex, then over the proposals, in both by the lanes of the chain's target
// (share_lanes).  One lane per chain, walking path and proposal together, ran
// each step until the wave's longest path was done: a joint step of 50,001
// chains of the ragged layered batch (mean 6.4 vertices, longest 32) took 62 us,
// 29 once the items were shared (a median wave's share was 8, the slowest waves'
// far targets about 20), and takes 20 since long waves start first (rj_order.hip).
// Where every chain's neighbours have other targets a lane is left with its own chain and still pays for items: 60 steps of 262,144 such
// chains take 1.08 (layered) to 1.3 times (homogeneous, two-region) what one lane
// per chain took in a kernel without items; with both forms in this one a lane per
// chain takes 1.2 to 1.7 times as long.
template <class R>
__device__ __forceinline__ void joint_move(const Tgt<R>& T, const PathRef<R, false>& ps, const WavePaths<R>& W, Lane<R>& ln,
                                           const StepCtx& sc, uint64_t step, bool act, R logu, int& accepted, R& logA) {
    const int n = ln.n, lane = W.lane;
    const R h = (R)sc.mala_h, hh = (R)0.5 * h, sh = Mth<R>::sqrt(h);
    const WavePlaces P = wave_places<R>(W, act ? n : 0);
    if (act) {
        const Vtx<R> f = ps.ld(0), e = ps.ld(n - 1);
        W.sty(P.at, f);
        W.sty(P.at + n - 1, e);
    }
    auto around = [](int k, int nq, int (&v)[5]) __attribute__((always_inline)) {
        v[0] = k > 0 ? k - 1 : 0;
        v[1] = k;
        v[2] = k + 1;
        v[3] = k + 2 < nq ? k + 2 : k + 1;
        v[4] = k + 3 < nq ? k + 3 : k + 1;
    };
    WaveItems it;
    it.init(lane, act ? n - 1 : 0, W.run);
    while (it.more()) {
        int q, k;
        const bool has = it.next(q, k);
        const WaveChain<R> c{W, q, __shfl(P.at, q, WAVE)};
        const int nq = __shfl(n, q, WAVE);
        if (has) {
            int v[5];
            V3<R> f[5], g;
            Seg<R> A;
            around(k, nq, v);
            c.xs(v, f);
            double t = -segment_grad(T, nq, k, f, g, A);
            const int j = k + 1;
            if (j <= nq - 2) {
                uint32_t d[4] = {W.chain0 + (uint32_t)q, (uint32_t)step, (uint32_t)(step >> 32), 2u + (uint32_t)j};
                philox4x32_10(d, sc.k0, sc.k1);
                V3<R> xi;
                box_muller3<R>(d[0], d[1], d[2], d[3], xi);
                t += 0.5 * (double)dot(xi, xi);
                const V3<R> y = f[2] + hh * g + sh * xi;
                W.sty(c.at + j, Vtx<R>{y.x, y.y, y.z, (R)0});
            }
            W.add(q, t);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    it.init(lane, act ? n - 1 : 0, W.run);
    while (it.more()) {
        int q, k;
        const bool has = it.next(q, k);
        const WaveChain<R> c{W, q, __shfl(P.at, q, WAVE)};
        const int nq = __shfl(n, q, WAVE);
        if (has) {
            int v[5];
            V3<R> f[5], g;
            Seg<R> A;
            around(k, nq, v);
            c.ys(v, f);
            double t = segment_grad(T, nq, k, f, g, A);
            const int j = k + 1;
            if (j <= nq - 2) {
                const V3<R> d = c.x(j) - f[2] - hh * g;
                t -= (double)dot(d, d) / (2.0 * (double)h);
            }
            W.styw(c.at + k, A.tb);
            W.add(q, t);
        }
    }
    settle_shared<R>(W, P, ln, act, logu, accepted, logA);
}

} // namespace rj
