// rj_sampler.hip -- the score kernel (log p, vertex gradients and parameter
// score of the current paths), the device step counter and the dispatch of
// the step-kernel variants (rj_step.h, rj_run.h).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rj_step.h"
#include "rj_wave.h"

namespace rj {

// ---------------------------------------------------------------------------
// Score kernel: log p, d log p / d vertices and the per-layer parameter score.
//
// Work split.  A wave takes 64 chains, in one of two forms (shares_segments).
// Shared: their vertices are read row by row (whole cache lines) into an LDS
// strip, chain after chain without gaps, and the (chain, segment) items go over
// all lanes: one lane per chain waits for the wave's longest path (mean n 6,
// longest 25 to 40 on the ragged batches).  The kernel alone, score sums of 2^20
// chains: of a run of the ragged layered batch 443 us by lanes, 205 shared (tables
// read from HBM and two waves per SIMD: 315); of snapshot paths of mean n 6, whose
// 109 MB a large copy moves in 23, 460 and 241.
// A lane per chain (PathWalk): where the lengths of a wave are alike, where
// they overflow the strip and where neighbouring chains have different targets
// that form is the better one (below).
//
// The score sums of a block whose chains belong to at most two targets go to
// an LDS table, per target the sum of the weights and per layer the weighted
// path length, scatterings and d log sigma / dg, which become the derivatives
// when the block adds them to the caller's sums; other blocks add per item.
// ---------------------------------------------------------------------------
// Facts of the launch's media that fold the lookups' tests (as in the step
// kernel): every medium homogeneous, every medium of several evenly spaced
// layers (both without the simplified-Liu term), or neither.
enum { GK_ANY = 0, GK_EVEN = 1, GK_HOM = 2 };

// Where a chain's score contributions go: the block's LDS table (layer sums)
// or the caller's array (derivatives).
struct ScoreDst {
    double* row; // the target's row: weight, then three per layer
    bool table;
    // path length len (weighted) in a layer with coefficients av, bv
    __device__ __forceinline__ void length(int l, double len, double av, double bv) const {
        double* const p = row + 1 + 3 * l;
        if (table) {
            atomicAdd(p, len);
        } else {
            // d/d lambda_s = -b^2 d/db, d/d lambda_a = -a^2 d/da, with d log p/da = -L_l and
            // d log p/db = N_l / b - L_l (L_l: path length in layer l, N_l: scatterings in l)
            atomicAdd(p, bv * bv * len);
            atomicAdd(p + 1, av * av * len);
        }
    }
    __device__ __forceinline__ void scatter(int l, double w, double dg, double bv) const {
        double* const p = row + 1 + 3 * l;
        if (table) atomicAdd(p + 1, w);
        else atomicAdd(p, -bv * w); // log b at a scattering vertex
        atomicAdd(p + 2, w * dg);
    }
};

// d log sigma / dg at a turn, q = |ua - ub|^2
__device__ __forceinline__ double dturn_dg(double g, double fsl, double q) {
    double mu = 1.0 - 0.5 * q;
    double den = (1 - g) * (1 - g) + g * q;
    double dhg = -2 * g / (1 - g * g) - 3 * (g - mu) / den;
    if (fsl == 0.0) return dhg;
    const double PI = 3.14159265358979323846;
    double lhg = log((1 - g * g) / (4 * PI)) - 1.5 * log(den);
    double lsl = log((1 + g) / (1 - g) / (4 * PI)) + 2 * g / (1 - g) * log(0.5 * (1 + mu));
    double dsl = 2.0 / ((1 + g) * (1 - g)) + 2.0 / ((1 - g) * (1 - g)) * log(0.5 * (1 + mu));
    double m = lhg > lsl ? lhg : lsl;
    double es = fsl * exp(lsl - m), eh = (1 - fsl) * exp(lhg - m);
    return (es * dsl + eh * dhg) / (es + eh);
}

// The score contributions of the segment P -> Q of weight w: its length per
// layer and, where `turn`, the scattering at P, which the unit vector um leads
// to.  Returns the segment's direction.
template <class R>
__device__ __forceinline__ V3<R> segment_score(const Tgt<R>& T, int off, const ScoreDst& D, double w, V3<R> P, V3<R> Q,
                                              bool turn, V3<R> um) {
    const V3<R> r = Q - P;
    const R l2 = dot(r, r), il = Mth<R>::rsqrt(l2);
    const V3<R> u = il * r;
    const double len = (double)(l2 * il);
    const double uP = axis_u(T, P), uQ = axis_u(T, Q);
    const int lP = layer_u(T, uP), lQ = layer_u(T, uQ);
    if (lP == lQ) {
        const LayV<R> ly = lay_at(T, lP);
        D.length(off + lP, w * len, (double)ly.a, (double)ly.b);
    } else {
        const double lo = uP < uQ ? uP : uQ, hi = uP < uQ ? uQ : uP;
        const int llo = lP < lQ ? lP : lQ, lhi = lP < lQ ? lQ : lP;
        const double scl = len / (hi - lo);
        for (int l = llo; l <= lhi; ++l) {
            const double in = ((l == lhi ? hi : T.edge[l + 1]) - (l == llo ? lo : T.edge[l])) * scl;
            const LayV<R> ly = lay_at(T, l);
            D.length(off + l, w * in, (double)ly.a, (double)ly.b);
        }
    }
    if (turn) {
        const LayV<R> ly = lay_at(T, lP);
        const V3<R> dd = um - u;
        D.scatter(off + lP, w, dturn_dg((double)ly.g, (double)ly.fsl, (double)dot(dd, dd)), (double)ly.b);
    }
    return u;
}

// The wave's vertices: vertex i of its chains in order, the first `M` in LDS.
template <class R> struct WaveStrip {
    LdsPtr<R> lds;
    const Vtx<R>* g; // vertex 0 of the wave's first chain
    size_t C;
    int M;
    // vertex v of chain q, whose vertex 0 is vertex `at` of the wave
    __device__ __forceinline__ V3<R> p(int at, int v, int q) const {
        const int i = at + v;
        if (i < M) return pos(lds_ld<R>(lds + i));
        return pos(g[(size_t)v * C + q]);
    }
};

// Layers of a medium from which a score pass whose sums go straight to the
// caller's array (chains of more than two targets in the block) shares
// segments: with fewer, the items of a window, which are one path's, add to the
// same few sums, while the lanes' own segments go to as many targets (16,384
// homogeneous chains, mean n 16, 16 neighbours per target: 629 us shared, 301 by
// lanes; of 100 layers, each chain with another target: 307 and 317).
constexpr int SCORE_LAYERS = 16;

// Whether a wave shares its chains' segments, or each lane walks its own chain.
// An item of the shared form costs more than a step of a walk, which keeps what
// the segment before left (both form a direction and two layer points, the
// gradients three segments instead of one), and a window of items of several
// targets loads a target per lane; a walk waits for the wave's longest path.
// The weights are fitted to both forms over mean lengths of 3 to 42, ragged and
// even, 1, 4, 16 and 64 targets per wave, 16,384 and 524,288 chains; they leave
// the choice of the shared form where the two are close, since a launch of both
// forms fetches the code of both.  Vertices beyond the strip are read where they
// lie, once for each of their segments, so an item costs more the more of them
// there are (from four strips on; two regions, 524,288 ragged chains of mean 42,
// log p: 732 and 390).  us, shared and by lanes: log p, even layers,
// 524,288 chains, mean n 6, longest of a wave 16: 68 and 67, all 12: 82 and 40;
// homogeneous, mean 42: 572 and 232; mixture, 16,384 chains, mean 11: 52 and 80;
// FP64 gradients, 16,384 chains, even layers, mean 17: 92 and 129, all 12: 50 and 26;
// score sums, 524,288 chains, all 12: 167 and 121.
template <class R, bool DV, int KIND, bool SCORE>
__device__ __forceinline__ bool shares_segments(int n, int t, int lane, int total, int strip, bool few) {
    constexpr bool F64 = sizeof(R) == 8;
    const int left = __shfl_up(t, 1, WAVE);
    const int more = __popcll(__ballot(lane > 0 && t >= 0 && left != t)); // targets after the first
    const int chains = __popcll(__ballot(n > 0)), windows = (total - chains + WAVE - 1) / WAVE;
    // in eighths of a step of a walk
    int item = SCORE ? 13
               : DV  ? (F64 || KIND == GK_ANY ? 14 : 18)
               : F64 ? (KIND == GK_ANY ? 10 : 12)
                     : KIND == GK_ANY ? (few ? 12 : 17) : KIND == GK_EVEN ? (few ? 18 : 24) : (few ? 20 : 28);
    const int load = F64 ? 5 : 8;
    if (total > strip) item += F64 ? item / 8 : SCORE || total <= 4 * strip ? item / 4 : 3 * item / 4;
    const int cost = item * windows + load * min(windows, more);
    return __any(8 * (n - 1) >= cost);
}

// LDS of a block: the media tables (tab_bytes, 0: read from HBM), the waves'
// strips (`strip` vertices each), per wave and chain log p and (lweight) the
// path length, the score table (lds_rows rows).
// DV: the vertex gradients are wanted too; SCORE: the score sums.
template <class R, bool DV, int KIND, bool SCORE>
__global__ void __launch_bounds__(256, sizeof(R) == 4 ? 3 : 1) grad_kernel(KArgs a, double* logp_out, Vtx<R>* dv,
                                                                          double* score, int L_total, int lds_rows,
                                                                          int lweight, int strip, int tab_bytes,
                                                                          int few) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int tmin_s[4], tmax_s[4];
    const size_t C = (size_t)a.C;
    const size_t row = 1 + 3 * (size_t)L_total;
    const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
    unsigned char* const behind = smem + tab_bytes + (size_t)4 * strip * sizeof(Vtx<R>);
    double* const slp = (double*)behind + wave * WAVE;
    double* const sL = (double*)behind + (4 + wave) * WAVE;
    double* const tab = (double*)behind + (lweight ? 8 : 4) * WAVE;
    const int c = blockIdx.x * blockDim.x + threadIdx.x, c0 = c - lane;
    int t = -1, n = 0;
    if (c < a.C) {
        t = a.target[c];
        n = a.n[c];
        if (t < 0 || t >= a.T || n < 2 || n > a.cap || a.medium[t] < 0 || a.medium[t] >= a.n_media) {
            if (logp_out) logp_out[c] = __builtin_nan("");
            t = -1;
            n = 0;
        }
    }
    MedTab<R> mt = hbm_tab<R>(a);
    if (KIND != GK_HOM && tab_bytes) mt = stage_tables<R>(a, smem);
    // block-uniform choice of the score destination
    bool local = false;
    int tmin = 0;
    if (SCORE && lds_rows > 0) {
        tmin = block_min_i32(t < 0 ? 0x7fffffff : t, tmin_s);
        const int tmax = block_max_i32(t, tmax_s);
        local = tmax >= 0 && tmax - tmin < lds_rows;
        if (local)
            for (size_t i = threadIdx.x; i < (size_t)lds_rows * row; i += blockDim.x) tab[i] = 0.0;
    }
    __syncthreads();
    const uint64_t some = __ballot(t >= 0);
    if (some) {
        const int upto = wave_prefix(n), at = upto - n;
        const int total = __builtin_amdgcn_readlane(upto, WAVE - 1);
        const bool share = SCORE && !local ? KIND != GK_HOM && L_total >= SCORE_LAYERS * a.n_media
                                           : shares_segments<R, DV, KIND, SCORE>(n, t, lane, total, strip, few);
        // the strip: all vertices, or nothing where a lane per chain reads the
        // paths' rows as they lie
        const WaveStrip<R> S{(LdsPtr<R>)((L4<R>*)(smem + tab_bytes) + (size_t)wave * strip), (const Vtx<R>*)a.verts + c0, C,
                             share || total <= strip ? strip : 0};
        for (int v = 0; S.M > 0 && __any(v < n); v += 4) {
            L4<R> x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (v + i < n && at + v + i < strip) x[i] = *(const L4<R>*)(S.g + ((size_t)(v + i) * C + lane));
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (v + i < n && at + v + i < strip) S.lds[at + v + i] = x[i];
        }
        slp[lane] = 0.0;
        if (lweight) sL[lane] = 0.0;
        if (DV && t >= 0) dv[c] = Vtx<R>{(R)0, (R)0, (R)0, (R)0}; // (vertex 0 never moves)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        auto load = [&](int tt, Tgt<R>& T) __attribute__((always_inline)) {
            load_target(a, tt, T, mt);
            if (KIND == GK_HOM) {
                T.mcnt = 1;
                T.hom = true;
            }
            if (KIND == GK_EVEN) {
                T.hom = false;
                T.uniform = 1;
            }
            T.sl = KIND == GK_ANY;
            if (KIND != GK_ANY) T.l0.fsl = (R)0;
        };
        auto dst = [&](int tt) __attribute__((always_inline)) {
            return ScoreDst{local ? tab + (size_t)(tt - tmin) * row : score + (size_t)tt * row, local};
        };
        // the weight of a chain in the score (0: it does not count), added to its target's
        auto weight = [&](double lp, double L) __attribute__((always_inline)) {
            double w = 0.0;
            if (t >= 0 && isfinite(lp) && a.status[c] == 0) {
                const double* lw = a.logw ? a.logw + (size_t)t * (a.cap + 1) : nullptr;
                w = lw ? exp(-lw[n]) : 1.0;
                if (lweight) w *= L;
            }
            if (w != 0.0) atomicAdd(dst(t).row, w);
            return w;
        };
        if (!share && t >= 0) {
            Tgt<R> T;
            load(t, T);
            PathWalk<R, DV> walk(T, S.p(at, 0, lane));
            V3<R> f = S.p(at, 1, lane), g, g1;
            double L = 0.0;
            for (int k = 1; k < n; ++k) {
                const V3<R> next = S.p(at, k + 1 < n ? k + 1 : k, lane);
                if (lweight) {
                    const V3<R> d = f - walk.fprev;
                    L += sqrt((double)dot(d, d));
                }
                walk.step(T, f, g);
                if (DV && k >= 3) dv[(size_t)(k - 2) * C + c] = Vtx<R>{g.x, g.y, g.z, (R)0};
                f = next;
            }
            const double lp = walk.finish(T, g, g1);
            if (logp_out) logp_out[c] = lp;
            if (DV) {
                if (n >= 3) dv[(size_t)(n - 2) * C + c] = Vtx<R>{g.x, g.y, g.z, (R)0};
                dv[(size_t)(n - 1) * C + c] = Vtx<R>{g1.x, g1.y, g1.z, (R)0};
            }
            if (SCORE) {
                const double w = weight(lp, L);
                if (w != 0.0) {
                    const ScoreDst D = dst(t);
                    const int off = a.minfo[a.medium[t]].off;
                    V3<R> f0 = S.p(at, 0, lane), f1 = S.p(at, 1, lane), um = f0;
                    for (int k = 0; k < n - 1; ++k) {
                        const V3<R> next = S.p(at, k + 2 < n ? k + 2 : k + 1, lane);
                        um = segment_score(T, off, D, w, f0, f1, k > 0, um);
                        f0 = f1;
                        f1 = next;
                    }
                }
            }
        }
        if (share) {
            // the lane's target at the moment: its item's, loaded when it changes
            // (the chains of a target are neighbours, so mostly once)
            Tgt<R> T;
            int tc = __builtin_amdgcn_readlane(t, __ffsll((unsigned long long)some) - 1);
            load(tc, T);
            WaveItems it;
            it.init(lane, n > 0 ? n - 1 : 0);
            while (it.more()) {
                int q, k;
                const bool has = it.next(q, k);
                const int aq = __shfl(at, q, WAVE), nq = __shfl(n, q, WAVE), tq = __shfl(t, q, WAVE);
                if (__any(has && tq != tc)) {
                    tc = has ? tq : tc;
                    load(tc, T);
                }
                if (has) {
                    auto p = [&](int v) __attribute__((always_inline)) { return S.p(aq, v, q); };
                    double f;
                    if constexpr (DV) {
                        V3<R> g;
                        const V3<R> f5[5] = {p(k > 0 ? k - 1 : 0), p(k), p(k + 1), p(k + 2 < nq ? k + 2 : k + 1),
                                             p(k + 3 < nq ? k + 3 : k + 1)};
                        Seg<R> A;
                        f = segment_grad(T, nq, k, f5, g, A);
                        dv[(size_t)(k + 1) * C + c0 + q] = Vtx<R>{g.x, g.y, g.z, (R)0};
                    } else {
                        R tb;
                        f = walk_term(T, nq, k, p(k), p(k + 1), p(k + 2 < nq ? k + 2 : k + 1), tb);
                    }
                    atomicAdd(slp + q, f);
                    if (lweight) {
                        // weight by the path length (FP64 sum of the segment lengths)
                        const V3<R> d = p(k + 1) - p(k);
                        atomicAdd(sL + q, sqrt((double)dot(d, d)));
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            const double lp = slp[lane];
            if (t >= 0 && logp_out) logp_out[c] = lp;
            if (SCORE) {
                const double w = weight(lp, lweight ? sL[lane] : 0.0);
                it.init(lane, w != 0.0 ? n - 1 : 0);
                while (it.more()) {
                    int q, k;
                    const bool has = it.next(q, k);
                    const int aq = __shfl(at, q, WAVE), tq = __shfl(t, q, WAVE);
                    const double wq = __shfl(w, q, WAVE);
                    if (__any(has && tq != tc)) {
                        tc = has ? tq : tc;
                        load(tc, T);
                    }
                    if (has) {
                        const V3<R> f0 = S.p(aq, k, q), f1 = S.p(aq, k + 1, q);
                        const V3<R> um = unit_dir(S.p(aq, k > 0 ? k - 1 : 0, q), f0);
                        segment_score(T, a.minfo[a.medium[tc]].off, dst(tc), wq, f0, f1, k > 0, um);
                    }
                }
            }
        }
    }
    if (SCORE && local) {
        // layer sums to derivatives
        __syncthreads();
        for (size_t i = threadIdx.x; i < (size_t)lds_rows * (1 + (size_t)L_total); i += blockDim.x) {
            const size_t r = i / (1 + (size_t)L_total), l = i % (1 + (size_t)L_total), tt = tmin + r;
            if (tt >= (size_t)a.T) continue;
            if (l == 0) {
                const double w = tab[r * row];
                if (w != 0.0) atomicAdd(score + tt * row, w);
                continue;
            }
            const double* s = tab + r * row + 1 + 3 * (l - 1);
            if (s[0] == 0.0 && s[1] == 0.0 && s[2] == 0.0) continue;
            const R* ly = (const R*)a.lay + (l - 1) * LY_NW;
            const double av = (double)ly[LY_A], bv = (double)ly[LY_B];
            double* o = score + tt * row + 1 + 3 * (l - 1);
            const double d0 = bv * bv * s[0] - bv * s[1];
            if (d0 != 0.0) atomicAdd(o, d0);
            if (s[0] != 0.0) atomicAdd(o + 1, av * av * s[0]);
            if (s[2] != 0.0) atomicAdd(o + 2, s[2]);
        }
    }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_run(const KArgs& a, int block, hipStream_t s) {
    if (a.prec == RJPATH_F64) {
        if (a.sampler == RJPATH_MALA) return launch_run_v<double, 1>(a, block, s);
        if (a.sampler == RJPATH_LMALA) return launch_run_v<double, 2>(a, block, s);
        if (a.sampler == RJPATH_TREE) return launch_run_v<double, 3>(a, block, s);
        return launch_run_v<double, 0>(a, block, s);
    }
    if (a.sampler == RJPATH_MALA) return launch_run_v<float, 1>(a, block, s);
    if (a.sampler == RJPATH_LMALA) return launch_run_v<float, 2>(a, block, s);
    if (a.sampler == RJPATH_TREE) return launch_run_v<float, 3>(a, block, s);
    return launch_run_v<float, 0>(a, block, s);
}

template <class R> static hipError_t set_grad_lds_limit() {
    const void* fns[] = {
        (const void*)grad_kernel<R, false, GK_ANY, false>,  (const void*)grad_kernel<R, true, GK_ANY, false>,
        (const void*)grad_kernel<R, false, GK_EVEN, false>, (const void*)grad_kernel<R, true, GK_EVEN, false>,
        (const void*)grad_kernel<R, false, GK_HOM, false>,  (const void*)grad_kernel<R, true, GK_HOM, false>,
        (const void*)grad_kernel<R, false, GK_ANY, true>,   (const void*)grad_kernel<R, true, GK_ANY, true>,
        (const void*)grad_kernel<R, false, GK_EVEN, true>,  (const void*)grad_kernel<R, true, GK_EVEN, true>,
        (const void*)grad_kernel<R, false, GK_HOM, true>,   (const void*)grad_kernel<R, true, GK_HOM, true>};
    for (const void* f : fns) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 144 * 1024);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t set_run_lds_limit() {
    hipError_t e = set_lds_limit_v<float, 0>();
    if (e == hipSuccess) e = set_lds_limit_v<float, 1>();
    if (e == hipSuccess) e = set_lds_limit_v<float, 2>();
    if (e == hipSuccess) e = set_lds_limit_v<float, 3>();
    if (e == hipSuccess) e = set_lds_limit_v<double, 0>();
    if (e == hipSuccess) e = set_lds_limit_v<double, 1>();
    if (e == hipSuccess) e = set_lds_limit_v<double, 2>();
    if (e == hipSuccess) e = set_lds_limit_v<double, 3>();
    if (e == hipSuccess) e = set_grad_lds_limit<float>();
    if (e == hipSuccess) e = set_grad_lds_limit<double>();
    return e;
}
__global__ void advance_kernel(uint64_t* counter, uint64_t steps) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *counter += steps;
}

hipError_t launch_advance(uint64_t* counter, uint64_t steps, hipStream_t s) {
    hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(64), 0, s, counter, steps);
    return hipGetLastError();
}

template <class R, int KIND>
static hipError_t launch_grad_t(const KArgs& a, double* logp_out, void* dv, double* score, int L_total, int lweight,
                                hipStream_t s) {
    const int block = 256, grid = (a.C + block - 1) / block;
    // LDS: the media tables (FP32 and FP64 alike, up to 16 KiB), a score table
    // for two targets per block when it fits in 64 KiB, and the waves' strips: 7
    // vertices per chain in FP32, which lets three blocks share a CU
    const size_t row_bytes = sizeof(double) * (1 + 3 * (size_t)L_total);
    const int rows = (score && 2 * row_bytes <= 64 * 1024) ? 2 : 0;
    size_t media = KIND == GK_HOM ? 0 : table_bytes<R>(a);
    if (media > 16 * 1024) media = 0;
    const int strip = (sizeof(R) == 4 ? 7 : 6) * WAVE;
    size_t strips = 4 * (size_t)strip * sizeof(Vtx<R>);
    const size_t lds = media + strips + (lweight ? 8 : 4) * WAVE * sizeof(double) + rows * row_bytes;
    const auto fn = score ? (dv ? grad_kernel<R, true, KIND, true> : grad_kernel<R, false, KIND, true>)
                          : (dv ? grad_kernel<R, true, KIND, false> : grad_kernel<R, false, KIND, false>);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(block), lds, s, a, logp_out, (Vtx<R>*)dv, score, L_total, rows, lweight, strip,
                       (int)media, grid <= 2 * device_cus());
    return hipGetLastError();
}

template <class R>
static hipError_t launch_grad_k(const KArgs& a, double* logp_out, void* dv, double* score, int L_total, int lweight,
                                hipStream_t s) {
    if (!a.has_sl && !a.layered) return launch_grad_t<R, GK_HOM>(a, logp_out, dv, score, L_total, lweight, s);
    if (!a.has_sl && a.even) return launch_grad_t<R, GK_EVEN>(a, logp_out, dv, score, L_total, lweight, s);
    return launch_grad_t<R, GK_ANY>(a, logp_out, dv, score, L_total, lweight, s);
}

hipError_t launch_grad(const KArgs& a, double* logp_out, void* dv, double* score, int L_total, int lweight,
                       hipStream_t s) {
    if (a.prec == RJPATH_F64) return launch_grad_k<double>(a, logp_out, dv, score, L_total, lweight, s);
    return launch_grad_k<float>(a, logp_out, dv, score, L_total, lweight, s);
}

} // namespace rj
