// rj_observe.hip -- estimators evaluated on snapshots of the chains' current
// paths (between sampler launches):
//  - the relative light yield of two sensors of one source by the geometric
//    bridge estimator over the cylinder map T (Sec. "Comparison of relative
//    light yield"; App. "Relative light yield transformation");
//  - per-target path-length histograms (Sec. "Comparison of timing
//    distributions": the arrival time is the path length over the speed of
//    light in the bulk).
// Both weight a chain by 1/w(n) so that tilted chains estimate untilted
// expectations, and both sum a block's lanes into an LDS table when the block
// covers at most two keys (targets are contiguous in the chain array), else
// add per lane.
#include <hip/hip_runtime.h>

#include "rj_kernels.h"
#include "rj_step.h"
#include "rj_wave.h"

namespace rj {

namespace {

constexpr int BLK = 256;

__device__ __forceinline__ uint32_t group_hash(uint32_t x) {
    // the chain -> jackknife group hash of the intensity estimator
    x ^= x >> 16;
    x *= 0x85ebca6bu;
    x ^= x >> 13;
    x *= 0xc2b2ae35u;
    x ^= x >> 16;
    return x;
}

using D3 = V3<double>;

__device__ __forceinline__ D3 cross(D3 a, D3 b) {
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ __forceinline__ D3 unit(D3 a) { return (1.0 / sqrt(dot(a, a))) * a; }
__device__ __forceinline__ D3 ld3(const double* p) { return {p[0], p[1], p[2]}; }

// ---------------------------------------------------------------------------
// The map T from paths ending on sensor 0 (target t0) to paths ending on
// sensor 1 (target t1) of the same source, in FP64.
//  Straight frame: k0 points from the source to sensor 0's centre, b0 = the
//  distance to its surface; interior vertex f has coordinates
//  (xbar, ybar, omega) = (f.m0, f.n0, f.k0) / b0.
//  Cylinder frame: k1 = the emission axis, the cylinder's tangent at the
//  source; m1 = minus the unit part of (sensor 1 - source) normal to k1, so the
//  axis of curvature passes through -r_C m1; n1 = k1 x m1; m0 = the unit part
//  of m1 normal to k0 and n0 = k0 x m0.  r_C = |B| / (2 sin psi) with
//  cos psi = k1 . B_hat puts sensor 1's centre on the circle at angle 2 psi;
//  Omega = 2 psi - R1 / r_C stops the image of the axis one sensor radius of
//  arc short of it, and b1 = r_C Omega.
//  Interior vertex: f -> -r_C m1 + (r_C + xbar b1)(cos(omega Omega) m1 +
//  sin(omega Omega) k1) + ybar b1 n1, with |dT/df| = b1^2 Omega (r_C + xbar b1) / b0^3;
//  defined for r_C + xbar b1 > 0 and |omega Omega| < pi.
//  End point: its offset from sensor 0's centre, in units of R0, is turned by
//  the rotation taking (m0, n0, k0) to the arrival frame (cos Omega m1 +
//  sin Omega k1, n1, -sin Omega m1 + cos Omega k1) and scaled to R1; the
//  surface element scales by (R1 / R0)^2.
// ---------------------------------------------------------------------------
struct YMap {
    D3 m0, n0, k0, m1, n1, k1, ar, at, e0, e1;
    double b0, b1, rC, Om, R0, R1, lc, le;
    bool ok;
};

__device__ YMap ymap(const KArgs& a, int t0, int t1) {
    YMap M;
    const D3 s0 = ld3(a.src + 3 * t0);
    M.e0 = ld3(a.sensor + 3 * t0) - s0;
    M.e1 = ld3(a.sensor + 3 * t1) - ld3(a.src + 3 * t1);
    M.R0 = a.radius[t0];
    M.R1 = a.radius[t1];
    const double D0 = sqrt(dot(M.e0, M.e0));
    M.k0 = (1.0 / D0) * M.e0;
    M.b0 = D0 - M.R0;
    const double Bn = sqrt(dot(M.e1, M.e1));
    const D3 Bh = (1.0 / Bn) * M.e1;
    M.k1 = unit(ld3(a.edir + 3 * t0));
    const double cpsi = fmin(1.0, fmax(-1.0, dot(M.k1, Bh)));
    const D3 c = Bh - cpsi * M.k1;
    const double cn = sqrt(dot(c, c));
    const D3 mk = c - dot(c, M.k0) * M.k0; // m1 is -c / |c|: its part normal to k0 is -mk / |c|
    const double mkn = sqrt(dot(mk, mk));
    M.ok = cn > 1e-12 && mkn > 1e-12 * cn && M.b0 > 0;
    if (!M.ok) return M;
    M.m1 = (-1.0 / cn) * c;
    M.n1 = cross(M.k1, M.m1);
    M.m0 = (-1.0 / mkn) * mk;
    M.n0 = cross(M.k0, M.m0);
    const double psi = acos(cpsi);
    M.rC = Bn / (2.0 * sin(psi));
    M.Om = 2.0 * psi - M.R1 / M.rC;
    M.b1 = M.rC * M.Om;
    const double cO = cos(M.Om), sO = sin(M.Om);
    M.ar = cO * M.m1 + sO * M.k1;
    M.at = (-sO) * M.m1 + cO * M.k1;
    M.lc = log(M.b1 * M.b1 * M.Om / (M.b0 * M.b0 * M.b0));
    M.le = 2.0 * log(M.R1 / M.R0);
    M.ok = M.Om > 0 && M.b1 > 0;
    return M;
}

// forward image of an interior vertex; rad <= 0 or |angle| >= pi: outside
__device__ __forceinline__ D3 yfwd(const YMap& M, D3 f, double& rad, bool& in) {
    const double ib0 = 1.0 / M.b0;
    const double xb = dot(f, M.m0) * ib0, yb = dot(f, M.n0) * ib0, om = dot(f, M.k0) * ib0;
    rad = M.rC + xb * M.b1;
    const double ang = om * M.Om;
    in = rad > 0 && fabs(ang) < 3.14159265358979323846;
    double sa, ca;
    sincos(ang, &sa, &ca);
    return (-M.rC) * M.m1 + rad * (ca * M.m1 + sa * M.k1) + (yb * M.b1) * M.n1;
}

__device__ __forceinline__ D3 yinv(const YMap& M, D3 g, double& rad) {
    const D3 v = g + M.rC * M.m1;
    const double pm = dot(v, M.m1), pk = dot(v, M.k1);
    rad = sqrt(pm * pm + pk * pk);
    const double xb = (rad - M.rC) / M.b1, yb = dot(v, M.n1) / M.b1, om = atan2(pk, pm) / M.Om;
    return (xb * M.b0) * M.m0 + (yb * M.b0) * M.n0 + (om * M.b0) * M.k0;
}

__device__ __forceinline__ D3 yend_fwd(const YMap& M, D3 f) {
    const D3 nu = f - M.e0;
    const double s = M.R1 / M.R0;
    return M.e1 + s * (dot(nu, M.m0) * M.ar + dot(nu, M.n0) * M.n1 + dot(nu, M.k0) * M.at);
}

__device__ __forceinline__ D3 yend_inv(const YMap& M, D3 g) {
    const D3 nu = g - M.e1;
    const double s = M.R0 / M.R1;
    return M.e0 + s * (dot(nu, M.ar) * M.m0 + dot(nu, M.n1) * M.n0 + dot(nu, M.at) * M.k0);
}

template <class R> __device__ __forceinline__ D3 vload(const Vtx<R>* base, size_t C, int v) {
    const Vtx<R> x = base[(size_t)v * C];
    return {(double)x.x, (double)x.y, (double)x.z};
}

// Block-level accumulation of (key, group, slot) sums: an LDS table when the
// block's keys span at most two values, else one atomic per lane.
struct BlockSums {
    double* tab;
    int kmin;
    bool local;
};

__device__ __forceinline__ BlockSums block_sums_begin(int key, double* tab, int nent_per_key, int* smin, int* smax) {
    BlockSums b;
    b.tab = tab;
    b.kmin = block_min_i32(key < 0 ? 0x7fffffff : key, smin);
    const int kmax = block_max_i32(key, smax);
    b.local = kmax >= 0 && kmax - b.kmin <= 1 && tab != nullptr;
    if (b.local) {
        for (int i = threadIdx.x; i < 2 * nent_per_key; i += blockDim.x) tab[i] = 0.0;
    }
    __syncthreads();
    return b;
}

__device__ __forceinline__ void block_sums_end(const BlockSums& b, double* out, int nent_per_key, int nkeys) {
    if (!b.local) return;
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * nent_per_key; i += blockDim.x) {
        const int k = b.kmin + i / nent_per_key;
        if (b.tab[i] != 0.0 && k < nkeys) atomicAdd(out + (size_t)b.kmin * nent_per_key + i, b.tab[i]);
    }
}

// ---------------------------------------------------------------------------
// Bridge sums.  role[t] = 2 k + side for a target in pair k (pairs[2k] = t0,
// pairs[2k + 1] = t1), else -1.  A chain of t0 (path x) takes
// log r = log p_t1(T x) + log|dT/dx| - log p_t0(x) (-inf outside T's domain);
// a chain of t1 (path y) takes log r = log p_t0(T^-1 y) - log p_t1(y) - log|dT/dx|
// at x = T^-1 y.  acc[((k * 2 + side) * groups + g) * 2 + {0, 1}] += {sqrt(r), 1} / w(n).
//
// Work split.  A wave owns `cpw` chains (64, or fewer where the chains would
// leave SIMDs without a wave) and shares their vertices over its lanes: a lane
// maps one vertex and takes the next two, of the path and of its image, from
// the lanes beside it (windows of 62), so that the map's FP64 sine, cosine or
// arc tangent is formed once per vertex and no lane waits for the longest
// path.  One lane per chain, mapping every vertex twice, took the kernel 545 us
// for the two-region test's 65,536 chains of 32 vertices; shared, 180 us.
// Where a wave has many targets or short paths of one length, a lane per chain
// is the better form (lane_densities, which maps a vertex once).
// ---------------------------------------------------------------------------
template <class R> __device__ __forceinline__ V3<R> lane_v3(V3<R> p, int from) {
    return {__shfl(p.x, from, WAVE), __shfl(p.y, from, WAVE), __shfl(p.z, from, WAVE)};
}

// Whether a wave shares its chains' vertices, or each lane maps its own chain's.
// A window of 62 shared vertices takes about as long as two of a lane's own, and
// every target of the wave has windows and a map to itself.  The call in us,
// shared and by lanes (262,144 chains of the two-region geometry, FP32): mean n
// 42, chains of a target together 850 and 1185, every n 6 119 and 80; dealt out
// over 128 targets, mean n 42, 2060 and 1260, mean 4 1605 and 107 (FP64, 65,536
// chains of mean n 10: 850 and 245).
template <class R> __device__ __forceinline__ bool shares_vertices(int items, int tc, int total) {
    constexpr int WINDOW = sizeof(R) == 4 ? 18 : 13, TARGET = sizeof(R) == 4 ? 4 : 3; // eighths of a lane's vertex
    int targets = 0;
    for (uint64_t rest = __ballot(items > 0); rest; ++targets) {
        const int tq = __builtin_amdgcn_readlane(tc, __ffsll((unsigned long long)rest) - 1);
        rest &= ~__ballot(tc == tq);
    }
    const int windows = max(targets, (total + (WAVE - 2) / 2 * (targets + 1)) / (WAVE - 2));
    return __any(8 * (items + 2) >= WINDOW * windows + TARGET * targets);
}

// One chain by one lane: `f(v)` is vertex v of its path of n vertices.  lp: log p
// of the path; img: of its image, +- log |dT/dx|; returns the chain's `outside`.
template <class R, class F>
__device__ __forceinline__ int lane_densities(const KArgs& a, int own, int other, int side, int n, F f, double& lp,
                                              double& img) {
    lp = img = 0.0;
    {
        const YMap M = ymap(a, side == 0 ? own : other, side == 0 ? other : own);
        if (!M.ok) return 2;
        Tgt<R> T;
        load_target(a, other, T, hbm_tab<R>(a));
        double lj = M.le + (n - 2) * M.lc;
        PathWalk<R, false> walk(T, f(0));
        V3<R> x = f(1), g;
        for (int k = 1; k < n; ++k) {
            const V3<R> next = f(k + 1 < n ? k + 1 : k);
            const D3 d = {(double)x.x, (double)x.y, (double)x.z};
            D3 y;
            if (k == n - 1) {
                y = side == 0 ? yend_fwd(M, d) : yend_inv(M, d);
            } else {
                double rad;
                bool in = true;
                if (side == 0) y = yfwd(M, d, rad, in);
                else y = yinv(M, d, rad);
                if (!in) return 1;
                lj += log(rad);
            }
            walk.step(T, V3<R>{(R)y.x, (R)y.y, (R)y.z}, g);
            x = next;
        }
        img = walk.finish(T, g, g) + (side == 0 ? lj : -lj);
    }
    Tgt<R> T;
    load_target(a, own, T, hbm_tab<R>(a));
    PathWalk<R, false> walk(T, f(0));
    V3<R> x = f(1), g;
    for (int k = 1; k < n; ++k) {
        const V3<R> next = f(k + 1 < n ? k + 1 : k);
        walk.step(T, x, g);
        x = next;
    }
    lp = walk.finish(T, g, g);
    return 0;
}

template <class R>
__global__ void __launch_bounds__(BLK, sizeof(R) == 4 ? 2 : 1)
    yield_kernel(KArgs a, int n_pairs, const int32_t* pairs, const int32_t* role, int groups, double* acc, double* logr,
                 int cpw, int strip) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double tab[2 * 64 * 2];
    __shared__ double own[BLK], img[BLK];
    __shared__ int outside[BLK];
    __shared__ YMap map[BLK / WAVE];
    __shared__ Tgt<R> tgt[BLK / WAVE][2];
    __shared__ int smin[BLK / 64], smax[BLK / 64];
    const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
    const int c0 = ((int)blockIdx.x * (BLK / WAVE) + wave) * cpw, c = c0 + lane;
    const bool mine = lane < cpw && c < a.C;
    int key = -1, tc = -1, to = -1, n = 0;
    if (mine) {
        tc = a.target[c];
        n = a.n[c];
        if (tc >= 0 && tc < a.T && a.status[c] == 0 && n >= 2 && n <= a.cap) {
            const int r = role[tc];
            const int k = r >> 1;
            if (r >= 0 && k < n_pairs && pairs[r] == tc) {
                to = pairs[2 * k + ((r & 1) ^ 1)];
                if (to >= 0 && to < a.T && to != tc && a.medium[to] == a.medium[tc] &&
                    a.medium[tc] >= 0 && a.medium[tc] < a.n_media && a.src[3 * to] == a.src[3 * tc] &&
                    a.src[3 * to + 1] == a.src[3 * tc + 1] && a.src[3 * to + 2] == a.src[3 * tc + 2])
                    key = r;
            }
        }
    }
    // log p of the path; log p of its image +- log |dT/dx|; 1: outside T's
    // domain (log r = -inf, whatever the densities), 2: no map for the pair
    double* const sown = own + wave * WAVE;
    double* const simg = img + wave * WAVE;
    int* const sout = outside + wave * WAVE;
    sown[lane] = 0.0;
    simg[lane] = 0.0;
    sout[lane] = 0;
    const int items = key >= 0 ? n : 0;
    const int upto = wave_prefix(items), at = upto - items, total = __builtin_amdgcn_readlane(upto, WAVE - 1);
    if (!shares_vertices<R>(items, tc, total)) {
        if (key >= 0) {
            const Vtx<R>* const path = (const Vtx<R>*)a.verts + c;
            sout[lane] = lane_densities<R>(
                a, tc, to, key & 1, n, [&](int v) __attribute__((always_inline)) { return pos(path[(size_t)v * a.C]); },
                sown[lane], simg[lane]);
        }
    } else if (total > 0) {
        // the vertices, read row by row into the wave's strip
        const LdsPtr<R> lds = (LdsPtr<R>)((L4<R>*)smem + (size_t)wave * strip);
        const Vtx<R>* const g = (const Vtx<R>*)a.verts + c0;
        const size_t C = (size_t)a.C;
        {
            const int q = lane & (cpw - 1), rows = WAVE / cpw;
            const int nq = __shfl(items, q, WAVE), aq = __shfl(at, q, WAVE);
            for (int v = lane / cpw; __any(v < nq); v += 4 * rows) {
                L4<R> x[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (v + i * rows < nq && aq + v + i * rows < strip)
                        x[i] = *(const L4<R>*)(g + ((size_t)(v + i * rows) * C + q));
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (v + i * rows < nq && aq + v + i * rows < strip) lds[aq + v + i * rows] = x[i];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        // target by target (one or two per wave where the chains of a target are
        // neighbours); the map and the two targets are kept in LDS (together
        // they would take 170 registers) and read where they are used
        const YMap& M = map[wave];
        uint64_t rest = __ballot(items > 0);
        while (rest) {
            const int from = __ffsll((unsigned long long)rest) - 1;
            const int tq = __builtin_amdgcn_readlane(tc, from), oq = __builtin_amdgcn_readlane(to, from);
            const int side = __builtin_amdgcn_readlane(key, from) & 1;
            const bool in_target = items > 0 && tc == tq;
            rest &= ~__ballot(in_target);
#pragma unroll 1
            for (int w = 0; w < 2; ++w) {
                Tgt<R> T;
                load_target(a, w == 0 ? tq : oq, T, hbm_tab<R>(a));
                if (lane == 0) tgt[wave][w] = T;
            }
            {
                const YMap m = ymap(a, side == 0 ? tq : oq, side == 0 ? oq : tq);
                if (lane == 0) map[wave] = m;
                if (in_target && !m.ok) sout[lane] = 2;
                if (!__builtin_amdgcn_readfirstlane(m.ok)) continue;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            WaveItems it;
            it.init(lane, in_target ? n : 0);
            while (it.more()) {
                asm volatile("" ::: "memory"); // (what LDS holds is read again, not kept)
                int q, k;
                const bool has = it.next(q, k);
                it.base -= 2; // (the last two lanes only lend their vertices)
                it.seen -= it.starts_at_end(2);
                const int aq = __shfl(at, q, WAVE), nq = __shfl(n, q, WAVE);
                V3<R> f = {(R)0, (R)0, (R)0}, h = f;
                double lj = 0.0;
                bool in = true;
                if (has) {
                    f = aq + k < strip ? pos(lds_ld<R>(lds + aq + k)) : pos(g[(size_t)k * C + q]);
                    const D3 x = {(double)f.x, (double)f.y, (double)f.z};
                    D3 y = x;
                    if (k == nq - 1) {
                        y = side == 0 ? yend_fwd(M, x) : yend_inv(M, x);
                    } else if (k > 0) {
                        double rad;
                        if (side == 0) y = yfwd(M, x, rad, in);
                        else y = yinv(M, x, rad);
                        lj = log(rad);
                    }
                    if (k == 0) lj = M.le + (nq - 2) * M.lc;
                    h = {(R)y.x, (R)y.y, (R)y.z};
                }
                // the image's walk, then the path's
                double term = side == 0 ? lj : -lj;
                V3<R> e = h;
#pragma unroll 1
                for (int w = 1; w >= 0; --w) {
                    const V3<R> e1 = lane_v3(e, lane + 1), e2 = lane_v3(e, lane + 2);
                    if (has && lane < WAVE - 2) {
                        if (k < nq - 1) {
                            const Tgt<R> T = tgt[wave][w];
                            R tb;
                            term += walk_term(T, nq, k, e, e1, e2, tb);
                        }
                        atomicAdd((w == 0 ? sown : simg) + q, term);
                        if (!in) sout[q] = 1;
                    }
                    term = 0.0;
                    e = f;
                }
            }
        }
    }
    __syncthreads();
    double lr = __builtin_nan("");
    if (key >= 0) {
        if (sout[lane] != 2) lr = sout[lane] ? -__builtin_inf() : simg[lane] - sown[lane];
        if (lr != lr || lr == __builtin_inf()) key = -1; // a non-finite own density, or no map: not a sample
    }
    if (mine && logr) logr[c] = lr;
    const int gr = (int)(group_hash((uint32_t)c) % (uint32_t)groups);
    const int nent = groups * 2;
    BlockSums b = block_sums_begin(key, tab, nent, smin, smax);
    if (key >= 0) {
        const double* lw = a.logw ? a.logw + (size_t)tc * (a.cap + 1) : nullptr;
        const double iw = lw ? exp(-lw[n]) : 1.0;
        const double s = lr == -__builtin_inf() ? 0.0 : exp(0.5 * lr);
        double* dst = b.local ? tab + (size_t)(key - b.kmin) * nent : acc + (size_t)key * nent;
        atomicAdd(dst + 2 * gr, iw * s);
        atomicAdd(dst + 2 * gr + 1, iw);
    }
    block_sums_end(b, acc, nent, 2 * n_pairs);
}

// ---------------------------------------------------------------------------
// Path-length histogram: hist[t * (bins + 1) + b] += 1 / w(n) for
// b = floor((L - l0) / width) in [0, bins), and hist[t * (bins + 1) + bins]
// += 1 / w(n) for every sample (the normaliser).  L is summed in FP64.
//
// A chain's segments are split over 64 / cpw lanes, lane p * cpw + q taking
// part p of the wave's chain q (rows of whole cache lines).  The rows come from
// HBM one latency per four, so few chains with long paths need more waves than
// one lane each gives; a block keeps 256 chains, so that its table is added
// to the result as seldom.  The two-region test's 65,536 chains of 32 vertices:
// 70 us with one lane each, 33 with four (the paths' 34 MB take 7 at the rate
// of a large copy).
// ---------------------------------------------------------------------------
constexpr int LHIST_PARTS = 4;

template <class R>
__global__ void __launch_bounds__(BLK * LHIST_PARTS) lhist_kernel(KArgs a, int bins, double l0, double width,
                                                                  double* hist, int use_lds, int cpw) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int smin[BLK * LHIST_PARTS / 64], smax[BLK * LHIST_PARTS / 64];
    const int lane = threadIdx.x % WAVE, part = lane / cpw, parts = WAVE / cpw;
    const int c = (blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE) * cpw + lane % cpw;
    int t = -1, n = 0;
    if (c < a.C) {
        t = a.target[c];
        n = a.n[c];
        if (t < 0 || t >= a.T || a.status[c] != 0 || n < 2 || n > a.cap) t = -1;
    }
    double L = 0;
    if (t >= 0) {
        // segments first .. last - 1, four rows in flight
        const int each = (n - 1 + parts - 1) / parts, first = part * each, last = min(first + each, n - 1);
        if (first < last) {
            const Vtx<R>* base = (const Vtx<R>*)a.verts + c;
            D3 p = vload(base, (size_t)a.C, first);
            for (int v = first + 1; v <= last; v += 4) {
                D3 q[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (v + i <= last) q[i] = vload(base, (size_t)a.C, v + i);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (v + i <= last) {
                        const D3 d = q[i] - p;
                        L += sqrt(dot(d, d));
                        p = q[i];
                    }
            }
        }
    }
    for (int m = cpw; m < WAVE; m *= 2) L += __shfl_xor(L, m, WAVE);
    if (part > 0) t = -1; // (the first part's lane counts the chain)
    const int nent = bins + 1;
    BlockSums b = block_sums_begin(t, use_lds ? (double*)smem : nullptr, nent, smin, smax);
    if (t >= 0) {
        const double* lw = a.logw ? a.logw + (size_t)t * (a.cap + 1) : nullptr;
        const double iw = lw ? exp(-lw[n]) : 1.0;
        double* dst = b.local ? (double*)smem + (size_t)(t - b.kmin) * nent : hist + (size_t)t * nent;
        const double x = floor((L - l0) / width);
        if (x >= 0 && x < (double)bins) atomicAdd(dst + (int)x, iw);
        atomicAdd(dst + bins, iw);
    }
    block_sums_end(b, hist, nent, a.T);
}

} // namespace

template <class R>
static hipError_t launch_yield_t(const KArgs& a, int n_pairs, const int32_t* pairs, const int32_t* role, int groups,
                                 double* acc, double* logr, hipStream_t s) {
    // chains per wave: 64 from the resident waves on (two per SIMD, one in FP64,
    // where 65,536 chains of 32 per wave took two rounds: mean n 10 149 us instead
    // of 135), fewer below, down to 8; a strip of 8 KiB per wave, so that two per
    // SIMD fit
    const int resident = (sizeof(R) == 4 ? 8 : 4) * device_cus();
    int cpw = WAVE;
    while (cpw > 8 && (long long)a.C < (long long)resident * cpw) cpw /= 2;
    const int strip = 8 * 1024 / (int)sizeof(Vtx<R>);
    const int chains = BLK / WAVE * cpw, grid = (a.C + chains - 1) / chains;
    hipLaunchKernelGGL(yield_kernel<R>, dim3(grid), dim3(BLK), (size_t)(BLK / WAVE) * 8 * 1024, s, a, n_pairs, pairs, role,
                       groups, acc, logr, cpw, strip);
    return hipGetLastError();
}

hipError_t launch_yield(const KArgs& a, int n_pairs, const int32_t* pairs, const int32_t* role, int groups,
                        double* acc, double* logr, hipStream_t s) {
    if (a.prec == RJPATH_F64) return launch_yield_t<double>(a, n_pairs, pairs, role, groups, acc, logr, s);
    return launch_yield_t<float>(a, n_pairs, pairs, role, groups, acc, logr, s);
}

hipError_t launch_lhist(const KArgs& a, int bins, double l0, double width, double* hist, hipStream_t s) {
    const int grid = (a.C + BLK - 1) / BLK;
    // lanes per chain: as many as keep the launch within four waves per SIMD
    // (chains of mean n 10 and 42, 1, 2 and 4 lanes each, us: 65,536 25, 21, 19 and
    // 98, 67, 52; 131,072 34, 27, 25 and 107, 92, 85, but 17, 17, 18 at mean n 4;
    // 262,144 37, 38, 43 and 165, 165, 193)
    int parts = LHIST_PARTS;
    while (parts > 1 && (long long)a.C * parts > 16LL * device_cus() * WAVE) parts /= 2;
    const dim3 block(BLK * parts);
    const size_t lds = 2 * sizeof(double) * ((size_t)bins + 1);
    const int use = lds <= 64 * 1024;
    if (a.prec == RJPATH_F64)
        hipLaunchKernelGGL(lhist_kernel<double>, dim3(grid), block, use ? lds : 0, s, a, bins, l0, width, hist, use,
                           WAVE / parts);
    else
        hipLaunchKernelGGL(lhist_kernel<float>, dim3(grid), block, use ? lds : 0, s, a, bins, l0, width, hist, use,
                           WAVE / parts);
    return hipGetLastError();
}

} // namespace rj
