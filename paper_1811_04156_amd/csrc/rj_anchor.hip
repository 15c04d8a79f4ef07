// rj_anchor.hip -- the anchor-sector integrals of the intensity estimator.
//
// The chains sample p(f) w(n) up to its normalisation; the integral of p over
// one sector n0 is computed here by deterministic quadrature, so that
// I = I_{n0} * E[1/w(n)] / E[1(n = n0) / w(n0)].
//   n0 = 2: I_2 = int over directions u from the source into the sensor of
//           eps(u) e^{-tau(hit)} rho(nu) dOmega  (dOmega = cos Phi dA / r^2,
//           App. "Final vertex").
//   n0 = 3: I_3 = int dOmega_0 eps(w0) int dr e^{-tau(0 -> r w0)} b(r w0) K(r w0),
//           K = int over directions into the sensor from r w0 of
//               sigma_sr(w0 . u) e^{-tau} rho dOmega  (d^3 f = r^2 dr dOmega_0
//           cancels the 1/|r|^2 of the first segment; App. "Intermediate vertex").
// Emission directions are parametrised by the inverse CDF of eps, which
// absorbs eps into the measure; sensor directions by
// v = sqrt(R^2 - D^2 sin^2 theta) / R (smooth at the cap rim).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rj_device.h"
#include "rj_kernels.h"
#include "rj_math64.h"

namespace rj {

namespace {

const double PI = 3.14159265358979323846;
const double EDGE_GAP = 10.0 * PI / 180.0; // rim gap below which a cone target takes the finer direction rule

__device__ double log_rho(const Tgt<double>& T, V3<double> nu) {
    if (T.dk != RJPATH_DET_PAPER) return 0.0;
    double cr = dot(nu, T.dd);
    return 3 * cr - 1 - log(cosh(2 * cr + 0.7));
}

__device__ void frame(V3<double> ax, V3<double>& e2, V3<double>& e3) { onb(ax, e2, e3); }

__device__ double depth_c(const Tgt<double>& T, V3<double> P, V3<double> Q) {
    V3<double> r = Q - P;
    double len = sqrt(dot(r, r)), tc, tb;
    seg_depth(T, P, Q, len, tc, tb);
    return tc;
}

// int over directions from P into the sensor of wfun(u) e^{-tau} rho dOmega
// (azimuths j0 .. j0 + nj - 1 of the npsi)
template <class W>
__device__ double cap_quad(const Tgt<double>& T, V3<double> P, const double* gx, const double* gw, int nv, int j0, int nj,
                           int npsi, W wfun) {
    V3<double> dv = T.eta - P;
    double D = sqrt(dot(dv, dv)), Rr = (double)T.rad;
    if (!(D > Rr)) return 0.0;
    V3<double> ax = (1.0 / D) * dv, e2, e3;
    frame(ax, e2, e3);
    double k2 = Rr * Rr / (D * D), sum = 0.0;
    for (int i = 0; i < nv; ++i) {
        double v = gx[i], wv = gw[i];
        double s2 = k2 * (1 - v * v);
        double ct = sqrt(1 - s2), st = sqrt(s2);
        double len = D * ct - Rr * v;
        double jac = k2 * v / ct;
        for (int j = j0; j < j0 + nj; ++j) {
            double ps = 2 * PI * (j + 0.5) / npsi;
            double sp, cp;
            sincos(ps, &sp, &cp);
            V3<double> u = ct * ax + st * (cp * e2 + sp * e3);
            V3<double> hit = P + len * u;
            V3<double> nu = (1.0 / Rr) * (hit - T.eta);
            double lw = wfun(u);
            if (lw == -__builtin_inf()) continue;
            sum += wv * (2 * PI / npsi) * jac * exp(lw - depth_c(T, P, hit) + log_rho(T, nu));
        }
    }
    return sum;
}

// direction of the emission inverse CDF at (x, psi); eps dOmega = dx dpsi / (2 pi)
__device__ V3<double> emit_dir_icdf(const Tgt<double>& T, double x, double ps) {
    V3<double> ax = T.ek == RJPATH_EMIT_ISO ? V3<double>{0, 0, 1} : T.ed, e2, e3;
    frame(ax, e2, e3);
    double c;
    if (T.ek == RJPATH_EMIT_ISO) c = 1 - 2 * x;
    else if (T.ek == RJPATH_EMIT_VMF) c = 1 + log(x + (1 - x) * exp(-2 * (double)T.kappa)) / (double)T.kappa;
    else c = 1 - x * (1 - (double)T.ecos);
    double s = sqrt(fmax(0.0, 1 - c * c)), sp, cp;
    sincos(ps, &sp, &cp);
    return c * ax + s * (cp * e2 + sp * e3);
}

// FP64 reciprocal, reciprocal square root and exponential from the hardware's
// starting values (good to 2^-24); arguments here are ordinary positive numbers,
// so the library forms' handling of zeros, infinities and subnormals is not
// needed.  Relative errors stay below 1, 1.5 and 2 times 2^-53.
__device__ __forceinline__ double rcp64(double x) { return rcp_from(x, __builtin_amdgcn_rcp(x)); }
__device__ __forceinline__ double rsq64(double x) { return rsq_from(x, __builtin_amdgcn_rsq(x)); }
__device__ __forceinline__ double exp64(double x) {
    double k;
    const double p = exp_series(x, k);
    return __builtin_amdgcn_ldexp(p, (int)fmax(k, -3000.0));
}

// The total depth from a point P in layer lP (axis coordinate uP) to a point
// of layer lQ at axis coordinate uQ along a direction with axis component du:
// same layer: c len; otherwise (K + B (uQ - e)) / d with d = +-du, the
// piecewise integral between the two coordinates over |du|.
struct DepthTo {
    double K, B, e, sgn, c;
    bool same;
};

__device__ __forceinline__ DepthTo depth_to(const Tgt<double>& T, int lP, double cP, double uP, int lQ) {
    DepthTo d;
    d.c = T.lay[(size_t)lQ * LY_NW + LY_C];
    d.same = lP == lQ;
    const bool up = lP < lQ;
    // up: c_P (edge[lP+1] - uP) + whole layers + c_Q (uQ - edge[lQ]); down: mirrored
    const double eP = T.mcnt == 1 ? uP : T.edge[up ? lP + 1 : lP];
    d.e = T.mcnt == 1 ? uP : T.edge[up ? lQ : lQ + 1];
    const double2 pP = T.pre[up ? lP + 1 : lP], pQ = T.pre[up ? lQ : lQ + 1];
    d.sgn = up ? 1.0 : -1.0;
    d.K = cP * (d.sgn * (eP - uP)) + d.sgn * (pQ.x - pP.x);
    d.B = d.sgn * d.c;
    return d;
}

__device__ __forceinline__ double depth_at(const DepthTo& d, double uQ, double du, double len) {
    if (d.same) return d.c * len; // (uniform over the wave)
    return (d.K + d.B * (uQ - d.e)) * rcp64(d.sgn * du);
}

// Which layers the sensor sphere touches: one layer lA (kind 0), the two
// layers lA, lA + 1 around one edge (kind 1), or more (kind 2).
struct SensorLayers {
    int lA, kind;
    double edge;
};

__device__ __forceinline__ SensorLayers sensor_layers(const Tgt<double>& T) {
    const double uc = axis_u(T, T.eta), Rm = T.rad * (1.0 + 1e-9) + 1e-9;
    SensorLayers S;
    S.lA = layer_u(T, uc - Rm);
    const int lB = layer_u(T, uc + Rm);
    S.kind = lB == S.lA ? 0 : (lB == S.lA + 1 ? 1 : 2);
    S.edge = S.kind == 1 ? T.edge[S.lA + 1] : 0.0;
    return S;
}

// Half of the 8 x 8 cap rule of one ray point for a layer without the
// simplified-Liu term and a uniform angular response: the four azimuths of
// sign `half` (+-1; azimuths j and j + 4 are opposite), all eight polar nodes.
// In the frame (ax, e2, e3) turned by the azimuth, the direction is
// (ct, st, 0) and w0 has components (c0, w2, w3), so
// |w0 - u|^2 = (c0 - ct)^2 + (w2 - st)^2 + w3^2 keeps the forward peak's
// precision, and the scattering function is a power of one reciprocal root.
template <bool TWO>
__device__ __forceinline__ double cap_half(const Tgt<double>& T, const LayV<double>& ly, V3<double> P, double uP, int lP,
                                           V3<double> w0, const SensorLayers& S, double half, const double* x8,
                                           const double* w8) {
    const double CPS[4] = {0.92387953251128675613, 0.38268343236508977173, -0.38268343236508977173,
                           -0.92387953251128675613};
    const double SPS[4] = {0.38268343236508977173, 0.92387953251128675613, 0.92387953251128675613,
                           0.38268343236508977173};
    const V3<double> dv = T.eta - P;
    const double D2 = dot(dv, dv), iD = rsq64(D2), D = D2 * iD, Rr = T.rad;
    const V3<double> ax = iD * dv;
    V3<double> e2, e3;
    onb(ax, e2, e3);
    const double k = Rr * iD, k2 = k * k;
    const V3<double> A = {T.ax, T.ay, T.az};
    const double A0 = dot(A, ax), A2 = half * dot(A, e2), A3 = half * dot(A, e3);
    const double c0 = dot(w0, ax), c2 = half * dot(w0, e2), c3 = half * dot(w0, e3);
    double At[4], w2[4], w3s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        At[j] = CPS[j] * A2 + SPS[j] * A3;
        w2[j] = CPS[j] * c2 + SPS[j] * c3;
        const double w3 = CPS[j] * c3 - SPS[j] * c2;
        w3s[j] = w3 * w3;
    }
    const DepthTo da = depth_to(T, lP, ly.c, uP, S.lA);
    DepthTo db = da;
    if (TWO) db = depth_to(T, lP, ly.c, uP, S.lA + 1);
    const double rhg = ly.hg1, g = ly.g;
    auto polar = [&](int i, double& ct, double& st, double& len, double& wj) __attribute__((always_inline)) {
        const double v = x8[i], sv2 = 1.0 - v * v;
        const double c2v = 1.0 - k2 * sv2, ic = rsq64(c2v);
        ct = c2v * ic;
        st = k * sqrt(sv2);
        len = D * ct - Rr * v;
        wj = w8[i] * v * ic;
    };
    auto depth = [&](double du, double len) __attribute__((always_inline)) {
        const double uQ = uP + len * du;
        const double t = depth_at(da, uQ, du, len);
        if (!TWO) return t;
        const double tb = depth_at(db, uQ, du, len);
        return uQ < S.edge ? t : tb;
    };
    // The depths of a cap differ by little (its size times the coefficients,
    // about 0.01 for a 0.165 m sensor): e^{-tau} = e^{-t0} e^{-(tau - t0)} with
    // the second factor a short series (below 2^-53 at 1/16); polar nodes with
    // a larger spread anywhere in the wave take the full exponential.
    double t0, near = 0.0, rest = 0.0;
    {
        double ct, st, len, wj;
        polar(0, ct, st, len, wj);
        t0 = depth(ct * A0 + st * At[0], len);
    }
#pragma unroll 1
    for (int i = 0; i < 8; ++i) {
        double ct, st, len, wj, p[4], d[4], far = 0.0;
        polar(i, ct, st, len, wj);
        const double a0 = ct * A0, qa = (c0 - ct) * (c0 - ct);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double b = w2[j] - st, q = qa + (b * b + w3s[j]);
            const double r = rsq64(rhg + g * q);
            p[j] = r * r * r;
            d[j] = t0 - depth(a0 + st * At[j], len);
            far = fmax(far, fabs(d[j]));
        }
        double s4 = 0.0;
        if (__all(far < 0.0625)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                double e = 1.0 / 40320.0;
                e = fma(e, d[j], 1.0 / 5040.0);
                e = fma(e, d[j], 1.0 / 720.0);
                e = fma(e, d[j], 1.0 / 120.0);
                e = fma(e, d[j], 1.0 / 24.0);
                e = fma(e, d[j], 1.0 / 6.0);
                e = fma(e, d[j], 0.5);
                e = fma(e, d[j], 1.0);
                e = fma(e, d[j], 1.0);
                s4 = fma(e, p[j], s4);
            }
            near = fma(wj, s4, near);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) s4 = fma(exp64(d[j] - t0), p[j], s4);
            rest = fma(wj, s4, rest);
        }
    }
    const double sum = fma(near, exp64(-t0), rest);
    return sum * k2;
}

// The targets of the lean kernel below: one scattering vertex, no
// simplified-Liu layer, a uniform angular response and a sensor that touches
// at most two layers.  The general kernel serves the rest, so that its library
// calls do not cost the lean one its registers (together: 294 registers, one
// wave per SIMD).
__device__ __forceinline__ bool lean_target(const KArgs& a, int t, const Tgt<double>& T, const SensorLayers& S) {
    return a.n0[t] == 3 && !a.has_sl && T.dk != RJPATH_DET_PAPER && S.kind < 2;
}

// n0 = 3: outer: 32 (inverse-CDF polar) x 32 (azimuth) directions (64 x 64
// near a cone's rim, below); along each
// ray, one 32-point Gauss rule per layer crossed (b jumps and tau kinks
// at the edges) and, past the last edge, the map r = a - log(1-x)/c
// that absorbs the exponential attenuation; inner 8 x 8 cap rule.
// (K peaks sharply in r along rays that pass close to the sensor: on a
// sample of cone targets in a 100-layer medium the 90th-percentile
// error against a finer rule was 7.7e-3 with 16 points per piece and
// 1.7e-3 with 32; more cap or direction nodes gained less per
// evaluation.)
// A sensor just outside a cone's rim sees rays along the rim pass
// close to it, where K peaks in direction as well: such targets (rim
// gap below EDGE_GAP) take 64 x 64 directions.  On cone targets in a
// 100-layer medium, 32 x 32 left errors of 3.5% and 0.9% at gaps of
// 1 and 3 degrees, 64 x 64 below 4e-4; at 8 degrees 32 x 32 was
// already within 1e-4.  (The choice is uniform over the block.)
//
// A wave takes one direction at a time and walks the ray's layer pieces
// together; its lanes are the 32 radial nodes of a piece times the two halves
// of the azimuths, so no lane waits for another ray's pieces.  This block's
// directions: chunk, chunk + nchunk, ... (in units of its waves).
// cap(ly, f1, l, w0, uP, half): the half of K at the ray point f1.
template <class Cap>
__device__ __forceinline__ double one_scatter(const Tgt<double>& T, const double* gx, const double* gw, int chunk,
                                              int nchunk, Cap cap) {
    const double* x32 = gx + 24; const double* w32 = gw + 24;
    const double* x64 = gx + 56; const double* w64 = gw + 56;
    const int cnt = T.mcnt;
    const double Dn = sqrt(dot(T.eta, T.eta));
    int nd = 32;
    const double* xo = x32;
    const double* wo = w32;
    if (T.ek == RJPATH_EMIT_CONE) {
        const double ca = dot(T.eta, T.ed) / (Dn * sqrt(dot(T.ed, T.ed)));
        const double gap = acos(fmin(1.0, fmax(-1.0, ca))) - acos(fmin(1.0, fmax(-1.0, (double)T.ecos)));
        if (gap < EDGE_GAP) {
            nd = 64;
            xo = x64;
            wo = w64;
        }
    }
    const int waves = blockDim.x / 64, lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
    const double y = x32[lane % 32], wy = w32[lane % 32];
    const double half = lane < 32 ? 1.0 : -1.0;
    double part = 0.0;
    for (int i = chunk * waves + wave; i < nd * nd; i += nchunk * waves) {
        int ix = i / nd, ip = i % nd;
        double x = xo[ix], wx = wo[ix];
        double ps = 2 * PI * (ip + 0.5) / nd;
        V3<double> w0 = emit_dir_icdf(T, x, ps);
        double du = T.ax * w0.x + T.ay * w0.y + T.az * w0.z;
        int l = __builtin_amdgcn_readfirstlane(layer_u(T, T.usrc)); // (the ray's layers are the wave's)
        double a = 0.0, taua = 0.0, ray = 0.0;
        for (int guard = 0; guard <= cnt; ++guard) {
            double bnd = 1e300;
            int lnext = l;
            if (du > 0 && l + 1 < cnt) {
                bnd = (T.edge[l + 1] - T.usrc) / du;
                lnext = l + 1;
            } else if (du < 0 && l > 0) {
                bnd = (T.edge[l] - T.usrc) / du;
                lnext = l - 1;
            }
            const bool tail = !(bnd < 1e299);
            const LayV<double> ly = lay_at(T, l);
            const double cm = ly.c, bm = ly.b;
            double r, wr;
            if (!tail) {
                r = a + (bnd - a) * y;
                wr = wy * (bnd - a) * exp(-taua - cm * (r - a));
            } else if (cm > 0) {
                r = a - log1p(-y) / cm;
                wr = wy * exp(-taua) / cm;
            } else {
                r = a + Dn * y / (1 - y);
                wr = wy * Dn / ((1 - y) * (1 - y)) * exp(-taua);
            }
            const V3<double> f1 = r * w0, df = T.eta - f1;
            if (bm > 0 && wr > 0 && dot(df, df) > (double)T.rad * (double)T.rad * 1.0000002)
                ray += wr * bm * cap(ly, f1, l, w0, T.usrc + r * du, half);
            if (tail) break;
            taua += cm * (bnd - a);
            a = bnd;
            l = __builtin_amdgcn_readfirstlane(lnext);
            if (taua > 60.0) break;
        }
        part += wx * (1.0 / nd) * ray;
    }
    return part;
}

// Sum of a value over the block (fixed order), returned to thread 0.
__device__ __forceinline__ double block_sum(double v, double* red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    return red[0];
}

// Bound by FP64 issue (about 45 instructions per node).  One block per target
// with one ray per thread, the library's log, exp and sincos per node and two
// layer lookups per node took 1.23 s for 200 targets of the 100-layer cone
// batch (200 blocks on 256 CUs, one wave per SIMD, the rim targets four times
// the rest); this form takes 17.3 ms (15 to 19 over drawn targets; two waves per SIMD; forced to three or
// four, with spills, 18.1 and 19.5 ms; the full exponential at every node 20.7).
__global__ void __launch_bounds__(256, 2) anchor_lean_kernel(KArgs a, const double* gx, const double* gw, int nchunk,
                                                          double* out) {
    const int t = blockIdx.x / nchunk, chunk = blockIdx.x % nchunk;
    // (block-uniform: every thread of the block leaves together)
    if (a.medium[t] < 0 || a.medium[t] >= a.n_media || a.n0[t] != 3) return;
    __shared__ double red[256];
    Tgt<double> T;
    load_target<double>(a, t, T, MedTab<double>{a.lay64, a.edge, a.pre});
    const SensorLayers S = sensor_layers(T);
    if (!lean_target(a, t, T, S)) return;
    const double* x8 = gx;
    const double* w8 = gw;
    const double part = one_scatter(T, gx, gw, chunk, nchunk, [&](const LayV<double>& ly, V3<double> f1, int l,
                                                                  V3<double> w0, double uP, double half) {
        const double K = S.kind == 0 ? cap_half<false>(T, ly, f1, uP, l, w0, S, half, x8, w8)
                                     : cap_half<true>(T, ly, f1, uP, l, w0, S, half, x8, w8);
        return K * ((2 * PI / 8) * exp(ly.hgn));
    });
    const double s = block_sum(part, red);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// n0 = 2: a 64 x 64 product rule, one block per target.  Targets without an
// anchor sector: NaN.  (The call for 200 direct sectors: 62 us, 7 of them the
// other kernels' launches; with the rule spread over the chunks of the general
// kernel, whose blocks read their targets each for themselves, 100; with all
// three in one kernel 83.)
__global__ void __launch_bounds__(256) anchor_direct_kernel(KArgs a, const double* gx, const double* gw,
                                                            double* anchor) {
    const int t = blockIdx.x;
    // block-uniform guards: every thread of the block leaves together
    if (a.medium[t] < 0 || a.medium[t] >= a.n_media || (a.n0[t] != 2 && a.n0[t] != 3)) {
        if (threadIdx.x == 0) anchor[t] = __builtin_nan("");
        return;
    }
    if (a.n0[t] != 2) return;
    Tgt<double> T;
    load_target<double>(a, t, T, MedTab<double>{a.lay64, a.edge, a.pre});
    __shared__ double red[256];
    const double* x64 = gx + 56; const double* w64 = gw + 56;
    double part = 0.0;
    // one direction per thread-iteration
    for (int i = threadIdx.x; i < 64 * 64; i += blockDim.x) {
        int iv = i / 64, ip = i % 64;
        V3<double> dv = T.eta;
        double D = sqrt(dot(dv, dv)), Rr = (double)T.rad;
        V3<double> ax = (1.0 / D) * dv, e2, e3;
        frame(ax, e2, e3);
        double k2 = Rr * Rr / (D * D);
        double v = x64[iv], wv = w64[iv];
        double s2 = k2 * (1 - v * v), ct = sqrt(1 - s2), st = sqrt(s2);
        double len = D * ct - Rr * v, jac = k2 * v / ct;
        double ps = 2 * PI * (ip + 0.5) / 64, sp, cp;
        sincos(ps, &sp, &cp);
        V3<double> u = ct * ax + st * (cp * e2 + sp * e3);
        V3<double> hit = len * u;
        V3<double> nu = (1.0 / Rr) * (hit - T.eta);
        double le = emit_term(T, u);
        if (le == -__builtin_inf()) continue;
        V3<double> o = {0, 0, 0};
        part += wv * (2 * PI / 64) * jac * exp(le - depth_c(T, o, hit) + log_rho(T, nu));
    }
    const double s = block_sum(part, red);
    if (threadIdx.x == 0) anchor[t] = s;
}

__global__ void __launch_bounds__(256) anchor_kernel(KArgs a, const double* gx, const double* gw, int nchunk,
                                                     double* out) {
    const int t = blockIdx.x / nchunk, chunk = blockIdx.x % nchunk;
    if (a.medium[t] < 0 || a.medium[t] >= a.n_media || a.n0[t] != 3) return;
    Tgt<double> T;
    load_target<double>(a, t, T, MedTab<double>{a.lay64, a.edge, a.pre});
    if (lean_target(a, t, T, sensor_layers(T))) return;
    __shared__ double red[256];
    const double* x8 = gx;
    const double* w8 = gw;
    const double part = one_scatter(T, gx, gw, chunk, nchunk, [&](const LayV<double>& ly, V3<double> f1, int l,
                                                                  V3<double> w0, double uP, double half) {
        return cap_quad(T, f1, x8, w8, 8, half > 0 ? 0 : 4, 4, 8, [&](V3<double> u) { return turn_term(ly, w0, u); });
    });
    const double s = block_sum(part, red);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// anchor[t] = the sum of its chunks, in a fixed order (targets of one scattering vertex)
__global__ void __launch_bounds__(64) anchor_sum_kernel(KArgs a, int nchunk, const double* part, double* anchor) {
    const int t = blockIdx.x;
    if (a.medium[t] < 0 || a.medium[t] >= a.n_media || a.n0[t] != 3) return;
    double s = 0.0;
    for (int i = threadIdx.x; i < nchunk; i += 64) s += part[(size_t)t * nchunk + i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (threadIdx.x == 0) anchor[t] = s;
}

} // namespace

// Blocks per target: enough that a few targets still fill the chip (about 16
// blocks per CU over all targets) and that the rim targets' fourfold
// work is spread, at most one direction per wave.  From 2^14 targets on their
// number alone fills it many times over, and 2^18 blocks are kept to as long
// as every target has one: a launch must stay below 2^32 threads (2^24 blocks,
// which 16 for each of 2^20 targets would reach), and the chunk sums within 2 MiB
// or one double per target.  (100-layer cone targets, 16 blocks each and by this
// rule: 20,000 1.46 and 1.29 s, 40,000 2.90 and 2.70 s.)
int anchor_chunks(int T) { return std::max(1, std::max(std::min(16, (1 << 18) / T), std::min(256, 4096 / T))); }

hipError_t launch_anchor(const KArgs& a, const double* gl_x, const double* gl_w, double* anchor, double* part,
                         int nchunk, hipStream_t s) {
    if (nchunk < 2) {
        nchunk = 1;
        part = anchor;
    }
    hipLaunchKernelGGL(anchor_direct_kernel, dim3(a.T), dim3(256), 0, s, a, gl_x, gl_w, anchor);
    hipLaunchKernelGGL(anchor_lean_kernel, dim3(a.T * nchunk), dim3(256), 0, s, a, gl_x, gl_w, nchunk, part);
    hipLaunchKernelGGL(anchor_kernel, dim3(a.T * nchunk), dim3(256), 0, s, a, gl_x, gl_w, nchunk, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nchunk == 1) return e;
    hipLaunchKernelGGL(anchor_sum_kernel, dim3(a.T), dim3(64), 0, s, a, nchunk, part, anchor);
    return hipGetLastError();
}

} // namespace rj
