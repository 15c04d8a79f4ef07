// rj_wave.h -- wavefront (64-lane) and block reductions, and the sharing of
// the items of a wave's chains over its lanes.
#pragma once

#include <hip/hip_runtime.h>

namespace rj {

__device__ __forceinline__ int wave_min_i32(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ __forceinline__ int wave_max_i32(int v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
    return v;
}

// Block-wide min / max (every thread of the block must call; s holds one int
// per wave and is not reused by the caller before the next barrier).
__device__ __forceinline__ int block_min_i32(int v, int* s) {
    v = wave_min_i32(v);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    int r = s[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) r = min(r, s[i]);
    return r;
}

__device__ __forceinline__ int block_max_i32(int v, int* s) {
    v = wave_max_i32(v);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    int r = s[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) r = max(r, s[i]);
    return r;
}

// Inclusive prefix sum over the 64 lanes by data-parallel moves (no LDS).
__device__ __forceinline__ int wave_prefix(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true); // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true); // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true); // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true); // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false); // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false); // row_bcast:31 into rows 2 and 3
    return v;
}

// The lanes that share the items of a run of chains (in one register): the
// chains' own, `own` from `lo` on, then `helpers` lanes without a chain from
// `hlo` on, behind all chains' lanes.
struct LaneRun {
    int v;
    __device__ __forceinline__ static LaneRun of(int lo, int own, int hlo, int helpers) {
        return LaneRun{lo | own << 6 | hlo << 13 | helpers << 19};
    }
    __device__ __forceinline__ int lo() const { return v & 63; }
    __device__ __forceinline__ int own() const { return (v >> 6) & 127; }
    __device__ __forceinline__ int hlo() const { return (v >> 13) & 63; }
    __device__ __forceinline__ int count() const { return own() + (v >> 19); }
    __device__ __forceinline__ uint64_t mask() const {
        return (~0ull >> (64 - own())) << lo() | ((1ull << (v >> 19)) - 1) << hlo();
    }
    __device__ __forceinline__ int place(int lane) const { return lane < lo() + own() ? lane - lo() : own() + lane - hlo(); }
    __device__ __forceinline__ int at(int place) const { return place < own() ? lo() + place : hlo() + place - own(); }
};

__device__ __forceinline__ LaneRun whole_wave() { return LaneRun{64 << 6}; }

// Neighbouring chains of one target t, lanes 0 .. cpw - 1, share their items;
// the lanes from cpw on (helpers, fewer than 64) go to the targets' runs such
// that every run has lanes in proportion to its items, as far as that goes.
// A helper's t becomes its run's.  (Where all of them followed the last chain,
// the slowest wave of the ragged joint Langevin batch, five chains of one
// target and 27 of the next, took 57 us per joint move and the median 15 us.)
__device__ __forceinline__ LaneRun share_lanes(int lane, int cpw, int items, int& t) {
    const uint64_t below = ~0ull >> (64 - cpw);
    const int left = __shfl_up(t, 1, 64);
    const uint64_t starts = __ballot(lane < cpw && (lane == 0 || left != t)); // lanes that begin a run
    const uint64_t upto = starts & (~0ull >> (63 - lane)), after = starts & ~(~0ull >> (63 - lane));
    int lo = 63 - __clzll((long long)upto); // (a helper's: the last run's)
    int own = (after ? __ffsll((unsigned long long)after) - 1 : cpw) - lo;
    int hlo = cpw & 63, helpers = 0;
    if (cpw < 64) {
        const int end = wave_prefix(lane < cpw ? items : 0);
        const int all = __shfl(end, cpw - 1, 64), last = __shfl(end, lo + own - 1, 64);
        const int first = __shfl(end, lo > 0 ? lo - 1 : 0, 64), mine = last - (lo > 0 ? first : 0);
        // lanes that the run lacks, scaled by all items; in its first lane
        const bool leads = lane < cpw && lane == lo;
        const float lacks = leads ? fmaxf((float)mine * 64.0f / (float)all - (float)own, 0.0f) : 0.0f;
        float total = 0.0f;
        for (uint64_t m = starts; m; m &= m - 1) total += __shfl(lacks, __ffsll((unsigned long long)m) - 1, 64);
        const float x = ((float)(lane - cpw) + 0.5f) * total / (float)(64 - cpw); // a helper's place among them
        float seen = 0.0f;
        int run = 0; // its run's first lane
        for (uint64_t m = starts; m; m &= m - 1) {
            const int q = __ffsll((unsigned long long)m) - 1;
            if (x >= seen) run = q;
            seen += __shfl(lacks, q, 64);
        }
        if (lane < cpw) run = lo;
        lo = run;
        own = __shfl(own, run, 64);
        t = __shfl(t, run, 64);
        // helpers of a run are neighbours: x grows with the lane
        for (uint64_t m = starts; m; m &= m - 1) {
            const int q = __ffsll((unsigned long long)m) - 1;
            const uint64_t h = __ballot(run == q) & ~below;
            if (run == q && h) {
                hlo = __ffsll((unsigned long long)h) - 1;
                helpers = __popcll(h);
            }
        }
    }
    return LaneRun::of(lo, own, hlo, helpers);
}

// Items of the wave's chains in chain order, shared by the lanes of a run, one
// per lane and window: `first` is the chain's first item and the count given to
// init() how many it has (0: none; a lane without a chain too), in its own lane.  next() gives each
// lane its item's chain and the item's place in it; the starts in the window
// are one bit mask, whose bits below a lane count the chains.
struct WaveItems {
    int lane, first, base, total, seen, nth;
    LaneRun run;
    uint64_t mask; // the window's starts
    bool has;
    __device__ __forceinline__ void init(int lane_, int cnt, LaneRun r) {
        lane = lane_;
        run = r;
        has = cnt > 0;
        const int end = wave_prefix(cnt);
        first = end - cnt;
        const int from = __shfl(first, run.lo(), 64); // the run's first item
        total = __shfl(end, run.lo() + run.own() - 1, 64) - from;
        first -= from;
        const uint64_t m = __ballot(has);
        const int n = __popcll(m);
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        nth = __builtin_amdgcn_ds_permute(4 * (has ? rank : n + lane - rank), lane); // lane r: the r-th chain's lane
        base = 0;
        seen = __shfl(rank, run.lo(), 64);
    }
    __device__ __forceinline__ void init(int lane_, int cnt) { init(lane_, cnt, whole_wave()); }
    __device__ __forceinline__ bool more() const { return __any(base < total); }
    // Starts among the last `m` lanes of the window just given (whole wave):
    // next() after base -= m gives those lanes' items again.
    __device__ __forceinline__ int starts_at_end(int m) const { return __popcll(mask >> (64 - m)); }
    // the window's items: true if this lane has one; q: its chain's lane, k: its place
    __device__ __forceinline__ bool next(int& q, int& k) {
        const int s = first - base;
        const bool in = has && s >= 0 && s < run.count();
        const uint64_t bit = in ? 1ull << run.at(s) : 0ull;
        // the starts are distinct, so their sum is their union
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane(wave_prefix((int)(uint32_t)bit), 63);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane(wave_prefix((int)(uint32_t)(bit >> 32)), 63);
        mask = ((uint64_t)hi << 32 | lo) & run.mask();
        const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
        const int upto = (int)below + (int)((mask >> lane) & 1u);
        q = __shfl(nth, (seen + upto - 1) & 63, 64);
        const int i = base + run.place(lane);
        k = i - __shfl(first, q, 64);
        seen += __popcll(mask);
        base += run.count();
        return i < total;
    }
};

} // namespace rj
