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

// Items of the wave's chains in chain order, 64 at a time: `first` is the
// chain's first item and `cnt` its count (0: none) in its own lane.  next()
// gives each lane its item's chain and the item's place in it; the starts in
// the window are one bit mask, whose bits below a lane count the chains.
struct WaveItems {
    int lane, first, base, total, seen, nth;
    uint64_t mask; // the window's starts
    bool has;
    __device__ __forceinline__ void init(int lane_, int cnt) {
        lane = lane_;
        has = cnt > 0;
        const int end = wave_prefix(cnt);
        total = __builtin_amdgcn_readlane(end, 63);
        first = end - cnt;
        const uint64_t m = __ballot(has);
        const int n = __popcll(m);
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        nth = __builtin_amdgcn_ds_permute(4 * (has ? rank : n + lane - rank), lane); // lane r: the r-th chain's lane
        base = 0;
        seen = 0;
    }
    __device__ __forceinline__ bool more() const { return base < total; }
    // Starts among the last `m` lanes of the window just given: next() after
    // base -= m gives those lanes' items again.
    __device__ __forceinline__ int starts_at_end(int m) const { return __popcll(mask >> (64 - m)); }
    // the window's items: true if this lane has one; q: its chain's lane, k: its place
    __device__ __forceinline__ bool next(int& q, int& k) {
        const int s = first - base;
        const bool in = has && s >= 0 && s < 64;
        const uint64_t bit = in ? 1ull << s : 0ull;
        // the starts are distinct, so their sum is their union
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane(wave_prefix((int)(uint32_t)bit), 63);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane(wave_prefix((int)(uint32_t)(bit >> 32)), 63);
        const int upto = (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u)) +
                         (int)(((lane < 32 ? lo : hi) >> (lane & 31)) & 1u);
        q = __shfl(nth, (seen + upto - 1) & (63), 64);
        k = base + lane - __shfl(first, q, 64);
        const bool mine = base + lane < total;
        mask = (uint64_t)hi << 32 | lo;
        seen += __popcll(mask);
        base += 64;
        return mine;
    }
};

} // namespace rj
