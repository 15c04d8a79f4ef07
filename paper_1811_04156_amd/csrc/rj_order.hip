// rj_order.hip -- the order in which a launch's waves take their chains.
#include <hip/hip_runtime.h>

#include "rj_kernels.h"
#include "rj_wave.h"

namespace rj {
namespace {

// A step's time grows with the vertices of the wave's chains, and the chains of
// a far target have several times as many as those of a near one.  Blocks
// beyond the resident ones start as others end, when the slowest of their
// waves does, so a launch whose long waves come last runs them on a nearly
// empty chip.  With the most vertices first the short waves fill the gaps, and
// the waves of a block end together: 200 steps of 262,144 chains of the ragged
// layered batch take 5.08 ms unordered and 4.26 ordered with tree moves, 1.87
// and 1.74 with single-vertex Langevin moves; of 50,001 with joint Langevin
// moves 4.03 and 3.12; of 1,048,576 plain ones 5.41 and 5.16.  (Ordered by
// blocks, 4.78, 1.80, 3.30 and 5.23.)
// The order lies in the status words of the first chains until the waves have
// read it (take_order): bits 8 and up of word i are the place of wave i's chains.
// Bits 0 to 7, the status itself, are nobody's but the chain's.
// One block sorts, with 16 weights per thread in registers: launches of more than
// ORDER_WAVES waves keep the order of the chains.  (The gain falls with the rounds
// that a launch takes: above, 7 to 16% at two rounds and 5% at eight, which
// ORDER_WAVES waves are.)

// vertices of each wave's chains (at most 64 x 4096) into word b
__global__ void __launch_bounds__(64) weight_kernel(const int32_t* n, int C, int cap, int per, int32_t* status) {
    const int b = blockIdx.x, lane = threadIdx.x, c = b * per + lane;
    const int all = wave_prefix(lane < per && c < C ? min(max(n[c], 0), cap) : 0);
    if (lane == 63) status[b] = all << 8 | (status[b] & 0xff);
}

// most vertices first: a counting sort of the nb <= ORDER_WAVES weights over
// ORDER_BINS bins (waves of one bin in any order)
__global__ void __launch_bounds__(ORDER_BINS) order_kernel(int nb, int32_t* status) {
    constexpr int K = ORDER_WAVES / ORDER_BINS;
    __shared__ int bins[ORDER_BINS], waves[ORDER_BINS / 64], most;
    __shared__ uint8_t low[ORDER_WAVES]; // the words' own bits
    const int tid = threadIdx.x, lane = tid & 63;
    int w[K], big = 0;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const int b = i * ORDER_BINS + tid;
        const uint32_t word = b < nb ? (uint32_t)status[b] : 0u;
        low[b] = (uint8_t)word;
        w[i] = (int)(word >> 8);
        big = max(big, w[i]);
    }
    bins[tid] = 0;
    if (tid == 0) most = 1;
    __syncthreads();
    atomicMax(&most, big);
    __syncthreads();
    const float scale = (float)(ORDER_BINS - 1) / (float)most;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        w[i] = ORDER_BINS - 1 - min((int)((float)w[i] * scale), ORDER_BINS - 1);
        if (i * ORDER_BINS + tid < nb) atomicAdd(&bins[w[i]], 1);
    }
    __syncthreads();
    const int mine = bins[tid], upto = wave_prefix(mine);
    if (lane == 63) waves[tid / 64] = upto;
    __syncthreads();
    int first = upto - mine;
    for (int v = 0; v < tid / 64; ++v) first += waves[v];
    bins[tid] = first;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const int b = i * ORDER_BINS + tid;
        if (b < nb) {
            const int place = atomicAdd(&bins[w[i]], 1);
            status[place] = b << 8 | low[place];
        }
    }
}

__global__ void __launch_bounds__(256) clear_kernel(int nb, int32_t* status) {
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b < nb) status[b] &= 0xff;
}

} // namespace

// Takes the order back where no launch follows to read it.
void clear_order(const KArgs& a, int per, hipStream_t s) {
    const int nb = (a.C + per - 1) / per;
    hipLaunchKernelGGL(clear_kernel, dim3((nb + 255) / 256), dim3(256), 0, s, nb, a.status);
}

hipError_t launch_order(const KArgs& a, int per, hipStream_t s) {
    const int nb = (a.C + per - 1) / per;
    hipLaunchKernelGGL(weight_kernel, dim3(nb), dim3(64), 0, s, a.n, a.C, a.cap, per, a.status);
    hipLaunchKernelGGL(order_kernel, dim3(1), dim3(ORDER_BINS), 0, s, nb, a.status);
    return hipGetLastError();
}

} // namespace rj
