// rj_run.h -- launchers of the step kernel, one explicit instantiation per
// precision and interior move (rj_run_{f32,f64}{,_mala,_lmala}.hip) so that
// the variants compile in parallel.
#pragma once

#include "rj_step.h"

namespace rj {

template <class R, int MK, int SAMP, bool SL, bool EVEN>
static hipError_t launch_run_t(const KArgs& a, int block, hipStream_t s) {
    constexpr bool SHARED = SAMP == SAMP_TREE || SAMP == SAMP_JOINT;
    const int chains = SHARED ? block / WAVE * a.cpw : block;
    int grid = (a.C + chains - 1) / chains;
    // media tables, then one tile of V + SLOT_PAD slots per wave, then the whole-path samplers' proposals
    size_t lds = (MK == MK_LAY_LDS ? a.tab_bytes : 0) + (size_t)(a.V + SLOT_PAD) * block * sizeof(Vtx<R>);
    if (SHARED && a.cpw == WAVE) lds += (size_t)a.Vy * block * sizeof(Vtx<R>);
    if constexpr (EVEN)
        hipLaunchKernelGGL((run_even_layers_kernel<R, MK, SAMP, SL>), dim3(grid), dim3(block), lds, s, a);
    else
        hipLaunchKernelGGL((run_kernel<R, MK, SAMP, SL>), dim3(grid), dim3(block), lds, s, a);
    return hipGetLastError();
}

template <class R, int MK, int SAMP, bool EVEN> static hipError_t launch_run_m(const KArgs& a, int block, hipStream_t s) {
    return a.has_sl ? launch_run_t<R, MK, SAMP, true, EVEN>(a, block, s)
                    : launch_run_t<R, MK, SAMP, false, EVEN>(a, block, s);
}

// FP64 always reads the layer tables from HBM (its LDS goes to vertex slots)
template <class R, int SAMP> hipError_t launch_run_v(const KArgs& a, int block, hipStream_t s) {
    if (!a.layered) return launch_run_m<R, MK_HOM, SAMP, false>(a, block, s);
    if constexpr (sizeof(R) == 4) {
        if (a.tab_bytes)
            return a.even ? launch_run_m<R, MK_LAY_LDS, SAMP, true>(a, block, s)
                          : launch_run_m<R, MK_LAY_LDS, SAMP, false>(a, block, s);
        return launch_run_m<R, MK_LAY, SAMP, false>(a, block, s);
    } else {
        return a.even ? launch_run_m<R, MK_LAY, SAMP, true>(a, block, s)
                      : launch_run_m<R, MK_LAY, SAMP, false>(a, block, s);
    }
}

template <class R, int SAMP> hipError_t set_lds_limit_v() {
    constexpr int MK_EVEN = sizeof(R) == 4 ? MK_LAY_LDS : MK_LAY;
    const void* fns[] = {
        (const void*)run_kernel<R, MK_HOM, SAMP, false>,
        (const void*)run_kernel<R, MK_HOM, SAMP, true>,
        (const void*)run_kernel<R, MK_LAY, SAMP, false>,
        (const void*)run_kernel<R, MK_LAY, SAMP, true>,
        (const void*)run_even_layers_kernel<R, MK_EVEN, SAMP, false>,
        (const void*)run_even_layers_kernel<R, MK_EVEN, SAMP, true>,
        (const void*)run_kernel<R, MK_LAY_LDS, SAMP, false>,
        (const void*)run_kernel<R, MK_LAY_LDS, SAMP, true>};
    const int nf = sizeof(R) == 4 ? 8 : 6;
    for (int i = 0; i < nf; ++i) {
        hipError_t e = hipFuncSetAttribute(fns[i], hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

} // namespace rj
