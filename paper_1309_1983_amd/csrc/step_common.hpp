// What the step kernels with one and with several points per work-item share
// (internal to the library).
#pragma once

#include "kernels.hpp"

namespace lbmk {

using namespace d3q19;

template <int FM>
__device__ __forceinline__ void load_force(const StepArgs& a, const float* __restrict__ ff, uint32_t c,
                                           float& Fx, float& Fy, float& Fz)
{
    if (FM == FORCE_UNIFORM) {
        Fx = a.Fx; Fy = a.Fy; Fz = a.Fz;
    } else if (FM == FORCE_FIELD) {
        Fx = ff[c];
        Fy = ff[(size_t)a.d.N + c];
        Fz = ff[2 * (size_t)a.d.N + c];
    } else {
        Fx = Fy = Fz = 0.0f;
    }
}

// Decode, add moving-wall terms, rebuild the unknowns of an on-site node
// (onsiteU != 0: its solid-source directions), collide. h ends as
// post-collision offsets.
template <class St, int FM, bool ONSITE>
__device__ __forceinline__ Macro decode_collide(const typename St::raw_t raw[Q], uint32_t mwmask,
                                                uint32_t onsiteU, bool onsite_moving,
                                                const StepArgs& a, const float F[3], float h[Q])
{
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        h[i] = St::off(raw[i], i);
        if (i > 0 && ((mwmask >> i) & 1u)) h[i] = h[i] + a.mw[i];
    }
    if (ONSITE && onsiteU) {
        const float ux = onsite_moving ? a.uw[0] : 0.0f;
        const float uy = onsite_moving ? a.uw[1] : 0.0f;
        const float uz = onsite_moving ? a.uw[2] : 0.0f;
        onsite_rebuild<FM != FORCE_NONE>(h, onsiteU, ux, uy, uz, F[0], F[1], F[2]);
    }
    return bgk_collide<FM != FORCE_NONE>(h, a.omega, a.cF, F[0], F[1], F[2]);
}

#define POINT_PROLOGUE(d)                                                                      \
    int x, y;                                                                                  \
    uint32_t z;                                                                                \
    if (!point_of((d), x, y, z)) return;                                                       \
    const uint32_t o = (uint32_t)y * (uint32_t)(d).nx + (uint32_t)x;                           \
    const uint32_t c = z * (d).nxy + o;                                                        \
    const uint32_t zm = wrap_m(z, (uint32_t)(d).nz), zp = wrap_p(z, (uint32_t)(d).nz);

// While t_resolve is set (resolve_step_kernel), the step dispatch records the
// kernel it would launch instead of launching it.
extern thread_local const void** t_resolve;
#define STEP_LAUNCH(K, GRID, BLOCK, SHMEM, STREAM, ...)                         \
    do {                                                                      \
        if (t_resolve) *t_resolve = reinterpret_cast<const void*>(&K);        \
        else hipLaunchKernelGGL(K, GRID, BLOCK, SHMEM, STREAM, __VA_ARGS__);  \
    } while (0)

}  // namespace lbmk
