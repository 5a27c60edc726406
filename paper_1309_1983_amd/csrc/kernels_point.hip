// Step kernels with one point per work-item for gfx950: the pull step of
// Algorithm 3 (Mawson & Revell, Section 4.2) between two arrays, and the
// single-array (AA) pattern.
#include "step_common.hpp"

namespace lbmk {

// ---------------------------------------------------------------------------
// AB pull step, one point per work-item: gather from x - e_i in `src`,
// bounce back at solid neighbours, collide, store into `dst`. Used where it is
// faster than several points per work-item (bound by its 38 accesses per point:
// 28 waves per compute unit keep more of them in flight than the vector step's
// 8 to 12), and where rows do not divide into vectors. MACROS: also store the
// in-step rho and u (the four extra stores per point of Section 4.1).
// ONSITE: rebuild the unknown populations of on-site velocity nodes.
// Solid points of a wave that holds fluid points are stored as the rest state,
// by the same store instructions: nothing reads them, but lines with holes
// are written back in part, which costs more than the whole line. MI355X, us
// per step: 256^3 FP16 cavity 345 -> 228, FP32 sphere duct 725 -> 468.
// STREAM: non-temporal stores.
// ---------------------------------------------------------------------------
template <class St, int FM, bool COLLIDE, bool MACROS, bool ONSITE, bool STREAM>
__global__ __launch_bounds__(1024) void k_step_ab(const typename St::raw_t* __restrict__ src,
                                                  typename St::raw_t* __restrict__ dst,
                                                  const uint8_t* __restrict__ flags,
                                                  const uint32_t* __restrict__ smask,
                                                  const uint32_t* __restrict__ mmask,
                                                  const float* __restrict__ ff, StepArgs a,
                                                  float* __restrict__ rho_out, float* __restrict__ u_out)
{
    using T = typename St::raw_t;
    const Dims& d = a.d;
    POINT_PROLOGUE(d)
    const uint8_t fl = flags[c];
    const bool fluid = (fl & TYPE_MASK) == 0;
    Macro m = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    T v[Q];
    if (fluid) {
        uint32_t on[Q];
        pull_offsets(d, x, y, on);
#pragma unroll
        for (int i = 0; i < Q; ++i) v[i] = ld(plane(src, d, i, src_slab(i, z, zm, zp)), on[i]);

        uint32_t mwmask = 0, solid = 0;
        if (fl & NEAR_WALL) {
            solid = smask[c];
            if (fl & NEAR_MOVING) mwmask = mmask[c];
#pragma unroll
            for (int i = 1; i < Q; ++i)
                if ((solid >> i) & 1u) v[i] = ld(plane(src, d, OPP[i], z), o);
        }
        if (COLLIDE) {
            float F[3], h[Q];
            load_force<FM>(a, ff, c, F[0], F[1], F[2]);
            m = decode_collide<St, FM, ONSITE>(v, mwmask, (fl & ONSITE_NODE) ? solid : 0u, (fl & ONSITE_MOVING) != 0,
                                               a, F, h);
#pragma unroll
            for (int i = 0; i < Q; ++i) v[i] = St::enc(h[i], i);
        }
    } else {
#pragma unroll
        for (int i = 0; i < Q; ++i) v[i] = St::enc(0.0f, i);
    }
    if (__builtin_amdgcn_ballot_w64(fluid) != 0ull) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            if (STREAM) st_nt(plane(dst, d, i, z), o, v[i]);
            else st(plane(dst, d, i, z), o, v[i]);
        }
    }
    if (MACROS) {
        rho_out[c] = m.rho;
        u_out[c] = m.ux; u_out[(size_t)d.N + c] = m.uy; u_out[2 * (size_t)d.N + c] = m.uz;
    }
}

// ---------------------------------------------------------------------------
// AA pattern, one array, in place.
// Parity 0 (array holds s_i(x) at slot [i][x]): read p_i from [i][x - e_i],
// or from [opp(i)][x] when x - e_i is solid; write s'_j into the slot that
// p_opp(j) was read from. Afterwards s'_j(x) sits at [opp(j)][x + e_j]
// (or at [j][x] when x + e_j is solid).
// Parity 1: p_i = [opp(i)][x] for every i (local); write s'_i to [i][x],
// restoring the natural layout. Each work-item reads and writes the same 19
// slots, and no two work-items share a slot, so the update is race-free. The
// local step stores the rest state at solid points beside fluid ones, as the
// two-array step does (sphere duct 128x128x256 in place, FP16 61.2 -> 58.1 us
// per step); the scatter's holes lie in other work-items' lines, and filling
// them by stores of their own cost 8%.
// ---------------------------------------------------------------------------
template <class St, int FM, bool COLLIDE, bool ONSITE>
__global__ __launch_bounds__(1024) void k_step_aa0(typename St::raw_t* f,
                                                   const uint8_t* __restrict__ flags,
                                                   const uint32_t* __restrict__ smask,
                                                   const uint32_t* __restrict__ mmask,
                                                   const float* __restrict__ ff, StepArgs a)
{
    using T = typename St::raw_t;
    const Dims& d = a.d;
    POINT_PROLOGUE(d)
    const uint8_t fl = flags[c];
    if (fl & TYPE_MASK) return;

    uint32_t on[Q];
    pull_offsets(d, x, y, on);
    T raw[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) raw[i] = ld(plane(f, d, i, src_slab(i, z, zm, zp)), on[i]);

    uint32_t solid = 0, mwmask = 0;
    if (fl & NEAR_WALL) {
        solid = smask[c];
        if (fl & NEAR_MOVING) mwmask = mmask[c];
#pragma unroll
        for (int i = 1; i < Q; ++i)
            if ((solid >> i) & 1u) raw[i] = ld(plane(f, d, OPP[i], z), o);
    }

    float F[3], h[Q];
    load_force<FM>(a, ff, c, F[0], F[1], F[2]);
    if (COLLIDE)
        decode_collide<St, FM, ONSITE>(raw, mwmask, (fl & ONSITE_NODE) ? solid : 0u, (fl & ONSITE_MOVING) != 0,
                                       a, F, h);
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        const int k = OPP[j];
        const T v = COLLIDE ? St::enc(h[j], j) : raw[j];
        if ((solid >> k) & 1u) st(plane(f, d, j, z), o, v);
        else st(plane(f, d, k, src_slab(k, z, zm, zp)), on[k], v);
    }
}

template <class St, int FM, bool COLLIDE, bool ONSITE>
__global__ __launch_bounds__(1024) void k_step_aa1(typename St::raw_t* f,
                                                   const uint8_t* __restrict__ flags,
                                                   const uint32_t* __restrict__ smask,
                                                   const uint32_t* __restrict__ mmask,
                                                   const float* __restrict__ ff, StepArgs a)
{
    using T = typename St::raw_t;
    const Dims& d = a.d;
    POINT_PROLOGUE(d)
    (void)zm; (void)zp;   // every access of the local step is in the point's own slab
    const uint8_t fl = flags[c];
    const bool fluid = (fl & TYPE_MASK) == 0;
    T v[Q];
    if (fluid) {
#pragma unroll
        for (int i = 0; i < Q; ++i) v[i] = ld(plane(f, d, OPP[i], z), o);
        if (COLLIDE) {
            uint32_t mwmask = 0, solid = 0;
            if (fl & NEAR_MOVING) mwmask = mmask[c];
            if (ONSITE && (fl & ONSITE_NODE)) solid = smask[c];
            float F[3], h[Q];
            load_force<FM>(a, ff, c, F[0], F[1], F[2]);
            decode_collide<St, FM, ONSITE>(v, mwmask, (fl & ONSITE_NODE) ? solid : 0u, (fl & ONSITE_MOVING) != 0, a,
                                           F, h);
#pragma unroll
            for (int i = 0; i < Q; ++i) v[i] = St::enc(h[i], i);
        }
    } else {   // its own slots, which no other work-item touches
#pragma unroll
        for (int i = 0; i < Q; ++i) v[i] = St::enc(0.0f, i);
    }
    if (__builtin_amdgcn_ballot_w64(fluid) == 0ull) return;
#pragma unroll
    for (int i = 0; i < Q; ++i) st(plane(f, d, i, z), o, v[i]);
}

template <class St, int FM, bool ONSITE>
static hipError_t step_fm(int pattern, int parity, bool collide, void* a, void* b,
                          const uint8_t* flags, const uint32_t* sm, const uint32_t* mm, const float* ff,
                          const StepArgs& args, const Launch& L, float* rho, float* u)
{
    using T = typename St::raw_t;
    T* A = static_cast<T*>(a);
    T* B = static_cast<T*>(b);
    if (pattern == 0) {
        if (collide && rho && args.stream)
            STEP_LAUNCH((k_step_ab<St, FM, true, true, ONSITE, true>), L.grid, L.block, L.shmem, L.stream, A, B, flags, sm, mm, ff, args, rho, u);
        else if (collide && rho)
            STEP_LAUNCH((k_step_ab<St, FM, true, true, ONSITE, false>), L.grid, L.block, L.shmem, L.stream, A, B, flags, sm, mm, ff, args, rho, u);
        else if (collide && args.stream)
            STEP_LAUNCH((k_step_ab<St, FM, true, false, ONSITE, true>), L.grid, L.block, L.shmem, L.stream, A, B, flags, sm, mm, ff, args, rho, u);
        else if (collide)
            STEP_LAUNCH((k_step_ab<St, FM, true, false, ONSITE, false>), L.grid, L.block, L.shmem, L.stream, A, B, flags, sm, mm, ff, args, rho, u);
        else
            STEP_LAUNCH((k_step_ab<St, FORCE_NONE, false, false, false, false>), L.grid, L.block, L.shmem, L.stream, A, B, flags, sm, mm, ff, args, rho, u);
    } else if (parity == 0) {
        if (collide)
            STEP_LAUNCH((k_step_aa0<St, FM, true, ONSITE>), L.grid, L.block, L.shmem, L.stream, A, flags, sm, mm, ff, args);
        else
            STEP_LAUNCH((k_step_aa0<St, FORCE_NONE, false, false>), L.grid, L.block, L.shmem, L.stream, A, flags, sm, mm, ff, args);
    } else {
        if (collide)
            STEP_LAUNCH((k_step_aa1<St, FM, true, ONSITE>), L.grid, L.block, L.shmem, L.stream, A, flags, sm, mm, ff, args);
        else
            STEP_LAUNCH((k_step_aa1<St, FORCE_NONE, false, false>), L.grid, L.block, L.shmem, L.stream, A, flags, sm, mm, ff, args);
    }
    return hipGetLastError();
}

template <class St, bool ONSITE>
static hipError_t step_st(int pattern, int parity, bool collide, int fm, void* a, void* b,
                          const uint8_t* flags, const uint32_t* sm, const uint32_t* mm, const float* ff,
                          const StepArgs& args, const Launch& L, float* rho, float* u)
{
    switch (fm) {
    case FORCE_UNIFORM: return step_fm<St, FORCE_UNIFORM, ONSITE>(pattern, parity, collide, a, b, flags, sm, mm, ff, args, L, rho, u);
    case FORCE_FIELD: return step_fm<St, FORCE_FIELD, ONSITE>(pattern, parity, collide, a, b, flags, sm, mm, ff, args, L, rho, u);
    default: return step_fm<St, FORCE_NONE, ONSITE>(pattern, parity, collide, a, b, flags, sm, mm, ff, args, L, rho, u);
    }
}

template <bool ONSITE>
static hipError_t step_os(int storage, int pattern, int parity, bool collide, int force_mode, void* a,
                          void* b, const uint8_t* flags, const uint32_t* sm, const uint32_t* mm,
                          const float* ffield, const StepArgs& args, const Launch& L, float* rho, float* u)
{
    switch (storage) {
    case 1: return step_st<StF16, ONSITE>(pattern, parity, collide, force_mode, a, b, flags, sm, mm, ffield, args, L, rho, u);
    case 2: return step_st<StBF16, ONSITE>(pattern, parity, collide, force_mode, a, b, flags, sm, mm, ffield, args, L, rho, u);
    default: return step_st<StF32, ONSITE>(pattern, parity, collide, force_mode, a, b, flags, sm, mm, ffield, args, L, rho, u);
    }
}

hipError_t launch_step(int storage, int pattern, int parity, bool collide, int force_mode, void* a,
                       void* b, const uint8_t* flags, const uint32_t* smask, const uint32_t* mmask,
                       const float* ffield, const StepArgs& args, const Launch& L, float* rho, float* u,
                       bool onsite)
{
    const StepArgs g = on_grid(args, L);
    return (onsite && collide)
               ? step_os<true>(storage, pattern, parity, collide, force_mode, a, b, flags, smask, mmask, ffield, g, L, rho, u)
               : step_os<false>(storage, pattern, parity, collide, force_mode, a, b, flags, smask, mmask, ffield, g, L, rho, u);
}

}  // namespace lbmk
