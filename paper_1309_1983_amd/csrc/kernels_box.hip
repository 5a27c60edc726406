// Two pull steps per launch on small lattices (two-array pattern) for gfx950.
//
// A lattice of a few 10^4 points lives in the caches and leaves most of the
// chip idle: its steps are bound by their launches and by one round of load
// latency each, not by bandwidth. Here a work-group computes s^{t+1} on a box
// of points and a halo one point wide into LDS, and s^{t+2} of the box from
// there: two steps take one launch and one round of loads, for 3.4 times the
// first step's arithmetic on units that were idle. Boxes of 16 x 4 x 2 points
// with one work-item per point of box and halo (432 of 448), so that 32^3
// gives each of the 256 compute units one work-group. MI355X, us per step, one
// step per launch / this: 32^3 periodic FP32 3.76 / 3.24, cavity 4.39 / 3.60, 24^3
// FP16 3.89 / 3.18, 28^3 duct with a force field 4.53 / 4.22. With more boxes than
// compute units it loses: 40^3 cavity 5.01 / 5.57, 56^3 6.3 / 10.0.
//
// Per point both steps do the arithmetic of the one-step kernels on values
// rounded to the storage format in between, so the result is the same bit for
// bit.
#include "kernels.hpp"

using namespace d3q19;

namespace lbmk {

constexpr int BX = BOX_X, BY = BOX_Y, BZ = BOX_Z;
constexpr int HX = BX + 2, HY = BY + 2, HZ = BZ + 2;
constexpr int POINTS = HX * HY * HZ, OUT = BX * BY * BZ;
constexpr int NT = (POINTS + 63) / 64 * 64;

template <class St, int FM, bool WALLS>
__global__ __launch_bounds__(NT) void k_step_box(const typename St::bits_t* __restrict__ src,
                                                 typename St::bits_t* __restrict__ dst,
                                                 const uint8_t* __restrict__ flags,
                                                 const uint32_t* __restrict__ smask,
                                                 const uint32_t* __restrict__ mmask,
                                                 const float* __restrict__ ff, StepArgs a)
{
    using B = typename St::bits_t;
    constexpr bool FORCE = FM != FORCE_NONE;
    __shared__ B ex[Q][POINTS];
    const Dims& d = a.d;
    const int x0 = blockIdx.x * BX - 1, y0 = blockIdx.y * BY - 1, z0 = blockIdx.z * BZ - 1;
    auto wrap = [](int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); };
    auto point = [&](float h[Q], uint32_t mv, size_t c) {
        if (WALLS && __builtin_amdgcn_ballot_w64(mv != 0u) != 0ull) {
#pragma unroll
            for (int i = 1; i < Q; ++i) h[i] = ((mv >> i) & 1u) ? h[i] + a.mw[i] : h[i];
        }
        float F[3] = {0, 0, 0};
        if (FM == FORCE_FIELD) {
#pragma unroll
            for (int k = 0; k < 3; ++k) F[k] = ff[k * (size_t)d.N + c];
        } else if (FM == FORCE_UNIFORM) {
            F[0] = a.Fx; F[1] = a.Fy; F[2] = a.Fz;
        }
        bgk_collide<FORCE>(h, a.omega, a.cF, F[0], F[1], F[2]);
    };
    const int p = threadIdx.x;
    {
        const int pz = p / (HX * HY), r = p - pz * (HX * HY), py = r / HX, px = r - py * HX;
        // not in the halo of the lattice's last boxes
        if (p < POINTS && x0 + px <= d.nx && y0 + py <= d.ny && z0 + pz <= d.nz) {
            const int x = wrap(x0 + px, d.nx), y = wrap(y0 + py, d.ny);
            const uint32_t z = (uint32_t)wrap(z0 + pz, d.nz);
            const uint32_t zm = wrap_m(z, (uint32_t)d.nz), zp = wrap_p(z, (uint32_t)d.nz);
            uint32_t on[Q];
            pull_offsets(d, x, y, on);
            const uint32_t c = z * d.nxy + on[0];
            uint32_t m = 0, mv = 0;
            if (WALLS) {
                const uint8_t fl = flags[c];
                if (fl & NEAR_WALL) m = smask[c];
                if (fl & NEAR_MOVING) mv = mmask[c];
            }
            B raw[Q];
            float h[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) raw[i] = src[((size_t)src_slab(i, z, zm, zp) * Q + i) * d.nxy + on[i]];
            if (WALLS && __builtin_amdgcn_ballot_w64(m != 0u) != 0ull) {
#pragma unroll
                for (int i = 1; i < Q; ++i)
                    if ((m >> i) & 1u) raw[i] = src[((size_t)z * Q + OPP[i]) * d.nxy + on[0]];
            }
#pragma unroll
            for (int i = 0; i < Q; ++i) h[i] = St::off_b(raw[i], i);
            point(h, mv, c);
#pragma unroll
            for (int i = 0; i < Q; ++i) ex[i][p] = St::enc_b(h[i], i);
        }
    }
    __syncthreads();
    const int pz = p / (BX * BY), r = p - pz * (BX * BY), py = r / BX, px = r - py * BX;
    const int x = x0 + 1 + px, y = y0 + 1 + py, z = z0 + 1 + pz;
    if (p >= OUT || x >= d.nx || y >= d.ny || z >= d.nz) return;
    const uint32_t o = (uint32_t)y * (uint32_t)d.nx + (uint32_t)x, c = (uint32_t)z * d.nxy + o;
    uint32_t m = 0, mv = 0, fl = 0;
    if (WALLS) {
        fl = flags[c];
        if (fl & NEAR_WALL) m = smask[c];
        if (fl & NEAR_MOVING) mv = mmask[c];
    }
    const int l = ((pz + 1) * HY + py + 1) * HX + px + 1;
    float h[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        B v = ex[i][l - EX[i] - EY[i] * HX - EZ[i] * HX * HY];
        if (WALLS && i > 0) {
            const B own = ex[OPP[i]][l];
            v = ((m >> i) & 1u) ? own : v;
        }
        h[i] = St::off_b(v, i);
    }
    point(h, mv, c);
#pragma unroll
    for (int i = 0; i < Q; ++i)   // solid points are stored as the rest state
        dst[((size_t)z * Q + i) * d.nxy + o] = St::enc_b((WALLS && (fl & TYPE_MASK)) ? 0.0f : h[i], i);
}

template <class St, int FM, bool WALLS>
static hipError_t box_launch(const void* a, void* b, const uint8_t* flags, const uint32_t* sm, const uint32_t* mm,
                     const float* ff, const StepArgs& args, hipStream_t s)
{
    using B = typename St::bits_t;
    const Dims& d = args.d;
    hipLaunchKernelGGL((k_step_box<St, FM, WALLS>),
                       dim3((d.nx + BX - 1) / BX, (d.ny + BY - 1) / BY, (d.nz + BZ - 1) / BZ), dim3(NT), 0, s,
                       static_cast<const B*>(a), static_cast<B*>(b), flags, sm, mm, ff, args);
    return hipGetLastError();
}

template <class St, bool WALLS>
static hipError_t box_fm(int fm, const void* a, void* b, const uint8_t* flags, const uint32_t* sm, const uint32_t* mm,
                         const float* ff, const StepArgs& args, hipStream_t s)
{
    switch (fm) {
    case FORCE_UNIFORM: return box_launch<St, FORCE_UNIFORM, WALLS>(a, b, flags, sm, mm, ff, args, s);
    case FORCE_FIELD: return box_launch<St, FORCE_FIELD, WALLS>(a, b, flags, sm, mm, ff, args, s);
    default: return box_launch<St, FORCE_NONE, WALLS>(a, b, flags, sm, mm, ff, args, s);
    }
}

template <bool WALLS>
static hipError_t box_st(int storage, int fm, const void* a, void* b, const uint8_t* flags, const uint32_t* sm,
                         const uint32_t* mm, const float* ff, const StepArgs& args, hipStream_t s)
{
    switch (storage) {
    case 1: return box_fm<StF16, WALLS>(fm, a, b, flags, sm, mm, ff, args, s);
    case 2: return box_fm<StBF16, WALLS>(fm, a, b, flags, sm, mm, ff, args, s);
    default: return box_fm<StF32, WALLS>(fm, a, b, flags, sm, mm, ff, args, s);
    }
}

hipError_t launch_step_box(int storage, int fm, const void* a, void* b, const uint8_t* flags, const uint32_t* sm,
                           const uint32_t* mm, const float* ff, const StepArgs& args, bool walls, hipStream_t s)
{
    return walls ? box_st<true>(storage, fm, a, b, flags, sm, mm, ff, args, s)
                 : box_st<false>(storage, fm, a, b, flags, sm, mm, ff, args, s);
}

}  // namespace lbmk
