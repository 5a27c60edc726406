// Two pull steps per launch (two-array pattern) for gfx950.
//
// A single step has to move the whole state through HBM once each way, and it
// already runs at the device's copy rate, so the only way to take less time
// per step is to move the state less often. A work-group marches along z over
// a tile of x and y. In each plane it computes s^{t+1} of the tile and of a
// halo one point wide (19 gathered loads, the pull of Algorithm 3 of Mawson &
// Revell), exchanges it with the lateral neighbours through LDS, and computes
// s^{t+2} of the tile one plane behind: per two steps the state is read and
// written once. The halo is computed again by the neighbouring tiles.
//
// MI355X, us per step, one step per launch / this: 256^3 FP32 cavity 411 / 279,
// periodic 417 / 260, sphere duct 128x128x256 107 / 86, 256^3 FP16 periodic 217 /
// 180. What bounds it: a plane's loads and stores, 256 of the 279 us with the
// arithmetic taken out; the arithmetic and LDS exchange alone take 99 to 114.
// Reads from memory are 1.13 to 1.35 times the state (the halo rows of
// neighbouring tiles that miss L2), writes exact. Tiles of 64 columns make a wave's stores one row; one
// work-group of 16 waves per compute unit, because halving it would double the
// halo, and 128 registers per work-item leave room for no second one.
//
// Per point both steps do the arithmetic of the one-step kernels on values
// rounded to the storage format in between, so the result is the same bit for
// bit.
#include "kernels.hpp"

using namespace d3q19;

namespace lbmk {

namespace {

constexpr int NT = PAIR_MAX_THREADS;
constexpr int P = PAIR_PITCH;

// Exchange planes of s^{t+1} in LDS: the 16 directions with a lateral
// component; with walls also 5 and 6, whose own-point values are the bounced
// ones of 6 and 5. Separate planes per direction: a wave then reads
// consecutive words, whatever its shift. (Grouping the directions of one
// neighbour into two-element words saved LDS instructions but measured 3%
// slower.)
template <class B, bool WALLS>
struct Exchange {
    B s[WALLS ? 18 : 16][NT];
    static constexpr int slot(int i) { return i < 5 ? i - 1 : (i < 7 ? i + 11 : i - 3); }
    __device__ __forceinline__ B& at(int i, int idx) { return s[slot(i)][idx]; }
    __device__ __forceinline__ B at(int i, int idx) const { return s[slot(i)][idx]; }
};

// Work-group barrier that orders LDS accesses only: the global loads of the
// next plane and the stores of the last one stay in flight across it.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// OR of v over the wave, as a scalar.
__device__ __forceinline__ uint32_t wave_or(uint32_t v)
{
    if (__builtin_amdgcn_ballot_w64(v != 0u) == 0ull) return 0u;
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);   // row_shr:4
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);   // row_shr:8
    return (uint32_t)(__builtin_amdgcn_readlane((int)v, 15) | __builtin_amdgcn_readlane((int)v, 31) |
                      __builtin_amdgcn_readlane((int)v, 47) | __builtin_amdgcn_readlane((int)v, 63));
}

// Store of one element (HINT 2: non-temporal); an offset of PAIR_DROP lies outside the
// resource and is discarded by the range check, so that every work-item
// issues the same stores (a branch around them would make the compiler wait
// for them before the next plane's loads are used).
constexpr uint32_t PAIR_DROP = 0xfffffff0u;
template <int HINT, class B>
__device__ __forceinline__ void store_or_drop(B v, B* base, uint32_t bytes, uint32_t off)
{
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, (short)0, (int)bytes, 0x00020000);
    if constexpr (sizeof(B) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, HINT);
    else
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, v), r, off, 0, HINT);
}

// The march of one (x, y) column along the planes z0 .. z0 + depth - 1.
// OUT: the wave holds output points; the others only provide s^{t+1} of the
// halo, and take the same barriers.
template <class St, int FM, bool WALLS, bool MOVING, bool ONSITE, bool STREAM, bool OUT>
__device__ __forceinline__ void pair_march(const typename St::bits_t* __restrict__ src,
                                           typename St::bits_t* __restrict__ dst, const uint8_t* __restrict__ flags,
                                           const uint32_t* __restrict__ smask, const uint32_t* __restrict__ mmask,
                                           const float* __restrict__ ff, const StepArgs& a,
                                           Exchange<typename St::bits_t, WALLS>* ex, int x, int y, int z0, int depth,
                                           int lidx, bool out)
{
    using B = typename St::bits_t;
    constexpr bool FORCE = FM != FORCE_NONE;
    const Dims& d = a.d;
    const uint32_t nz = (uint32_t)d.nz;
    uint32_t on[Q];
    pull_offsets(d, x, y, on);
    const uint32_t o = on[0];
#pragma unroll
    for (int i = 0; i < Q; ++i) on[i] *= (uint32_t)sizeof(B);   // byte offsets
    auto at = [](const B* base, uint32_t bytes) -> B {
        return *reinterpret_cast<const B*>(reinterpret_cast<const char*>(base) + bytes);
    };
    const int zend = z0 + depth;   // the last plane of s^{t+1}
    auto wrapz = [&](int z) -> uint32_t {
        z = z < 0 ? z + (int)nz : z;
        return (uint32_t)(z >= (int)nz ? z - (int)nz : z);
    };

    // Gather of plane z in flight. Bounced directions take the point's own
    // opposite population instead: m holds the point's solid-neighbour bits,
    // w their OR over the wave, so that a wave only runs the directions that
    // one of its points bounces.
    B raw[Q];
    auto fetch = [&](uint32_t z, uint32_t m, uint32_t w) {
        const uint32_t zm = wrap_m(z, nz), zp = wrap_p(z, nz);
#pragma unroll
        for (int i = 0; i < Q; ++i) raw[i] = at(plane(src, d, i, src_slab(i, z, zm, zp)), on[i]);
        if (WALLS && w) {
#pragma unroll
            for (int i = 1; i < Q; ++i)
                if ((w >> i) & 1u) {
                    if ((m >> i) & 1u) raw[i] = at(plane(src, d, OPP[i], z), on[0]);
                }
        }
    };
    float h[Q];
    auto decode = [&]() {
#pragma unroll
        for (int i = 0; i < Q; ++i) h[i] = St::off_b(raw[i], i);
    };

    // Flag bytes and masks, loaded ahead of their use: the flag byte three
    // planes before the plane is computed, the masks (only where the flag
    // says so) two, the gather one. Mask words: neighbour bits | flag << 24.
    constexpr uint32_t BITS = 0x7fffeu;
    auto flag_at = [&](int z) -> uint32_t { return flags[(size_t)wrapz(min(z, zend)) * d.nxy + o]; };
    auto bits_at = [&](const uint32_t* masks, bool near, int z) -> uint32_t {
        uint32_t m = 0;
        if (near) m = masks[(size_t)wrapz(min(z, zend)) * d.nxy + o];
        return m;
    };
    uint32_t mp = 0, m0 = 0, m1 = 0, fl2 = 0;   // planes zt-1, zt, zt+1, zt+2
    uint32_t wp = 0, w0 = 0, w1 = 0;
    uint32_t vp = 0, v0 = 0, v1 = 0;            // moving-wall bits
    if (WALLS) {
        const uint32_t f0 = flag_at(z0 - 1), f1 = flag_at(z0);
        fl2 = flag_at(z0 + 1);
        m0 = bits_at(smask, f0 & NEAR_WALL, z0 - 1) | (f0 << 24);
        if (MOVING) v0 = bits_at(mmask, f0 & NEAR_MOVING, z0 - 1);
        m1 = bits_at(smask, f1 & NEAR_WALL, z0) | (f1 << 24);
        if (MOVING) v1 = bits_at(mmask, f1 & NEAR_MOVING, z0);
        w0 = wave_or(m0 & BITS);
        w1 = wave_or(m1 & BITS);
    }
    float Fp[3] = {0, 0, 0}, F0[3] = {0, 0, 0}, F1[3] = {0, 0, 0};   // force field, planes zt-1, zt, zt+1
    auto force_at = [&](int z, float F[3]) {
        if (FM == FORCE_FIELD) {
            const float* p = ff + (size_t)wrapz(min(z, zend)) * d.nxy + o;
#pragma unroll
            for (int k = 0; k < 3; ++k) F[k] = p[k * (size_t)d.N];
        }
    };
    // moving-wall terms and collision of one point
    auto point = [&](uint32_t w, uint32_t v, const float F[3]) {
        const float Fx = FM == FORCE_FIELD ? F[0] : (FM == FORCE_UNIFORM ? a.Fx : 0.0f);
        const float Fy = FM == FORCE_FIELD ? F[1] : (FM == FORCE_UNIFORM ? a.Fy : 0.0f);
        const float Fz = FM == FORCE_FIELD ? F[2] : (FM == FORCE_UNIFORM ? a.Fz : 0.0f);
        if (MOVING && __builtin_amdgcn_ballot_w64(v != 0u) != 0ull) {
#pragma unroll
            for (int i = 1; i < Q; ++i)
                if ((w >> i) & 1u) h[i] = ((v >> i) & 1u) ? h[i] + a.mw[i] : h[i];
        }
        bgk_collide<FORCE>(h, a.omega, a.cF, Fx, Fy, Fz);
    };

    // Rebuilds the unknowns of on-site nodes from their neighbour bits, as the
    // one-step kernels do before they collide.
    static_assert(!(ONSITE && FORCE), "the forced kernels have no registers left for the rebuild");
    auto rebuild = [&](uint32_t m) {
        if (!ONSITE || !((m >> 24) & ONSITE_NODE)) return;
        const bool mv = ((m >> 24) & ONSITE_MOVING) != 0u;
        onsite_rebuild<false>(h, m & BITS, mv ? a.uw[0] : 0.0f, mv ? a.uw[1] : 0.0f, mv ? a.uw[2] : 0.0f, 0.0f, 0.0f,
                              0.0f);
    };

    force_at(z0 - 1, F0);
    fetch(wrapz(z0 - 1), m0, w0);
    decode();
    // keeps this decode out of the loop: merged with the one at its end it
    // would run after the next plane's loads are issued, and wait for them
#pragma unroll
    for (int i = 0; i < Q; ++i) asm volatile("" : "+v"(h[i]));
    // s^{t+1} gathered for the next output plane (e_z = 0 and +1 in q) and for
    // the one after it (e_z = +1 in up)
    B q[Q], up[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) { q[i] = B(0); up[i] = B(0); }
    const int lo = out ? lidx : P + 1;   // work-items without an output point read some point of the tile

    for (int it = 0; it < depth + 2; ++it) {
        const int zt = z0 - 1 + it;   // plane of s^{t+1}
        rebuild(m0);   // before the loads, whose registers it can use (after them 5 spill, 256^3 361 -> 378 us)
        uint32_t sm2 = 0, v2 = 0, fl3 = 0;
        // the wave issues its loads at raised priority: they get into the
        // memory pipeline before other waves' arithmetic (3% on the cavity)
        __builtin_amdgcn_s_setprio(2);
        if (WALLS) {
            fl3 = flag_at(zt + 3);
            sm2 = bits_at(smask, fl2 & NEAR_WALL, zt + 2);
            if (MOVING) v2 = bits_at(mmask, fl2 & NEAR_MOVING, zt + 2);
        }
        force_at(zt + 1, F1);
        fetch(wrapz(min(zt + 1, zend)), m1, w1);
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);   // the loads stay in front of the arithmetic

        point(w0, v0, F0);
        auto& cur = ex[it & 1];
        const auto& prev = ex[(it & 1) ^ 1];
        B e[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            e[i] = St::enc_b(h[i], i);
            if (i != 0 && (WALLS || (i != 5 && i != 6))) cur.at(i, lidx) = e[i];
        }
        // One barrier per plane: the buffer written in the next plane was last
        // read by other work-items before this barrier.
        lds_barrier();

        if (OUT) {
            // second step, plane zt - 1
            auto near = [&](int i) -> B { return cur.at(i, lo - EX[i] - EY[i] * P); };
            q[6] = e[6];
#pragma unroll
            for (int i = 1; i < Q; ++i)
                if (EZ[i] == -1 && i != 6) q[i] = near(i);
            if (WALLS && wp) {
#pragma unroll
                for (int i = 1; i < Q; ++i)
                    if ((wp >> i) & 1u) {
                        const B own = prev.at(OPP[i], lidx);
                        q[i] = ((mp >> i) & 1u) ? own : q[i];
                    }
            }
#pragma unroll
            for (int i = 0; i < Q; ++i) h[i] = St::off_b(q[i], i);
            rebuild(mp);
            point(wp, vp, Fp);
            if (WALLS) {
                // solid points inside a tile are stored as the rest state, as
                // the one-step kernels do: holes would cost partial lines
                const bool sol = ((mp >> 24) & TYPE_MASK) != 0u;
                if (__builtin_amdgcn_ballot_w64(sol) != 0ull) {
#pragma unroll
                    for (int i = 0; i < Q; ++i) h[i] = sol ? 0.0f : h[i];
                }
            }
            const uint32_t off = (out && it >= 2) ? on[0] : PAIR_DROP;
            const uint32_t zo = (uint32_t)max(zt - 1, 0);
#pragma unroll
            for (int i = 0; i < Q; ++i)
                store_or_drop<STREAM ? 2 : 0>(St::enc_b(h[i], i), plane(dst, d, i, zo), d.nxy * (uint32_t)sizeof(B),
                                              off);
            // gathers of plane zt for the output planes zt and zt + 1
            q[0] = e[0];
            q[5] = up[5];
            up[5] = e[5];
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                if (i == 5 || EZ[i] == -1) continue;
                if (EZ[i] == 1) {
                    q[i] = up[i];
                    up[i] = near(i);
                } else {
                    q[i] = near(i);
                }
            }
        }
        if (WALLS) {
            mp = m0; m0 = m1; m1 = sm2 | (fl2 << 24); fl2 = fl3;
            vp = v0; v0 = v1; v1 = v2;
            wp = w0; w0 = w1; w1 = wave_or(m1 & BITS);
        }
        if (FM == FORCE_FIELD) {
#pragma unroll
            for (int k = 0; k < 3; ++k) { Fp[k] = F0[k]; F0[k] = F1[k]; }
        }
        __builtin_amdgcn_sched_barrier(0);
        decode();
    }
}

}  // namespace

template <class St, int FM, bool WALLS, bool MOVING, bool ONSITE, bool STREAM>
__global__ __launch_bounds__(NT, NT / 256) void k_step_pair(const typename St::bits_t* __restrict__ src,
                                                            typename St::bits_t* __restrict__ dst,
                                                            const uint8_t* __restrict__ flags,
                                                            const uint32_t* __restrict__ smask,
                                                            const uint32_t* __restrict__ mmask,
                                                            const float* __restrict__ ff, StepArgs a, PairShape ps)
{
    __shared__ Exchange<typename St::bits_t, WALLS> ex[2];   // current and previous plane
    const Dims& d = a.d;
    const int tid = threadIdx.x;

    // Work-groups go to the 8 XCDs in turn; each XCD takes consecutive tiles
    // (x fastest, then y, then z), whose overlapping reads meet in its L2.
    const uint32_t per_xcd = (ps.groups + 7u) / 8u;
    const uint32_t t = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if (t >= ps.groups) return;
    const uint32_t tz = t / (ps.ntx * ps.nty), txy = t - tz * (ps.ntx * ps.nty);
    const uint32_t ty = txy / ps.ntx, tx = txy - ty * ps.ntx;
    const int z0 = (int)(tz * ps.depth);
    const int depth = min((int)ps.depth, d.nz - z0);

    // The first rows * tx work-items take the columns of the tile, row by row,
    // so that a wave's stores are whole rows; the rest the two halo columns.
    const int TX = (int)ps.tx, R = (int)ps.rows;
    int lrow, lcol;
    if (tid < R * TX) {
        lrow = tid / TX;
        lcol = tid - lrow * TX + 1;
    } else {
        const int k = tid - R * TX;
        lrow = min(k >> 1, R - 1);   // surplus work-items repeat a halo point
        lcol = (k & 1) ? TX + 1 : 0;
    }
    const int lidx = lrow * P + lcol;
    int x = (int)(tx * ps.tx) + lcol - 1, y = (int)ty * (R - 2) + lrow - 1;
    const bool out = tid < R * TX && lrow >= 1 && lrow <= R - 2 && x < d.nx && y < d.ny;
    x = x < 0 ? x + d.nx : (x >= d.nx ? x - d.nx : x);
    y = y < 0 ? y + d.ny : (y >= d.ny ? y - d.ny : y);
    if (!WALLS || __builtin_amdgcn_ballot_w64(out) != 0ull)
        pair_march<St, FM, WALLS, MOVING, ONSITE, STREAM, true>(src, dst, flags, smask, mmask, ff, a, ex, x, y, z0, depth, lidx, out);
    else
        pair_march<St, FM, WALLS, MOVING, ONSITE, STREAM, false>(src, dst, flags, smask, mmask, ff, a, ex, x, y, z0, depth, lidx, out);
}

template <class St, int FM, bool WALLS, bool MOVING, bool ONSITE, bool STREAM>
static hipError_t pair_stream(const void* a, void* b, const uint8_t* flags, const uint32_t* sm, const uint32_t* mm,
                              const float* ff, const StepArgs& args, const PairShape& ps, hipStream_t s, const void** name)
{
    using B = typename St::bits_t;
    if (name) {
        *name = reinterpret_cast<const void*>(&k_step_pair<St, FM, WALLS, MOVING, ONSITE, STREAM>);
        return hipSuccess;
    }
    hipLaunchKernelGGL((k_step_pair<St, FM, WALLS, MOVING, ONSITE, STREAM>), dim3((ps.groups + 7u) / 8u * 8u), dim3(ps.threads), 0,
                       s, static_cast<const B*>(a), static_cast<B*>(b), flags, sm, mm, ff, args, ps);
    return hipGetLastError();
}

template <class St, int FM, bool WALLS, bool MOVING, bool ONSITE>
static hipError_t pair_launch(const void* a, void* b, const uint8_t* flags, const uint32_t* sm, const uint32_t* mm,
                              const float* ff, const StepArgs& args, const PairShape& ps, hipStream_t s, const void** name)
{
    return ps.stream ? pair_stream<St, FM, WALLS, MOVING, ONSITE, true>(a, b, flags, sm, mm, ff, args, ps, s, name)
                     : pair_stream<St, FM, WALLS, MOVING, ONSITE, false>(a, b, flags, sm, mm, ff, args, ps, s, name);
}

template <class St, bool WALLS, bool MOVING, bool ONSITE>
static hipError_t pair_fm(int fm, const void* a, void* b, const uint8_t* flags, const uint32_t* sm, const uint32_t* mm,
                          const float* ff, const StepArgs& args, const PairShape& ps, hipStream_t s, const void** name)
{
    switch (fm) {
    case FORCE_UNIFORM:   // FP32 only
        if constexpr (sizeof(typename St::bits_t) == 4)
            return pair_launch<St, FORCE_UNIFORM, WALLS, MOVING, ONSITE>(a, b, flags, sm, mm, ff, args, ps, s, name);
        return hipErrorInvalidValue;
    case FORCE_FIELD: return pair_launch<St, FORCE_FIELD, WALLS, MOVING, ONSITE>(a, b, flags, sm, mm, ff, args, ps, s, name);
    default: return pair_launch<St, FORCE_NONE, WALLS, MOVING, ONSITE>(a, b, flags, sm, mm, ff, args, ps, s, name);
    }
}

hipError_t launch_step_pair(int storage, int fm, const void* a, void* b, const uint8_t* flags, const uint32_t* sm,
                            const uint32_t* mm, const float* ff, const StepArgs& args, const PairShape& ps, bool walls,
                            bool moving, bool onsite, hipStream_t s, const void** name)
{
    if (ps.rows < 3 || ps.rows * P > (uint32_t)NT || ps.tx + 2 > (uint32_t)P || ps.threads > (uint32_t)NT ||
        ps.rows * (ps.tx + 2) > ps.threads)
        return hipErrorInvalidValue;
    if (onsite) {
        if (storage != 0 || !walls || moving || fm != FORCE_NONE) return hipErrorInvalidValue;
        return pair_launch<StF32, FORCE_NONE, true, false, true>(a, b, flags, sm, mm, ff, args, ps, s, name);
    }
    if (storage == 0 && walls && moving) return pair_fm<StF32, true, true, false>(fm, a, b, flags, sm, mm, ff, args, ps, s, name);
    if (storage == 0 && walls) return pair_fm<StF32, true, false, false>(fm, a, b, flags, sm, mm, ff, args, ps, s, name);
    if (storage == 0) return pair_fm<StF32, false, false, false>(fm, a, b, flags, sm, mm, ff, args, ps, s, name);
    if (storage == 1 && !walls) return pair_fm<StF16, false, false, false>(fm, a, b, flags, sm, mm, ff, args, ps, s, name);
    if (storage == 2 && !walls) return pair_fm<StBF16, false, false, false>(fm, a, b, flags, sm, mm, ff, args, ps, s, name);
    return hipErrorInvalidValue;
}

}  // namespace lbmk
