// Device helpers shared by the sweep and adjoint kernels: complex product,
// register butterflies, the register layouts of a tile and the LDS transposes
// between them. See sweep.hip for the tiling scheme; the layouts of 14-bit tiles
// are in sweep14.hip.
#pragma once

#include "internal.h"

namespace qnae {
namespace tile {

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}

// Butterfly on register bit S of a register array of size NE:
// own' = own - i t partner for both members of each pair.
template <int NE, int S>
__device__ __forceinline__ void bfly(float2 (&v)[NE], float t) {
#pragma unroll
    for (int j = 0; j < NE; ++j) {
        if (j & (1 << S)) continue;
        const float2 a = v[j], b = v[j | (1 << S)];
        v[j] = make_float2(fmaf(t, b.y, a.x), fmaf(-t, b.x, a.y));
        v[j | (1 << S)] = make_float2(fmaf(t, a.y, b.x), fmaf(-t, a.x, b.y));
    }
}

// LDS operations of one wave complete in order, so a transpose that moves data
// only inside each wave's own part of the LDS tile needs no workgroup barrier:
// this keeps the compiler from moving LDS accesses across the point
// (wavefront-scope fences emit no code).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS position of element e of a reverse tile: two padding slots after every 64
// elements. The map is additive over disjoint bit sets of e, so an address is
// a per-thread base plus a compile-time constant per slot.
__device__ __forceinline__ constexpr uint32_t phys(uint32_t e) { return e + 2u * (e >> 6); }
template <int TB>
constexpr uint32_t lds_elems() { return phys((1u << TB) - 1u) + 1u; }

template <int C>
__device__ __forceinline__ float part(const float2& a) { return C == 0 ? a.x : a.y; }
template <int C>
__device__ __forceinline__ void set_part(float2& a, float x) {
    if (C == 0) a.x = x;
    else a.y = x;
}

// ---------------------------------------------------------------------------
// Layouts of the forward sweeps: tiles of 2^12 or 2^13 elements, 16 a
// thread (256 or 512 threads). Element e of the tile splits into a thread
// part (lane and wave bits) and a slot part (4 bits):
//   0  slots e{0, 7, 8, 9},  lanes e{1..5, 10},           waves e{6, 11..}
//   2  slots e{1, 2, 3, 4},  lanes e{0, 7, 8, 9, 10, 5},  waves e{6, 11..}
//   4  slots e{6, 11, 12, 4} (12 tile bits: e{6, 11, 7, 4}), lanes e{0..3, 10, 5},
//      the rest in the waves
// and layouts 1, 3 and 5 are 0, 2 and 4 with slot bit 3 and lane bit 5
// exchanged (e9 with e10, e4 with e5): one 32-lane permute swap per two registers,
// no LDS. Layouts 0 and 1 are the global ones (tile bit 0 pairs in one 16-byte
// access, 512 consecutive bytes a wave); transposes among 0..3 stay inside each
// wave's part of the LDS tile, those from or to 4 and 5 go through the whole
// tile. Mixed in each: 0 e{0, 7, 8, 9}; 1 e10; 2 e{1, 2, 3, 4}; 3 e5; 4 e{6, 11..},
// and, when the group's low run is not mixed and 2 and 3 are skipped, e4 in 4
// and e5 in 5.
//
// Half-state tiles (VIRT): the elements with the top tile bit set are the
// mirrored ones. In memory, LDS and layouts 0..3, where the top bit is a wave
// bit, they keep their storage order, in which their other tile bits read
// complemented; a butterfly on any other bit pairs the same elements either way.
// Layouts 4 and 5, which mix the top bit and hold it in a slot, take them by
// their true position: slots with the bit set address the complemented place,
// again a per-thread base plus a constant per slot.
// ---------------------------------------------------------------------------
template <int TB>
struct SLay {
    static constexpr int slot[6][4] = {{0, 7, 8, 9},
                                       {0, 7, 8, 10},
                                       {1, 2, 3, 4},
                                       {1, 2, 3, 5},
                                       {6, 11, TB == 12 ? 7 : 12, 4},
                                       {6, 11, TB == 12 ? 7 : 12, 5}};
    static constexpr int lane[6][6] = {{1, 2, 3, 4, 5, 10}, {1, 2, 3, 4, 5, 9},  {0, 7, 8, 9, 10, 5},
                                       {0, 7, 8, 9, 10, 4}, {0, 1, 2, 3, 10, 5}, {0, 1, 2, 3, 10, 4}};
    static constexpr int wave0[3] = {6, 11, 12};                           // layouts 0..3
    static constexpr int wave4[3] = {TB == 13 ? 7 : 8, TB == 13 ? 8 : 9, 9};  // layouts 4, 5
    static constexpr int top_slot = TB - 11;                                      // of the top tile bit in 4, 5
};
template <int TB>
constexpr int kSweepThreads = 1 << (TB - 4);
template <int TB, int LY>
__device__ __forceinline__ uint32_t st(uint32_t lane, uint32_t wave) {
    uint32_t e = 0u;
#pragma unroll
    for (int i = 0; i < 6; ++i) e |= ((lane >> i) & 1u) << SLay<TB>::lane[LY][i];
#pragma unroll
    for (int i = 0; i < TB - 10; ++i) e |= ((wave >> i) & 1u) << (LY < 4 ? SLay<TB>::wave0[i] : SLay<TB>::wave4[i]);
    return e;
}
template <int TB, int LY>
__host__ __device__ __forceinline__ constexpr uint32_t ss(int j) {
    uint32_t e = 0u;
    for (int i = 0; i < 4; ++i) e |= (uint32_t)((j >> i) & 1) << SLay<TB>::slot[LY][i];
    return e;
}

// Tile bits that send a launch through layouts 2 and 3 (USE1) when its masks
// hold one of them.
constexpr uint32_t low_bits = 0xfu;
// Tile bits mixed in layout LY.
template <int TB, int LY, bool USE1>
constexpr uint32_t s_mixed() {
    if (LY == 0) return (USE1 ? 1u : 0u) | 0x380u;
    if (LY == 1) return 0x400u;
    if (LY == 2) return 0x1eu;
    if (LY == 3) return 0x20u;
    if (LY == 4) return 0x40u | ((1u << TB) - 0x800u) | (!USE1 ? 0x10u : 0u);
    return !USE1 ? 0x20u : 0u;
}
// Slot bits layout LY can mix (compile time; the others get no butterfly), and
// those it mixes for tile mask m.
template <int TB, int LY, bool USE1>
constexpr uint32_t s_possible() {
    uint32_t r = 0u;
    for (int i = 0; i < 4; ++i) r |= ((s_mixed<TB, LY, USE1>() >> SLay<TB>::slot[LY][i]) & 1u) << i;
    return r;
}
template <int TB, int LY>
__device__ __forceinline__ uint32_t s_slots(uint32_t m) {
    uint32_t r = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) r |= ((m >> SLay<TB>::slot[LY][i]) & 1u) << i;
    return r;
}

// Slot bit 3 <-> lane bit 5: a 32-lane permute swap of registers (A, B) leaves
// A's low and B's low half in A and the high halves in B.
__device__ __forceinline__ void s_swap(float2 (&v)[16]) {
    auto swap = [](float& a, float& b) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    };
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        swap(v[j].x, v[j | 8].x);
        swap(v[j].y, v[j | 8].y);
    }
}

// LDS place of element e, of whole float2 elements and of component planes (one
// float per element, half the LDS): e + sum of c_i over its set bits i >= 6,
// non-decreasing sums chosen so that accesses of 32 lanes in layouts 2, 3
// (e{0, 7..10}) and 4, 5 (e{0..3, 10}) hit 32 distinct banks (b32) or bank pairs
// (b64). Two padding slots per 64 elements, which serve 16 lanes, put e10's lanes
// on the same pairs as the others': 4 conflict cycles per access in the half
// state's middle kind, half state n = 27, p = 10 3.93 -> 3.91 ms.
__device__ __forceinline__ constexpr uint32_t splace(uint32_t e) {
    constexpr uint32_t c[7] = {0, 2, 4, 8, 16, 32, 64};
    uint32_t p = e;
    for (int i = 0; i < 7; ++i) p += ((e >> (6 + i)) & 1u) * c[i];
    return p;
}
// floats of LDS a tile takes
template <int TB, bool PLANES>
constexpr uint32_t s_lds_floats() {
    return (PLANES ? 1u : 2u) * ((splace((1u << TB) - 1u) + 2u) / 2u * 2u);
}

// Calls f(j, place) for every slot j of layout LY.
template <int TB, int LY, bool VIRT, bool PLANES, typename F>
__device__ __forceinline__ void s_places(uint32_t lane, uint32_t wave, F&& f) {
    constexpr uint32_t top = 1u << (TB - 1), slots = ss<TB, LY>(15) & ~top;  // slot bits but the top one
    constexpr uint32_t threads = ((1u << TB) - 1u) & ~slots & ~top;
    const uint32_t t = st<TB, LY>(lane, wave);
    const uint32_t b = splace(t);
    const uint32_t bc = VIRT && LY >= 4 ? splace(top | (threads ^ t)) : b;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        if (VIRT && LY >= 4 && (ss<TB, LY>(j) & top)) f(j, bc + splace(slots ^ (ss<TB, LY>(j) & ~top)));
        else f(j, b + splace(ss<TB, LY>(j)));
    }
}

// The tile in layout LY to and from LDS: whole elements,
template <int TB, int LY, bool VIRT>
__device__ __forceinline__ void to_s(float2* lds, const float2 (&v)[16], uint32_t lane, uint32_t wave) {
    if constexpr (LY < 2) {
        float2* const b = lds + splace(st<TB, LY>(lane, wave));
#pragma unroll
        for (int jj = 0; jj < 8; ++jj)
            *(float4*)(b + splace(ss<TB, LY>(2 * jj))) =
                make_float4(v[2 * jj].x, v[2 * jj].y, v[2 * jj + 1].x, v[2 * jj + 1].y);
    } else {
        s_places<TB, LY, VIRT, false>(lane, wave, [&](int j, uint32_t at) { lds[at] = v[j]; });
    }
}
template <int TB, int LY, bool VIRT>
__device__ __forceinline__ void from_s(const float2* lds, float2 (&v)[16], uint32_t lane, uint32_t wave) {
    if constexpr (LY < 2) {
        const float2* const b = lds + splace(st<TB, LY>(lane, wave));
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            const float4 q = *(const float4*)(b + splace(ss<TB, LY>(2 * jj)));
            v[2 * jj] = make_float2(q.x, q.y);
            v[2 * jj + 1] = make_float2(q.z, q.w);
        }
    } else {
        s_places<TB, LY, VIRT, false>(lane, wave, [&](int j, uint32_t at) { v[j] = lds[at]; });
    }
}
// or component C to and from a plane.
template <int TB, int LY, bool VIRT, int C>
__device__ __forceinline__ void to_s_plane(float* lds, const float2 (&v)[16], uint32_t lane, uint32_t wave) {
    if constexpr (LY < 2) {
        float* const b = lds + splace(st<TB, LY>(lane, wave));
#pragma unroll
        for (int jj = 0; jj < 8; ++jj)
            *(float2*)(b + splace(ss<TB, LY>(2 * jj))) = make_float2(part<C>(v[2 * jj]), part<C>(v[2 * jj + 1]));
    } else {
        s_places<TB, LY, VIRT, true>(lane, wave, [&](int j, uint32_t at) { lds[at] = part<C>(v[j]); });
    }
}
template <int TB, int LY, bool VIRT, int C>
__device__ __forceinline__ void from_s_plane(const float* lds, float2 (&v)[16], uint32_t lane, uint32_t wave) {
    if constexpr (LY < 2) {
        const float* const b = lds + splace(st<TB, LY>(lane, wave));
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            const float2 q = *(const float2*)(b + splace(ss<TB, LY>(2 * jj)));
            set_part<C>(v[2 * jj], q.x);
            set_part<C>(v[2 * jj + 1], q.y);
        }
    } else {
        s_places<TB, LY, VIRT, true>(lane, wave, [&](int j, uint32_t at) { set_part<C>(v[j], lds[at]); });
    }
}

}  // namespace tile
}  // namespace qnae
