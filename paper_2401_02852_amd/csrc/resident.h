// Register layouts of small whole states (n = 10 .. 14, 16 amplitudes a thread,
// 2^(n-4) threads), shared by the circuit and the gradient kernels. Element x
// splits into slot, lane and wave bits in two layouts, each with a partner that 16-
// and 32-lane permute swaps reach without LDS:
//   A  slots e{0, 1, 2, 3}, lanes e{6, 7, 8, 9, 4, 5}; A2: e{2, 3} and e{4, 5}
//      exchanged (lane bits 4 and 5 with slot bits 2 and 3);
//   B  slots e{6, 7, 8, 9}, lane bits 4 and 5 e{10, 11}; B2: e{8, 9} and e{10, 11}
//      exchanged; e12 and e13 on lane bits 0 and 1, where a butterfly's partner
//      is one lane-permuted move away.
// A layer is two trips through LDS, A2 -> B and B2 -> A, with qubits mixed in
// ascending order; phases and sums in A, where a thread's costs are 16
// consecutive ones, held in registers.
#pragma once

#include <type_traits>

#include "sweep_common.h"

namespace qnae {
namespace tile {

template <int NB>
struct RLay {
    static constexpr int lane_a[6] = {6, 7, 8, 9, 4, 5}, wave_a[4] = {10, 11, 12, 13};
    static constexpr int lane_b[6] = {NB >= 13 ? 12 : 0, NB == 14 ? 13 : NB == 13 ? 0 : 1, NB == 14 ? 0 : NB == 13 ? 1 : 2,
                                      NB == 14 ? 1 : 3,  NB >= 11 ? 10 : 4,                NB >= 12 ? 11 : NB == 11 ? 4 : 5};
    static constexpr int wave_b[4] = {NB >= 13 ? 2 : NB == 12 ? 4 : 5, NB == 14 ? 3 : NB == 13 ? 4 : 5, NB == 14 ? 4 : 5, 5};
    static constexpr int waves = NB - 10;  // wave bits
};
template <int NB>
constexpr int kRegThreads = 1 << (NB - 4);

// LDS place of element e: additive over its bits, no two elements alike (each
// bit's step exceeds the largest sum of the lower ones), and 16 consecutive
// lanes with single elements on 16 bank pairs, 8 with pairs on 8 16-byte groups.
__device__ __forceinline__ constexpr uint32_t rplace(uint32_t e) {
    constexpr uint32_t c[8] = {2, 4, 8, 16, 32, 64, 132, 264};
    uint32_t p = e;
    for (int i = 0; i < 8; ++i) p += ((e >> (6 + i)) & 1u) * c[i];
    return p;
}
constexpr uint32_t reg_lds(int nb) { return (rplace((1u << nb) - 1u) + 2u) / 2u * 2u; }

// Slot bit 2 <-> lane bit 4: a 16-lane permute swap of registers (A, B) leaves
// rows (A0, B0, A2, B2) in A and (A1, B1, A3, B3) in B.
__device__ __forceinline__ void r_swap16(float2 (&v)[16]) {
    auto swap = [](float& a, float& b) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    };
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        if (j & 4) continue;
        swap(v[j].x, v[j | 4].x);
        swap(v[j].y, v[j | 4].y);
    }
}

// Butterfly with the lane that a quad permutation gives as partner.
template <int CTRL>
__device__ __forceinline__ void lane_bfly(float2 (&v)[16], float t) {
    auto other = [](float x) {
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true));
    };
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const float px = other(v[j].x), py = other(v[j].y);
        v[j] = make_float2(fmaf(t, py, v[j].x), fmaf(-t, px, v[j].y));
    }
}
constexpr int kLaneXor1 = 0xB1, kLaneXor2 = 0x4E;  // quad permutations [1, 0, 3, 2] and [2, 3, 0, 1]

// A thread's 16 costs, at x0 .. x0 + 15 or (flip) at the mirrored places.
template <int NB, typename CT>
__device__ __forceinline__ void load_costs(uint32_t (&c)[4 * sizeof(CT)], const CT* cost, uint32_t x0, bool flip) {
    constexpr int W = 4 * (int)sizeof(CT);
    const uint4* const q = (const uint4*)(cost + (flip ? (1u << NB) - 16u - x0 : x0));
    uint32_t w[W];
#pragma unroll
    for (int i = 0; i < W / 4; ++i) {
        const uint4 u = q[i];
        w[4 * i] = u.x, w[4 * i + 1] = u.y, w[4 * i + 2] = u.z, w[4 * i + 3] = u.w;
    }
    auto rev = [](uint32_t x) { return sizeof(CT) == 1 ? __builtin_bswap32(x) : (x >> 16) | (x << 16); };
#pragma unroll
    for (int i = 0; i < W; ++i) c[i] = flip ? rev(w[W - 1 - i]) : w[i];
}
template <typename CT>
__device__ __forceinline__ uint32_t cost_of(const uint32_t (&c)[4 * sizeof(CT)], int j) {
    return sizeof(CT) == 1 ? (c[j >> 2] >> (8 * (j & 3))) & 0xffu : (c[j >> 1] >> (16 * (j & 1))) & 0xffffu;
}

// A thread's places: its elements in the four layouts as LDS offsets, and its
// first element in A.
template <int NB>
struct RegPlaces {
    uint32_t a, a2, b, b2, x0;
    __device__ __forceinline__ RegPlaces(uint32_t lane, uint32_t wave) {
        uint32_t ea = 0u, eb = 0u;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            ea |= ((lane >> i) & 1u) << RLay<NB>::lane_a[i];
            eb |= ((lane >> i) & 1u) << RLay<NB>::lane_b[i];
        }
#pragma unroll
        for (int i = 0; i < RLay<NB>::waves; ++i) {
            ea |= ((wave >> i) & 1u) << RLay<NB>::wave_a[i];
            eb |= ((wave >> i) & 1u) << RLay<NB>::wave_b[i];
        }
        // A2 and B2: lane bits 4 and 5 hold what their slots held
        constexpr uint32_t out_b = (NB >= 11 ? 1u << 10 : 0u) | (NB >= 12 ? 1u << 11 : 0u);
        const uint32_t ea2 = (ea & ~0x30u) | (lane & 0x30u) >> 2;
        const uint32_t eb2 = (eb & ~out_b) | (NB >= 11 ? (lane >> 4 & 1u) << 8 : 0u) | (NB >= 12 ? (lane >> 5) << 9 : 0u);
        a = rplace(ea), a2 = rplace(ea2), b = rplace(eb), b2 = rplace(eb2), x0 = ea;
    }
    __device__ __forceinline__ void put_a2(float2* lds, const float2 (&v)[16]) const {
#pragma unroll
        for (int j = 0; j < 16; j += 2)
            *(float4*)(lds + a2 + rplace((uint32_t)(j & 3) | (uint32_t)(j & 12) << 2)) =
                make_float4(v[j].x, v[j].y, v[j + 1].x, v[j + 1].y);
    }
    __device__ __forceinline__ void get_b(const float2* lds, float2 (&v)[16]) const {
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = lds[b + rplace((uint32_t)j << 6)];
    }
    __device__ __forceinline__ void put_b2(float2* lds, const float2 (&v)[16]) const {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const uint32_t e = (uint32_t)(j & 3) << 6 | (uint32_t)(j >> 2 & 1) << (NB >= 11 ? 10 : 8) |
                               (uint32_t)(j >> 3) << (NB >= 12 ? 11 : 9);
            lds[b2 + rplace(e)] = v[j];
        }
    }
    __device__ __forceinline__ void get_a(const float2* lds, float2 (&v)[16]) const {
#pragma unroll
        for (int j = 0; j < 16; j += 2) {
            const float4 q = *(const float4*)(lds + a + j);
            v[j] = make_float2(q.x, q.y);
            v[j + 1] = make_float2(q.z, q.w);
        }
    }
};

}  // namespace tile
}  // namespace qnae
