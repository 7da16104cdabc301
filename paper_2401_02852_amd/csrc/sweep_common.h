// Device code shared by the sweep kernels: state accesses, tile order, readout
// sums and the instance search of ragged batches.
#pragma once

#include <type_traits>

#include "tile.h"

namespace qnae {

// 14-bit tiles (sweep14.hip); see launch_sweep and launch_sweep_batch.
hipError_t launch_sweep14(int dtype, int kind, const SweepArgs& a, hipStream_t s);
hipError_t launch_sweep14_batch(int dtype, int kind, const SweepArgs* args, const uint32_t* first, int count,
                                uint32_t blocks, LaunchTo to, bool virt, int l1);

namespace {

using namespace tile;

// Every sweep streams the state through nontemporal loads and stores: each
// amplitude is touched once per sweep, and keeping it out of the caches'
// normal replacement measured faster in every kind (with the current qubit
// groups; the cost bytes, which neighbouring tiles share in the L2, keep
// ordinary loads).
typedef float f4v __attribute__((ext_vector_type(4)));
typedef float f2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float4 ld_state(const float2* p) {
    const f4v v = __builtin_nontemporal_load((const f4v*)p);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st_state(float2* p, float4 q) {
    f4v v = {q.x, q.y, q.z, q.w};
    __builtin_nontemporal_store(v, (f4v*)p);
}
__device__ __forceinline__ void st_state(float2* p, float2 q) {
    f2v v = {q.x, q.y};
    __builtin_nontemporal_store(v, (f2v*)p);
}

// First index of tile t. Consecutive tiles go to one XCD (blocks are dealt
// round-robin over the 8 XCDs), so tiles that share cache lines of the cost
// diagonal share an L2: each XCD takes one contiguous eighth of the tiles,
// except in the boundary kind, where each XCD takes every eighth chunk of 32
// consecutive tiles, so the 8 XCDs work on neighbouring chunks at once
// (measured faster there: 3.41 -> 3.29 ms at n = 30; slower for the middle
// kind). The tile index is deposited into the bits outside the tile (scalar
// ALU only).
template <int KIND>
__device__ __forceinline__ uint64_t tile_base(const SweepArgs& a, uint32_t t) {
    const uint32_t ntiles = 1u << a.nw;
    constexpr uint32_t kChunk = 32;
    uint64_t w = (KIND == SK_BOUNDARY && ntiles >= 8 * kChunk)
                     ? (uint64_t)((t >> 3) / kChunk) * (8 * kChunk) + (uint64_t)(t & 7u) * kChunk + ((t >> 3) % kChunk)
                 : ntiles >= 8 ? (uint64_t)(t & 7u) * (ntiles >> 3) + (t >> 3)
                               : (uint64_t)t;
    uint64_t base = 0;
    for (uint64_t m = a.wmask; m != 0ull; m &= m - 1ull) {
        if (w & 1ull) base |= m & (~m + 1ull);
        w >>= 1;
    }
    return base;
}

// The three readout sums of a workgroup (NW waves, costs cval(j)) to
// partial[0..2]. A thread's slots with and without the top slot bit TOP are
// summed apart, as balanced trees over the other slot bits: the sums do not
// depend on the order of the slots, a tile and its mirror image sum alike, and
// a run on the half state and one on the whole of a symmetric state agree to
// the rounding of the FP64 sums that follow. (A product fused into one of the
// two sides of an addition would break that.)
template <int NE, int TOP, int NW, typename C>
__device__ __forceinline__ void readout(const float2 (&v)[NE], C&& cval, double (&red)[3][NW], double* partial,
                                        uint32_t lane, uint32_t wave) {
    double d0 = 0.0, d1 = 0.0, d2 = 0.0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        constexpr int LV = NE == 32 ? 4 : 3;  // levels of a tree
        float t0[LV + 1], t1[LV + 1], t2[LV + 1];
#pragma unroll
        for (int i = 0; i < NE / 2; ++i) {
            constexpr int low = (1 << TOP) - 1;
            const int j = (i & low) | ((i & ~low) << 1) | (h << TOP);
            const float pr = fmaf(v[j].x, v[j].x, v[j].y * v[j].y);
            const uint32_t c = cval(j);
            float x0 = c == 0u ? pr : 0.f, x1 = (float)c * pr, x2 = pr;
            asm("" : "+v"(x1));  // a product of its own
            int k = 0;
#pragma unroll
            for (; k < LV && ((i >> k) & 1); ++k) {
                x0 += t0[k];
                x1 += t1[k];
                x2 += t2[k];
            }
            t0[k] = x0;
            t1[k] = x1;
            t2[k] = x2;
        }
        d0 += (double)t0[LV];
        d1 += (double)t1[LV];
        d2 += (double)t2[LV];
    }
    for (int off = 32; off > 0; off >>= 1) {
        d0 += __shfl_xor(d0, off);
        d1 += __shfl_xor(d1, off);
        d2 += __shfl_xor(d2, off);
    }
    if (lane == 0) {
        red[0][wave] = d0;
        red[1][wave] = d1;
        red[2][wave] = d2;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double sum = 0.0;
        for (int q = 0; q < NW; ++q) sum += red[threadIdx.x][q];
        partial[threadIdx.x] = sum;
    }
}

// Instance of work item b in a ragged batch: the largest i with first[i] <= b.
__device__ __forceinline__ int batch_item(const uint32_t* first, int count, uint32_t b) {
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Calls f(kind, virt, use1) with compile-time values.
template <typename F>
hipError_t by_kind(int kind, bool virt, bool use1, F&& f) {
    using std::integral_constant;
    auto rest = [&](auto k) {
        if (virt) return use1 ? f(k, std::true_type{}, std::true_type{}) : f(k, std::true_type{}, std::false_type{});
        return use1 ? f(k, std::false_type{}, std::true_type{}) : f(k, std::false_type{}, std::false_type{});
    };
    switch (kind) {
        case SK_FIRST: return rest(integral_constant<int, SK_FIRST>{});
        case SK_MIDDLE: return rest(integral_constant<int, SK_MIDDLE>{});
        case SK_BOUNDARY: return rest(integral_constant<int, SK_BOUNDARY>{});
        case SK_FINAL: return rest(integral_constant<int, SK_FINAL>{});
        case SK_P0:
            return virt ? f(integral_constant<int, SK_P0>{}, std::true_type{}, std::false_type{})
                        : f(integral_constant<int, SK_P0>{}, std::false_type{}, std::false_type{});
        default: return hipErrorInvalidValue;
    }
}

}  // namespace
}  // namespace qnae
