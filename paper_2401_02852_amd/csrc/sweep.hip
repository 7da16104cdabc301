// State sweeps: phase, mixer and readout on complex64 statevectors.
//
// The mixer U_B(beta) = prod_j exp(-i beta X_j) (Section 2.1; Appendix A.4)
// is a product of commuting one-qubit factors, so any subset of qubits can be
// applied in one pass. A sweep moves the state through the chip once: every
// workgroup owns a tile of 2^TB amplitudes whose indices vary on TB chosen bits
// of x (the lowest four among them, so global accesses run over 128 bytes at
// least), keeps it in registers and LDS, applies the phase table (the diagonal
// exp(-i gamma C(x)), Section 3.2) and the selected qubit butterflies, and
// writes it back.
//
// Each thread holds 16 amplitudes in 32 registers: 50 to 65 registers in all
// (boundary kind 60 to 85), so a CU holds 16 to 32 waves of two to four workgroups, which hide each
// other's loads, LDS transposes and barriers. (Tiles of 32 amplitudes a thread
// at two waves per SIMD: n = 17, p = 8 with cost build 147 us, n = 22 full
// state, p = 12, 269 us, n = 30 half state, p = 10, 32.9 ms; with 16 125 us, 240 us
// and 31.6 ms; tiles of 2^14 amplitudes keep 32 a thread, see sweep14.hip.)
// Layouts and transposes: tile.h.
//
// The butterfly on a pair (a, b) is own' = own - i t partner (two FMAs per
// amplitude); see MixForm for how t, the dropped X and the scalar factor
// encode R(beta) = cos(beta) I - i sin(beta) X. A layout's butterflies run as
// straight-line code over the slot bits it can mix, with t = 0 (an exact
// identity) on those the group does not.
#include <type_traits>

#include "sweep_common.h"

namespace qnae {
namespace {

template <uint32_t POSS>
__device__ __forceinline__ void mix16(float2 (&v)[16], uint32_t sm, float t) {
    if constexpr ((POSS & 1u) != 0u) bfly<16, 0>(v, (sm & 1u) ? t : 0.f);
    if constexpr ((POSS & 2u) != 0u) bfly<16, 1>(v, (sm & 2u) ? t : 0.f);
    if constexpr ((POSS & 4u) != 0u) bfly<16, 2>(v, (sm & 4u) ? t : 0.f);
    if constexpr ((POSS & 8u) != 0u) bfly<16, 3>(v, (sm & 8u) ? t : 0.f);
}

// The butterflies of layout LY on slot bits in ONLY.
template <int TB, int LY, bool USE1, uint32_t ONLY = 15u>
__device__ __forceinline__ void mix_layout(float2 (&v)[16], uint32_t m, float t) {
    mix16<s_possible<TB, LY, USE1>() & ONLY>(v, s_slots<TB, LY>(m), t);
}

// The tile from one layout to another through LDS: whole elements, or (PLANES)
// the real parts and then the imaginary parts in half the LDS.
template <int TB, int FROM, int TO, bool VIRT, bool PLANES>
__device__ __forceinline__ void move(float* lds, float2 (&v)[16], uint32_t lane, uint32_t wave) {
    constexpr bool CROSS = FROM >= 4 || TO >= 4;
    auto sync = [] {
        if (CROSS) __syncthreads();
        else wave_lds_sync();
    };
    if (FROM >= 4) __syncthreads();  // every wave has read its part of the transpose into layout 4
    if constexpr (PLANES) {
        to_s_plane<TB, FROM, VIRT, 0>(lds, v, lane, wave);
        sync();
        from_s_plane<TB, TO, VIRT, 0>(lds, v, lane, wave);
        sync();
        to_s_plane<TB, FROM, VIRT, 1>(lds, v, lane, wave);
        sync();
        from_s_plane<TB, TO, VIRT, 1>(lds, v, lane, wave);
    } else {
        to_s<TB, FROM, VIRT>((float2*)lds, v, lane, wave);
        sync();
        from_s<TB, TO, VIRT>((const float2*)lds, v, lane, wave);
    }
    if (!CROSS) wave_lds_sync();
}

// The layout between a group's two mixings, of the phase and the readout.
template <int TB, bool USE1>
constexpr int kInner = USE1 ? 4 : 5;

// One group's mixing from layout 0 to kInner, or from kInner to layout 1. The
// order of the qubits is the same in both and for every kind of tile:
// e0, e7..10, e1..5, e6, e11.. (e4, e5 last where layouts 2 and 3 are skipped),
// respectively e6, e11.. (e4, e5), e1..5, e0, e7..10.
template <int TB, bool USE1, bool VIRT, bool PLANES>
__device__ __forceinline__ void mix_down(float* lds, float2 (&v)[16], uint32_t m, float t, uint32_t lane,
                                         uint32_t wave) {
    mix_layout<TB, 0, USE1>(v, m, t);
    s_swap(v);
    mix_layout<TB, 1, USE1>(v, m, t);
    if constexpr (USE1) {
        move<TB, 1, 2, VIRT, PLANES>(lds, v, lane, wave);
        mix_layout<TB, 2, USE1>(v, m, t);
        s_swap(v);
        mix_layout<TB, 3, USE1>(v, m, t);
        move<TB, 3, 4, VIRT, PLANES>(lds, v, lane, wave);
    } else {
        move<TB, 1, 4, VIRT, PLANES>(lds, v, lane, wave);
    }
    mix_layout<TB, 4, USE1>(v, m, t);
    if constexpr (kInner<TB, USE1> == 5) {
        s_swap(v);
        mix_layout<TB, 5, USE1>(v, m, t);
    }
}
template <int TB, bool USE1, bool VIRT, bool PLANES>
__device__ __forceinline__ void mix_up(float* lds, float2 (&v)[16], uint32_t m, float t, uint32_t lane,
                                       uint32_t wave) {
    if constexpr (kInner<TB, USE1> == 4) {
        mix_layout<TB, 4, USE1>(v, m, t);
    } else {
        mix_layout<TB, 4, USE1, 7u>(v, m, t);  // slot bits 0..2 are those of layout 5
        s_swap(v);
        mix_layout<TB, 4, USE1, 8u>(v, m, t);
        s_swap(v);
        mix_layout<TB, 5, USE1>(v, m, t);
    }
    if constexpr (USE1) {
        move<TB, 4, 2, VIRT, PLANES>(lds, v, lane, wave);
        mix_layout<TB, 2, USE1>(v, m, t);
        s_swap(v);
        mix_layout<TB, 3, USE1>(v, m, t);
        move<TB, 3, 0, VIRT, PLANES>(lds, v, lane, wave);
    } else {
        move<TB, kInner<TB, USE1>, 0, VIRT, PLANES>(lds, v, lane, wave);
    }
    mix_layout<TB, 0, USE1>(v, m, t);
    s_swap(v);
    mix_layout<TB, 1, USE1>(v, m, t);
}

// Transposes through component planes (half the LDS, twice the workgroups in a
// CU) in the kinds that move state one way, never in the boundary kind (n = 30
// half state 31.9 -> 32.4 ms with it, n = 20 114 -> 118 us), and in the middle kind
// while the state fits the last-level cache: up to 2^24 amplitudes (n = 23 half
// state 323 -> 316 us, n = 24 632 -> 613 us with three groups; 2^26: 3.90 -> 3.92 ms
// per run, 2^29: 31.9 -> 32.2 ms).
constexpr bool sweep_planes(int kind, bool small) { return kind == SK_FIRST || kind == SK_FINAL || (kind == SK_MIDDLE && small); }
// Waves per SIMD a kernel is register-allocated for: what the LDS admits.
constexpr int sweep_waves(int kind, bool small) { return sweep_planes(kind, small) ? 8 : 4; }

// One workgroup's work on tile t of one sweep. Readout kinds write the three
// block sums to partial[0..2]. VIRT: a half-state sweep whose group mixes bit
// n-1, which is the tile's top bit (a group's bits ascend); the elements with it
// set are stored at mir - y for the index y of their other bits. Half-state
// sweeps of other groups are whole-state sweeps over n-1 bits.
template <int TB, typename CT, int KIND, bool VIRT, bool CKPT, bool USE1, bool SMALL>
__device__ __forceinline__ void sweep_tile(const SweepArgs& a, uint32_t t, double* partial) {
    constexpr int NT = kSweepThreads<TB>, WB = TB - 10;
    constexpr bool INIT = KIND == SK_FIRST || KIND == SK_P0;
    constexpr bool PHASE = KIND == SK_BOUNDARY;
    constexpr bool REDUCE = KIND == SK_FINAL || KIND == SK_P0;
    constexpr bool COST3 = PHASE || REDUCE;  // costs of the inner layout's elements
    constexpr bool NEED_LUT = INIT || PHASE;
    constexpr bool LUT_LDS = sizeof(CT) == 1;
    constexpr int PK = 4 / (int)sizeof(CT);
    constexpr int NC = COST3 ? 16 / PK : 1;
    constexpr bool PLANES = sweep_planes(KIND, SMALL);
    __shared__ __align__(16) float lds[KIND == SK_P0 ? 1 : s_lds_floats<TB, PLANES>()];
    __shared__ float2 lut_s[NEED_LUT && LUT_LDS ? 256 : 1];
    __shared__ double red[3][1 << WB];

    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = VIRT ? (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : threadIdx.x >> 6;
    constexpr uint32_t kTop = 1u << (TB - 1);
    uint64_t bitval[TB];
#pragma unroll
    for (int i = 0; i < TB; ++i) bitval[i] = 1ull << a.pos[i];
    auto scat = [&](uint32_t e) -> uint64_t {
        uint64_t x = 0;
#pragma unroll
        for (int i = 0; i < (VIRT ? TB - 1 : TB); ++i)
            if ((e >> i) & 1u) x |= bitval[i];
        return x;
    };
    const uint64_t base = tile_base<KIND>(a, t);
    // Layouts 0 and 1 hold the top tile bit in the wave index: a mirrored wave's
    // elements, in storage order, start where the tile's mirror image does.
    const uint64_t base0 = VIRT && (wave >> (WB - 1)) != 0u ? a.mir - base - a.tile_bits : base;
    // Index of the element in slot j of the inner layout: o3 + off3(j), or
    // mirrored (up3) mir - o3 - off3(j).
    constexpr int IN = kInner<TB, USE1>;
    const uint64_t o3 = base + scat(st<TB, IN>(lane, wave));
    auto up3 = [](int j) -> bool { return VIRT && (ss<TB, IN>(j) & kTop) != 0u; };
    auto off3 = [&](int j) -> uint64_t { return scat(ss<TB, IN>(j)); };
    auto at3 = [&](int j) -> uint64_t { return up3(j) ? a.mir - o3 - off3(j) : o3 + off3(j); };

    // What the tile reads goes out together, before any of it is waited for: the
    // table, the costs, the state. (With the costs packed before the state was asked for,
    // the compiler made a chain of two costs at a time of them in the final kind
    // and with 16-bit costs: whole state, n = 30, one layer 6.76 -> 6.36 ms, ten with 16-bit
    // costs 73.5 -> 65.4, half state 37.5 -> 33.2.)
    static_assert(!LUT_LDS || NT >= 256, "a table entry per thread");
    float2 entry = make_float2(0.f, 0.f);
    if (NEED_LUT && LUT_LDS && (int)threadIdx.x < a.lut_len) entry = a.lut[threadIdx.x];
    CT raw[COST3 ? 16 : 1];
    if (COST3) {
        // with cflip (never on a half state) the costs are read at the complemented index
        const uint64_t all = (1ull << a.n) - 1ull;
        const bool cf = !VIRT && a.cflip != 0;
        const CT* const c3 = (const CT*)a.cost + (cf ? o3 ^ all : o3);
        const CT* const cv = VIRT ? (const CT*)a.cost + (a.mir - o3) : c3;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int64_t d = (int64_t)off3(j);
            raw[j] = up3(j) ? cv[-d] : c3[cf ? -d : d];
        }
    }
    float2 v[16];
    if (!INIT) {
        const float2* const p0 = a.psi_in + base0 + scat(st<TB, 0>(lane, wave));
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            const float4 q = ld_state(p0 + scat(ss<TB, 0>(2 * jj)));
            v[2 * jj] = make_float2(q.x, q.y);
            v[2 * jj + 1] = make_float2(q.z, q.w);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (NEED_LUT && LUT_LDS && (int)threadIdx.x < a.lut_len) lut_s[threadIdx.x] = entry;
    uint32_t cvp[NC];
    if (COST3) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            uint32_t wv = 0u;
#pragma unroll
            for (int q = 0; q < PK; ++q) wv |= (uint32_t)raw[PK * i + q] << (8 * sizeof(CT) * q);
            cvp[i] = wv;
        }
        // packed as they arrive, with the state loads still in flight
#pragma unroll
        for (int i = 0; i < NC; ++i) asm volatile("" : "+v"(cvp[i]));
    }
    // Cost values above m are a caller error; the clamp keeps table reads in bounds.
    const uint32_t lut_last = (uint32_t)a.lut_len - 1u;
    auto lut = [&](uint32_t c) -> float2 { return LUT_LDS ? lut_s[c] : a.lut[min(c, lut_last)]; };
    auto cval = [&](int j) -> uint32_t {
        return (cvp[j / PK] >> (8 * sizeof(CT) * (j % PK))) & (sizeof(CT) == 1 ? 0xffu : 0xffffu);
    };

    if (KIND == SK_FIRST) {
        // adjacent costs of a slot pair along tile bit 0; 64 lanes cover 128
        using PT = typename std::conditional<sizeof(CT) == 1, uint16_t, uint32_t>::type;
        constexpr uint32_t CB = 8 * sizeof(CT);
        const CT* const c0 = (const CT*)a.cost + base0 + scat(st<TB, 0>(lane, wave));
        PT cp[8];
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) cp[jj] = *(const PT*)(c0 + scat(ss<TB, 0>(2 * jj)));
        __syncthreads();  // phase table visible
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            v[2 * jj] = lut((uint32_t)cp[jj] & ((1u << CB) - 1u));
            v[2 * jj + 1] = lut((uint32_t)cp[jj] >> CB);
        }
        mix_down<TB, USE1, VIRT, PLANES>(lds, v, a.post_mask, a.post_t, lane, wave);
    } else if (KIND == SK_P0) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = lut(cval(j));
    } else {
        mix_down<TB, USE1, VIRT, PLANES>(lds, v, a.pre_mask, a.pre_t, lane, wave);
    }
    if (CKPT) {
        // (t | s) ^ (2^n - 1) = (t ^ (2^n - 1)) - s for disjoint t and s
        const uint64_t all = (1ull << a.n) - 1ull;
        const float2 f = a.ckpt_scale;
        if (!VIRT && a.cflip) {
#pragma unroll
            for (int j = 0; j < 16; ++j) st_state(a.ckpt + (o3 ^ all) - off3(j), cmul(v[j], f));
        } else {
#pragma unroll
            for (int j = 0; j < 16; ++j) st_state(a.ckpt + at3(j), cmul(v[j], f));
        }
    }
    if (PHASE) {
        if constexpr (LUT_LDS) {
#pragma unroll
            for (int j = 0; j < 16; ++j) v[j] = cmul(v[j], lut(cval(j)));
        } else {
            // eight reads of the table in memory at a time: left alone they are a chain of 16
#pragma unroll
            for (int h = 0; h < 16; h += 8) {
                float2 e[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) e[j] = lut(cval(h + j));
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 8; ++j) v[h + j] = cmul(v[h + j], e[j]);
            }
        }
        mix_up<TB, USE1, VIRT, PLANES>(lds, v, a.post_mask, a.post_t, lane, wave);
        float2* const p0 = a.psi + base0 + scat(st<TB, 1>(lane, wave));
#pragma unroll
        for (int jj = 0; jj < 8; ++jj)
            st_state(p0 + scat(ss<TB, 1>(2 * jj)),
                     make_float4(v[2 * jj].x, v[2 * jj].y, v[2 * jj + 1].x, v[2 * jj + 1].y));
        return;
    }
    if (REDUCE) {
        readout<16, SLay<TB>::top_slot, 1 << WB>(v, cval, red, partial, lane, wave);
        if (!a.store) return;
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = cmul(v[j], a.store_scale);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) st_state(a.psi + at3(j), v[j]);
    // Whole-state output of a half-state run: the upper half mirrors the lower one.
    if (KIND == SK_FINAL && a.expand) {
        const uint64_t all = (1ull << a.n) - 1ull;
#pragma unroll
        for (int j = 0; j < 16; ++j) st_state(a.psi + (all - at3(j)), v[j]);
    }
}

// One sweep over one state: block b handles tile b.
template <int TB, typename CT, int KIND, bool VIRT, bool CKPT, bool USE1, bool SMALL>
__global__ __launch_bounds__(kSweepThreads<TB>) __attribute__((amdgpu_waves_per_eu(sweep_waves(KIND, SMALL)))) void sweep_kernel(
    const SweepArgs a) {
    sweep_tile<TB, CT, KIND, VIRT, CKPT, USE1, SMALL>(a, blockIdx.x, a.partials + 3 * (size_t)blockIdx.x);
}

// One sweep step over many states at once (ragged): instance i owns blocks
// first[i] .. first[i+1]-1, one per tile, with its own arguments.
template <int TB, typename CT, int KIND, bool VIRT, bool USE1>
__global__ __launch_bounds__(kSweepThreads<TB>) __attribute__((amdgpu_waves_per_eu(sweep_waves(KIND, true)))) void sweep_batch_kernel(
    const SweepArgs* args, const uint32_t* first, int count) {
    const int i = batch_item(first, count, blockIdx.x);
    const SweepArgs a = args[i];
    const uint32_t t = blockIdx.x - first[i];
    sweep_tile<TB, CT, KIND, VIRT, false, USE1, true>(a, t, a.partials + 3 * (size_t)t);
}

// psi[x] <-> psi[N - 1 - x]: undoes an X on every qubit (N >= 4).
__global__ __launch_bounds__(256) void reverse_kernel(float2* psi, uint64_t N) {
    const uint64_t i = ((uint64_t)blockIdx.x * 256 + threadIdx.x) * 2;
    if (i >= N / 2) return;
    float4* lo = (float4*)(psi + i);
    float4* hi = (float4*)(psi + (N - 2 - i));
    const float4 a = *lo, b = *hi;
    *lo = make_float4(b.z, b.w, b.x, b.y);
    *hi = make_float4(a.z, a.w, a.x, a.y);
}

__device__ __forceinline__ void final_reduce_body(const double* partials, int64_t blocks, double* out) {
    __shared__ double red[3][16];
    double t0 = 0.0, t1 = 0.0, t2 = 0.0;
    for (int64_t i = threadIdx.x; i < blocks; i += 1024) {
        t0 += partials[3 * i];
        t1 += partials[3 * i + 1];
        t2 += partials[3 * i + 2];
    }
    for (int off = 32; off > 0; off >>= 1) {
        t0 += __shfl_xor(t0, off);
        t1 += __shfl_xor(t1, off);
        t2 += __shfl_xor(t2, off);
    }
    if ((threadIdx.x & 63u) == 0) {
        red[0][threadIdx.x >> 6] = t0;
        red[1][threadIdx.x >> 6] = t1;
        red[2][threadIdx.x >> 6] = t2;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double t = 0.0;
        for (int q = 0; q < 16; ++q) t += red[threadIdx.x][q];
        out[threadIdx.x] = t;
    }
}

__global__ __launch_bounds__(1024) void final_reduce_kernel(const double* partials, int64_t blocks, double* out) {
    final_reduce_body(partials, blocks, out);
}

// One workgroup per row of `blocks` triples.
__global__ __launch_bounds__(1024) void final_reduce_rows_kernel(const double* partials, int64_t blocks, double* out) {
    final_reduce_body(partials + 3 * blocks * blockIdx.x, blocks, out + 3 * (size_t)blockIdx.x);
}

// One workgroup per instance i: blocks[i] triples at partials[i] -> outs[i].
__global__ __launch_bounds__(1024) void final_reduce_batch_kernel(const double* const* partials, const uint32_t* blocks,
                                                                   double* const* outs) {
    final_reduce_body(partials[blockIdx.x], blocks[blockIdx.x], outs[blockIdx.x]);
}

template <int TB, typename CT>
hipError_t launch_tb(int kind, const SweepArgs& a, bool ckpt, hipStream_t s) {
    const dim3 grid(1u << a.nw), block(kSweepThreads<TB>);
    const bool virt = a.half && a.vbit >= 0;
    return by_kind(kind, virt, sweep_l1(TB, kind, a.pre_mask, a.post_mask) == 1, [&](auto k, auto vi, auto u) {
        if constexpr (k.value == SK_BOUNDARY && TB == kAdjointTileBits) {
            if (ckpt) {
                hipLaunchKernelGGL((sweep_kernel<TB, CT, SK_BOUNDARY, vi.value, true, u.value, false>), grid, block, 0,
                                   s, a);
                return hipGetLastError();
            }
        }
        if (ckpt) return hipErrorInvalidValue;
        if constexpr (k.value == SK_MIDDLE) {
            if (a.nw + TB <= 24) {
                hipLaunchKernelGGL((sweep_kernel<TB, CT, SK_MIDDLE, vi.value, false, u.value, true>), grid, block, 0, s,
                                   a);
                return hipGetLastError();
            }
        }
        hipLaunchKernelGGL((sweep_kernel<TB, CT, k.value, vi.value, false, u.value, false>), grid, block, 0, s, a);
        return hipGetLastError();
    });
}

template <int TB, typename CT>
hipError_t launch_batch_tb(int kind, const SweepArgs* args, const uint32_t* first, int count, uint32_t blocks, bool virt,
                          int l1, LaunchTo to) {
    return by_kind(kind, virt, l1 != 2, [&](auto k, auto vi, auto u) {
        return launch_to(to, dim3(blocks), dim3(kSweepThreads<TB>),
                         sweep_batch_kernel<TB, CT, k.value, vi.value, u.value>, args, first, count);
    });
}

}  // namespace

int sweep_l1(int tb, int kind, uint32_t pre_mask, uint32_t post_mask) {
    const bool pre = kind == SK_MIDDLE || kind == SK_BOUNDARY || kind == SK_FINAL;
    const bool post = kind == SK_FIRST || kind == SK_BOUNDARY;
    return (((pre ? pre_mask : 0u) | (post ? post_mask : 0u)) & (tb == 14 ? 0x3eu : low_bits)) != 0u ? 1 : 2;
}

hipError_t launch_sweep(int tb, int dtype, int kind, const SweepArgs& a, hipStream_t s) {
    switch (tb) {
        case 12: return dtype == 1 ? launch_tb<12, uint8_t>(kind, a, false, s) : launch_tb<12, uint16_t>(kind, a, false, s);
        case 13: return dtype == 1 ? launch_tb<13, uint8_t>(kind, a, false, s) : launch_tb<13, uint16_t>(kind, a, false, s);
        case 14: return launch_sweep14(dtype, kind, a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_sweep_ckpt(int dtype, const SweepArgs& a, hipStream_t s) {
    if (!a.ckpt || a.nw < 0) return hipErrorInvalidValue;
    constexpr int TB = kAdjointTileBits;
    return dtype == 1 ? launch_tb<TB, uint8_t>(SK_BOUNDARY, a, true, s) : launch_tb<TB, uint16_t>(SK_BOUNDARY, a, true, s);
}

hipError_t launch_sweep_batch(int tb, int dtype, int kind, const SweepArgs* args, const uint32_t* first, int count,
                              uint32_t blocks, LaunchTo to, bool virt, int l1) {
    auto run = [&](auto tbits) {
        return dtype == 1 ? launch_batch_tb<tbits.value, uint8_t>(kind, args, first, count, blocks, virt, l1, to)
                          : launch_batch_tb<tbits.value, uint16_t>(kind, args, first, count, blocks, virt, l1, to);
    };
    switch (tb) {
        case 12: return run(std::integral_constant<int, 12>{});
        case 13: return run(std::integral_constant<int, 13>{});
        case 14: return launch_sweep14_batch(dtype, kind, args, first, count, blocks, to, virt, l1);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_reverse(float2* psi, uint64_t N, LaunchTo to) {
    const uint64_t threads = N / 4;
    return launch_to(to, dim3((uint32_t)((threads + 255) / 256)), dim3(256), reverse_kernel, psi, N);
}

hipError_t launch_final_reduce(const double* partials, int64_t blocks, double* out, hipStream_t s) {
    hipLaunchKernelGGL(final_reduce_kernel, dim3(1), dim3(1024), 0, s, partials, blocks, out);
    return hipGetLastError();
}

hipError_t launch_final_reduce_rows(const double* partials, int64_t blocks, double* out, int count, hipStream_t s) {
    hipLaunchKernelGGL(final_reduce_rows_kernel, dim3((uint32_t)count), dim3(1024), 0, s, partials, blocks, out);
    return hipGetLastError();
}

hipError_t launch_final_reduce_batch(const double* const* partials, const uint32_t* blocks, double* const* outs,
                                     int count, LaunchTo to) {
    return launch_to(to, dim3(count), dim3(1024), final_reduce_batch_kernel, partials, blocks, outs);
}

}  // namespace qnae
