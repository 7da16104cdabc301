// State sweeps on tiles of 2^14 amplitudes (see sweep.hip for the method): 512
// threads of 32 amplitudes, all transposes through component planes, two
// workgroups to a CU. 16 amplitudes a thread (1024 threads), which the smaller
// tiles use, measured slower here: n = 24, p = 10 382 -> 412 us on the half state
// and 652 -> 716 us on the whole one, n = 33, p = 4 105 -> 111 ms (a workgroup
// of 16 waves waits for all of them at each of seven barriers).
#include "sweep_common.h"

namespace qnae {
namespace {

// Layouts of 2^14-element tiles, 32 elements a thread (512 threads): element e
// splits into a thread part and a slot part (5 bits)
//   L0  slots e{0, 7, 8, 9, 10}, lanes e{1..6},        waves e{11..13}  (16-byte global accesses)
//   L1  slots e{1..5},           lanes e{0, 6..10},    waves e{11..13}
//   L2  slots e{6, 11, 12, 13, 7}, lanes e{0..5},      waves e{8, 9, 10} (phase, readout)
// L0 mixes e{0, 7..10}, L1 e{1..5}, L2 e{6, 11, 12, 13}; groups that mix none of
// e{1..5} skip L1. VIRT as in tile.h: L2 takes the elements with the top tile bit
// by their true position.
constexpr int TB = 14, WB = 3, NT = 512;
__device__ __forceinline__ uint32_t t0(uint32_t lane, uint32_t wave) { return (lane << 1) | (wave << 11); }
__device__ __forceinline__ constexpr uint32_t s0(int j) { return (uint32_t)(j & 1) | ((uint32_t)(j >> 1) << 7); }
__device__ __forceinline__ uint32_t t1(uint32_t lane, uint32_t wave) {
    return (lane & 1u) | ((lane >> 1) << 6) | (wave << 11);
}
__device__ __forceinline__ constexpr uint32_t s1(int j) { return (uint32_t)j << 1; }
__device__ __forceinline__ uint32_t t2(uint32_t lane, uint32_t wave) { return lane | (wave << 8); }
__device__ __forceinline__ constexpr uint32_t s2(int j) {
    constexpr int slot[5] = {6, 11, 12, 13, 7};
    uint32_t e = 0u;
    for (int i = 0; i < 5; ++i) e |= (uint32_t)((j >> i) & 1) << slot[i];
    return e;
}
constexpr uint32_t kTop = 1u << (TB - 1);
constexpr int kTopSlot = 3;
// Slot masks of the tile bits each layout mixes.
__device__ __forceinline__ uint32_t sm0(uint32_t m) { return (m & 1u) | (((m >> 7) & 15u) << 1); }
__device__ __forceinline__ uint32_t sm1(uint32_t m) { return (m >> 1) & 31u; }
__device__ __forceinline__ uint32_t sm2(uint32_t m) { return ((m >> 6) & 1u) | ((m >> 10) & 0xeu); }

// Butterflies on the slot bits in sm, t = 0 (an exact identity) on the others:
// straight-line code lets the compiler rename registers.
__device__ __forceinline__ void mix32(float2 (&v)[32], uint32_t sm, float t) {
    bfly<32, 0>(v, (sm & 1u) ? t : 0.f);
    bfly<32, 1>(v, (sm & 2u) ? t : 0.f);
    bfly<32, 2>(v, (sm & 4u) ? t : 0.f);
    bfly<32, 3>(v, (sm & 8u) ? t : 0.f);
    bfly<32, 4>(v, (sm & 16u) ? t : 0.f);
}

// Component planes: the real parts of a tile go through LDS first, then the
// imaginary parts (66 KiB, two workgroups to a CU; whole elements fit one).
// Element e sits at e + sum of c_i over its set bits i >= 6, non-decreasing sums
// chosen so that b32 accesses of 32 lanes in L1 and L2 and b64 accesses in L0
// hit 32 distinct banks.
__device__ __forceinline__ constexpr uint32_t place(uint32_t e) {
    constexpr uint32_t c[8] = {2, 4, 8, 16, 32, 64, 128, 256};
    uint32_t p = e;
    for (int i = 0; i < 8; ++i) p += ((e >> (6 + i)) & 1u) * c[i];
    return p;
}
constexpr uint32_t kPlaneFloats = (1u << TB) + 512u;
static_assert(place((1u << TB) - 1u) < kPlaneFloats, "a plane fits");

template <int LY, bool VIRT, typename F>
__device__ __forceinline__ void places(uint32_t lane, uint32_t wave, F&& f) {
    const uint32_t t = LY == 0 ? t0(lane, wave) : LY == 1 ? t1(lane, wave) : t2(lane, wave);
    constexpr uint32_t slots = s2(31) & ~kTop, threads = ((1u << TB) - 1u) & ~s2(31);
    const uint32_t b = place(t), bc = VIRT && LY == 2 ? place(kTop | (threads ^ t)) : b;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        const uint32_t se = LY == 0 ? s0(j) : LY == 1 ? s1(j) : s2(j);
        if (VIRT && LY == 2 && (se & kTop)) f(j, bc + place(slots ^ (se & ~kTop)));
        else f(j, b + place(se));
    }
}

// The tile from layout A to layout B. CROSS: the layouts differ in the wave
// index (workgroup barriers); otherwise each wave stays inside its own part. The
// caller orders this against earlier LDS reads of the buffer by other waves.
template <int A, int B, bool CROSS, bool VIRT>
__device__ __forceinline__ void move(float* lds, float2 (&v)[32], uint32_t lane, uint32_t wave) {
    auto sync = [] {
        if (CROSS) __syncthreads();
        else wave_lds_sync();
    };
    places<A, VIRT>(lane, wave, [&](int j, uint32_t at) { lds[at] = v[j].x; });
    sync();
    places<B, VIRT>(lane, wave, [&](int j, uint32_t at) { v[j].x = lds[at]; });
    sync();
    places<A, VIRT>(lane, wave, [&](int j, uint32_t at) { lds[at] = v[j].y; });
    sync();
    places<B, VIRT>(lane, wave, [&](int j, uint32_t at) { v[j].y = lds[at]; });
}

// Waves per SIMD a kernel is register-allocated for (128 registers: the two
// workgroups that the LDS admits).
constexpr int waves(int kind) { return kind == SK_BOUNDARY || kind == SK_FINAL ? 4 : 1; }

// One workgroup's work on tile t of one sweep. Readout kinds write the three
// block sums to partial[0..2]. USE1: the tiles pass through layout L1, fixed per
// launch (a branch around the transposes raises the register demand: 21 spilled
// dwords a lane in the boundary kind instead of 3).
// VIRT: a half-state sweep whose group mixes bit n-1, which is the tile's top
// bit (a group's bits ascend); the elements with it set are stored at mir - y
// for the index y of their other bits. Half-state sweeps of other groups are
// whole-state sweeps over n-1 bits.
template <typename CT, int KIND, bool VIRT, bool USE1>
__device__ __forceinline__ void sweep_tile(const SweepArgs& a, uint32_t t, double* partial) {
    constexpr bool INIT = KIND == SK_FIRST || KIND == SK_P0;  // start from phase table 0
    constexpr bool PRE = KIND == SK_MIDDLE || KIND == SK_BOUNDARY || KIND == SK_FINAL;
    constexpr bool PHASE = KIND == SK_BOUNDARY;
    constexpr bool POST = KIND == SK_FIRST || KIND == SK_BOUNDARY;
    constexpr bool REDUCE = KIND == SK_FINAL || KIND == SK_P0;
    constexpr bool NEED_COST = INIT || PHASE || REDUCE;
    constexpr bool NEED_LUT = INIT || PHASE;
    constexpr bool LUT_LDS = sizeof(CT) == 1;
    constexpr int PK = 4 / (int)sizeof(CT);  // cost values per packed register
    constexpr int NC = NEED_COST ? 32 / PK : 1;
    __shared__ __align__(16) float lds[KIND == SK_P0 ? 1 : kPlaneFloats];
    __shared__ float2 lut_s[NEED_LUT && LUT_LDS ? 256 : 1];
    __shared__ double red[3][1 << WB];

    const uint32_t lane = threadIdx.x & 63u;
    // (uniform: a mirrored wave's place is a scalar choice)
    const uint32_t wave = VIRT ? (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : threadIdx.x >> 6;
    // Tile bit i sits at bit pos[i] of x; the tile index fills the other
    // bits (wmask, ascending). Both maps are bit deposits, so offsets are
    // additive (XOR-linear) over disjoint bit sets of e: an address splits
    // into a per-thread offset and a per-slot offset that is the same for
    // every lane (scalar registers).
    // VIRT: the top tile bit contributes no offset.
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
    // Layout L0 holds the top tile bit in the wave index: a mirrored wave's
    // elements, in storage order, start where the tile's mirror image does.
    const uint64_t base0 = VIRT && (wave >> (WB - 1)) != 0u ? a.mir - base - a.tile_bits : base;

    // Cost values of the 32 amplitudes in layout L2, loaded first; packed 4
    // (uint8) or 2 (uint16) per register. With cflip the stored state is the
    // true one with every qubit flipped (see MixForm), so cost values are read
    // at the complemented index: complemented tile base, thread part and slot.
    uint32_t cvp[NC];
    if (NEED_COST && VIRT && KIND != SK_FIRST) {
        // symmetric cost: no complemented reads, mirrored places instead
        const uint64_t fwd = base + scat(t2(lane, wave));
        const CT* const cf = (const CT*)a.cost + fwd;
        const CT* const cv = (const CT*)a.cost + (a.mir - fwd);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            uint32_t wv = 0u;
#pragma unroll
            for (int q = 0; q < PK; ++q) {
                const uint32_t se = s2(PK * i + q);
                const int64_t so = (int64_t)scat(se);
                wv |= (uint32_t)((se & kTop) ? cv[-so] : cf[so]) << (8 * sizeof(CT) * q);
            }
            cvp[i] = wv;
        }
#pragma unroll
        for (int i = 0; i < NC; ++i) asm volatile("" : "+v"(cvp[i]));  // packed as they arrive
        if (NEED_LUT && LUT_LDS)
            for (int i = threadIdx.x; i < a.lut_len; i += NT) lut_s[i] = a.lut[i];
    } else if (NEED_COST && KIND != SK_FIRST) {
        const bool cf = a.cflip != 0;
        const uint64_t cbase = cf ? base ^ ((((uint64_t)1 << a.n) - 1ull) ^ a.tile_bits) : base;
        const uint32_t ct = cf ? t2(lane, wave) ^ t2(63u, (1u << WB) - 1u) : t2(lane, wave);
        const int cj = cf ? 31 : 0;
        const CT* const c2 = (const CT*)a.cost + cbase + scat(ct);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            uint32_t wv = 0u;
#pragma unroll
            for (int q = 0; q < PK; ++q) wv |= (uint32_t)c2[scat(s2((PK * i + q) ^ cj))] << (8 * sizeof(CT) * q);
            cvp[i] = wv;
        }
#pragma unroll
        for (int i = 0; i < NC; ++i) asm volatile("" : "+v"(cvp[i]));  // packed as they arrive
        if (NEED_LUT && LUT_LDS)
            for (int i = threadIdx.x; i < a.lut_len; i += NT) lut_s[i] = a.lut[i];
    }
    // Cost values above m are a caller error; the clamp keeps table reads in bounds.
    const uint32_t lut_last = (uint32_t)a.lut_len - 1u;
    auto lut = [&](uint32_t cidx) -> float2 { return LUT_LDS ? lut_s[cidx] : a.lut[min(cidx, lut_last)]; };
    auto cval = [&](int j) -> uint32_t {
        return (cvp[j / PK] >> (8 * sizeof(CT) * (j % PK))) & (sizeof(CT) == 1 ? 0xffu : 0xffffu);
    };

    // The tile from layout L2 to the state.
    auto store2 = [&](const float2(&x)[32]) {
        const uint64_t fwd = base + scat(t2(lane, wave));
        float2* const pf = a.psi + fwd;
        float2* const pv = VIRT ? a.psi + (a.mir - fwd) : pf;
#pragma unroll
        for (int j = 0; j < 32; ++j) {
            const uint32_t se = s2(j);
            const uint64_t so = scat(se);
            st_state(VIRT && (se & kTop) ? pv - so : pf + so, x[j]);
        }
    };
    if (KIND == SK_FIRST) {
        // In layout L0 the pair of a thread's slots along tile bit 0 are
        // adjacent costs, and the 64 lanes cover tile bits 1..6, so a wave
        // reads 128 consecutive cost bytes per load (layout L2 reads four
        // runs of 16). The tile is then mixed in L0, L1, L2 and stored from
        // L2; the order of the mixings within a layer does not matter.
        using PT = typename std::conditional<sizeof(CT) == 1, uint16_t, uint32_t>::type;
        PT cp[16];
        const CT* const c0 = (const CT*)a.cost + base0 + scat(t0(lane, wave));
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) cp[jj] = *(const PT*)(c0 + scat(s0(2 * jj)));
        if (LUT_LDS)
            for (int i = threadIdx.x; i < a.lut_len; i += NT) lut_s[i] = a.lut[i];
        __syncthreads();  // phase table visible
        constexpr uint32_t CB = 8 * sizeof(CT);
        float2 v[32];
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) {
            v[2 * jj] = lut((uint32_t)cp[jj] & ((1u << CB) - 1u));
            v[2 * jj + 1] = lut((uint32_t)cp[jj] >> CB);
        }
        const uint32_t m = a.post_mask;
        const float tt = a.post_t;
        mix32(v, sm0(m), tt);
        if (USE1) {
            move<0, 1, false, VIRT>(lds, v, lane, wave);  // inside the wave's quarter
            mix32(v, sm1(m), tt);
            wave_lds_sync();
            move<1, 2, true, VIRT>(lds, v, lane, wave);
        } else {
            move<0, 2, true, VIRT>(lds, v, lane, wave);
        }
        mix32(v, sm2(m), tt);
        store2(v);
        return;
    }

    float2 v[32];
    if (INIT) {
        __syncthreads();  // phase table visible
#pragma unroll
        for (int j = 0; j < 32; ++j) v[j] = lut(cval(j));
    } else {
        const float2* const p0 = a.psi_in + base0 + scat(t0(lane, wave));
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) {
            const float4 q = ld_state(p0 + scat(s0(2 * jj)));
            v[2 * jj] = make_float2(q.x, q.y);
            v[2 * jj + 1] = make_float2(q.z, q.w);
        }
    }
    if (PRE) {
        const uint32_t m = a.pre_mask;
        const float tt = a.pre_t;
        mix32(v, sm0(m), tt);
        if (USE1) {
            move<0, 1, false, VIRT>(lds, v, lane, wave);  // inside the wave's quarter
            mix32(v, sm1(m), tt);
            wave_lds_sync();
            move<1, 2, true, VIRT>(lds, v, lane, wave);
        } else {
            move<0, 2, true, VIRT>(lds, v, lane, wave);
        }
        mix32(v, sm2(m), tt);
    }
    if (PHASE) {
#pragma unroll
        for (int j = 0; j < 32; ++j) v[j] = cmul(v[j], lut(cval(j)));
    }
    if (POST) {
        const uint32_t m = a.post_mask;
        const float tt = a.post_t;
        mix32(v, sm2(m), tt);
        if (PRE) __syncthreads();  // every wave has read its L2 part
        if (USE1) {
            move<2, 1, true, VIRT>(lds, v, lane, wave);
            mix32(v, sm1(m), tt);
            wave_lds_sync();
            move<1, 0, false, VIRT>(lds, v, lane, wave);  // inside the wave's quarter
        } else {
            move<2, 0, true, VIRT>(lds, v, lane, wave);
        }
        mix32(v, sm0(m), tt);
        float2* const p0 = a.psi + base0 + scat(t0(lane, wave));
#pragma unroll
        for (int jj = 0; jj < 16; ++jj)
            st_state(p0 + scat(s0(2 * jj)), make_float4(v[2 * jj].x, v[2 * jj].y, v[2 * jj + 1].x, v[2 * jj + 1].y));
        return;
    }
    if (REDUCE) {
        readout<32, kTopSlot, 1 << WB>(v, cval, red, partial, lane, wave);
    }
    if (KIND == SK_MIDDLE || (REDUCE && a.store)) {
        if (REDUCE) {
#pragma unroll
            for (int j = 0; j < 32; ++j) v[j] = cmul(v[j], a.store_scale);
        }
        store2(v);
        // Whole-state output of a half-state run: the upper half mirrors the
        // lower one.
        if (KIND == SK_FINAL && a.expand) {
            const uint64_t all = (1ull << a.n) - 1ull;
            const uint64_t fwd = base + scat(t2(lane, wave));
            float2* const pf = a.psi + (all - fwd);
            float2* const pv = VIRT ? a.psi + (all - a.mir + fwd) : pf;
#pragma unroll
            for (int j = 0; j < 32; ++j) {
                const uint32_t se = s2(j);
                const uint64_t so = scat(se);
                st_state(VIRT && (se & kTop) ? pv + so : pf - so, v[j]);
            }
        }
    }
}

// One sweep over one state: block b handles tile b.
template <typename CT, int KIND, bool VIRT, bool USE1>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(waves(KIND)))) void sweep14_kernel(
    const SweepArgs a) {
    sweep_tile<CT, KIND, VIRT, USE1>(a, blockIdx.x, a.partials + 3 * (size_t)blockIdx.x);
}

// One sweep step over many states at once (ragged): instance i owns blocks
// first[i] .. first[i+1]-1, one per tile, with its own arguments.
template <typename CT, int KIND, bool VIRT, bool USE1>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(waves(KIND)))) void sweep14_batch_kernel(
    const SweepArgs* args, const uint32_t* first, int count) {
    const int i = batch_item(first, count, blockIdx.x);
    const SweepArgs a = args[i];
    const uint32_t t = blockIdx.x - first[i];
    sweep_tile<CT, KIND, VIRT, USE1>(a, t, a.partials + 3 * (size_t)t);
}

template <typename CT>
hipError_t launch_ct(int kind, const SweepArgs& a, hipStream_t s) {
    const bool virt = a.half && a.vbit >= 0;
    return by_kind(kind, virt, sweep_l1(TB, kind, a.pre_mask, a.post_mask) == 1, [&](auto k, auto vi, auto u) {
        hipLaunchKernelGGL((sweep14_kernel<CT, k.value, vi.value, u.value>), dim3(1u << a.nw), dim3(NT), 0, s, a);
        return hipGetLastError();
    });
}

template <typename CT>
hipError_t launch_batch_ct(int kind, const SweepArgs* args, const uint32_t* first, int count, uint32_t blocks, bool virt,
                           int l1, LaunchTo to) {
    return by_kind(kind, virt, l1 != 2, [&](auto k, auto vi, auto u) {
        return launch_to(to, dim3(blocks), dim3(NT), sweep14_batch_kernel<CT, k.value, vi.value, u.value>, args, first,
                         count);
    });
}

}  // namespace

hipError_t launch_sweep14(int dtype, int kind, const SweepArgs& a, hipStream_t s) {
    return dtype == 1 ? launch_ct<uint8_t>(kind, a, s) : launch_ct<uint16_t>(kind, a, s);
}

hipError_t launch_sweep14_batch(int dtype, int kind, const SweepArgs* args, const uint32_t* first, int count,
                                uint32_t blocks, LaunchTo to, bool virt, int l1) {
    return dtype == 1 ? launch_batch_ct<uint8_t>(kind, args, first, count, blocks, virt, l1, to)
                      : launch_batch_ct<uint16_t>(kind, args, first, count, blocks, virt, l1, to);
}

}  // namespace qnae
