// Whole circuits of small states (n <= 14) in one workgroup.
//
// From n = 10 on the state lives in registers, 16 amplitudes a thread: 2^(n-4)
// threads, layouts in resident.h.
// What bounds it is the depth of that chain:
// a single workgroup, four barriers a layer (and at n = 14 the CU's FP32 rate: about
// 11 of 17 thousand cycles a layer). Keeping the state in LDS, with a pass per three
// or four qubits and one for the phase, took per call (three layers, n = 12, 13,
// 14) 36, 46 and 60 us, this 28, 34 and 44; sixteen layers 81, 143 and 228, 55, 86 and 136.
// Below n = 10 (at most half a wave at 16 amplitudes a thread) the state
// stays in LDS. A batch has one workgroup of 1024 threads per instance; the waves
// that a smaller state leaves over only meet its barriers.
#include "resident.h"

namespace qnae {
namespace {

using namespace tile;

// ---------------------------------------------------------------------------
// n <= 9
// ---------------------------------------------------------------------------

// LDS slot of amplitude x: one pad slot per 16, so that the threads of the
// bits-0..3 pass, each holding 16 consecutive amplitudes, fall in different
// banks instead of all in one (a stride of 16 float2 is 32 banks).
__device__ __forceinline__ uint32_t rslot(uint32_t x) { return x + (x >> 4); }

constexpr int kResidentThreads = 1024;  // of small states, and of every workgroup of a batch

// Radix-2^NBP butterfly passes of one layer over the LDS state: each task
// holds the 2^nb amplitudes of one coset of nb consecutive qubits.
template <int NBP>
__device__ __forceinline__ void resident_mix(float2* s, int n, uint32_t N, float t) {
    for (int g0 = 0; g0 < n; g0 += NBP) {
        const int nb = n - g0 < NBP ? n - g0 : NBP;
        const uint32_t tasks = N >> nb;
        for (uint32_t task = threadIdx.x; task < tasks; task += kResidentThreads) {
            const uint32_t bs = ((task >> g0) << (g0 + nb)) | (task & ((1u << g0) - 1u));
            float2 v[1 << NBP];
#pragma unroll
            for (int i = 0; i < (1 << NBP); ++i)
                v[i] = i < (1 << nb) ? s[rslot(bs | ((uint32_t)i << g0))] : make_float2(0.f, 0.f);
            if (nb > 0) bfly<(1 << NBP), 0>(v, t);
            if (NBP > 1 && nb > 1) bfly<(1 << NBP), (NBP > 1 ? 1 : 0)>(v, t);
            if (NBP > 2 && nb > 2) bfly<(1 << NBP), (NBP > 2 ? 2 : 0)>(v, t);
            if (NBP > 3 && nb > 3) bfly<(1 << NBP), (NBP > 3 ? 3 : 0)>(v, t);
#pragma unroll
            for (int i = 0; i < (1 << NBP); ++i)
                if (i < (1 << nb)) s[rslot(bs | ((uint32_t)i << g0))] = v[i];
        }
        __syncthreads();
    }
}

template <typename CT>
__device__ __forceinline__ void small_body(const ResidentArgs& a, float2* s, CT* cs, double (*red)[16]) {
    constexpr uint32_t NT = kResidentThreads;
    const int n = a.n;
    const uint32_t N = 1u << n;
    const uint32_t tid = threadIdx.x;
    const CT* const cost_g = (const CT*)a.cost;
    for (uint32_t x = tid; x < N; x += NT) cs[x] = cost_g[x];
    __syncthreads();
    const CT* const cost = cs;
    const uint32_t last = (uint32_t)a.lut_len - 1u;
    const int layers = a.p > 0 ? a.p : 1;
    // The butterflies drop the X of the cot form; `flip` records that the
    // stored state is the true one with every qubit flipped.
    uint32_t flip = 0u;
    for (int l = 0; l < layers; ++l) {
        const float2* lut = a.luts + (size_t)l * a.lut_len;
        for (uint32_t x = tid; x < N; x += NT) {
            const float2 e = lut[min((uint32_t)cost[x ^ flip], last)];
            s[rslot(x)] = l > 0 ? cmul(s[rslot(x)], e) : a.state_in ? cmul(a.state_in[x], e) : e;
        }
        __syncthreads();
        if (a.p == 0) break;
        const MixForm f = a.forms[l];
        resident_mix<3>(s, n, N, f.t);
        if (f.flip) flip ^= N - 1u;
    }
    float s0 = 0.f, s1 = 0.f, s2 = 0.f;
    for (uint32_t x = tid; x < N; x += NT) {
        const float2 q = s[rslot(x)];
        const float pr = fmaf(q.x, q.x, q.y * q.y);
        const uint32_t cx = cost[x ^ flip];
        s2 += pr;
        s1 = fmaf((float)cx, pr, s1);
        s0 += cx == 0u ? pr : 0.f;
        if (a.state_out) a.state_out[x ^ flip] = cmul(q, a.store_scale);
    }
    double d0 = s0, d1 = s1, d2 = s2;
    for (int off = 32; off > 0; off >>= 1) {
        d0 += __shfl_xor(d0, off);
        d1 += __shfl_xor(d1, off);
        d2 += __shfl_xor(d2, off);
    }
    if ((tid & 63u) == 0) {
        red[0][tid >> 6] = d0;
        red[1][tid >> 6] = d1;
        red[2][tid >> 6] = d2;
    }
    __syncthreads();
    if (tid < 3) {
        double sum = 0.0;
        for (uint32_t w = 0; w < NT / 64; ++w) sum += red[tid][w];
        a.out[tid] = sum;
    }
}

// ---------------------------------------------------------------------------
// n = 10 .. 14
// ---------------------------------------------------------------------------
// Waves past the state's own (workgroups of a batch) keep its barriers company.
constexpr int kTabMax = 2048;  // phase table entries kept in LDS; longer ones are read where they are
template <int NB, typename CT>
__device__ __forceinline__ void reg_body(const ResidentArgs& a, float2* lds, float2* tab, bool in_tab,
                                         double (*red)[16]) {
    constexpr uint32_t N = 1u << NB;
    constexpr int NW = kRegThreads<NB> / 64;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int layers = a.p > 0 ? a.p : 1;
    if (!in_tab && rows_fit(layers, a.lut_len, kTabMax)) {
        for (int i = threadIdx.x; i < layers * a.lut_len; i += blockDim.x) tab[i] = a.luts[i];
        in_tab = true;
    }
    __syncthreads();
    if (wave >= (uint32_t)NW) {
        for (int l = 0; l < 4 * a.p; ++l) __syncthreads();
        __syncthreads();
        return;
    }
    const RegPlaces<NB> at(lane, wave);
    const uint32_t x0 = at.x0;

    uint32_t c[4 * sizeof(CT)];
    load_costs<NB, CT>(c, (const CT*)a.cost, x0, false);
    const uint32_t last = (uint32_t)a.lut_len - 1u;
    // The butterflies drop the X of the cot form; `flip` records that the
    // stored state is the true one with every qubit flipped.
    bool flip = false;
    float2 v[16];
    for (int l = 0; l < layers; ++l) {
        auto phase = [&](const float2* row) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const float2 e = row[min(cost_of<CT>(c, j), last)];
                v[j] = l > 0 ? cmul(v[j], e) : a.state_in ? cmul(a.state_in[x0 + j], e) : e;
            }
        };
        if (in_tab) phase(tab + l * a.lut_len);
        else phase(a.luts + (size_t)l * a.lut_len);
        if (a.p == 0) break;
        const MixForm f = a.forms[l];
        if (f.flip) {
            flip = !flip;
            load_costs<NB, CT>(c, (const CT*)a.cost, x0, flip);
        }
        const float t = f.t;
        bfly<16, 0>(v, t);
        bfly<16, 1>(v, t);
        bfly<16, 2>(v, t);
        bfly<16, 3>(v, t);
        r_swap16(v);
        s_swap(v);
        bfly<16, 2>(v, t);  // e4, e5
        bfly<16, 3>(v, t);
        __syncthreads();
        at.put_a2(lds, v);
        __syncthreads();
        at.get_b(lds, v);
        bfly<16, 0>(v, t);
        bfly<16, 1>(v, t);
        bfly<16, 2>(v, t);
        bfly<16, 3>(v, t);
        if constexpr (NB >= 11) {
            r_swap16(v);
            if constexpr (NB >= 12) s_swap(v);
            bfly<16, 2>(v, t);  // e10
        }
        if constexpr (NB >= 12) bfly<16, 3>(v, t);  // e11
        if constexpr (NB >= 13) lane_bfly<kLaneXor1>(v, t);
        if constexpr (NB >= 14) lane_bfly<kLaneXor2>(v, t);
        __syncthreads();
        at.put_b2(lds, v);
        __syncthreads();
        at.get_a(lds, v);
    }
    double d0 = 0.0, d1 = 0.0, d2 = 0.0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const double pr = (double)fmaf(v[j].x, v[j].x, v[j].y * v[j].y);
        const uint32_t cx = cost_of<CT>(c, j);
        d2 += pr;
        d1 = fma((double)cx, pr, d1);
        d0 += cx == 0u ? pr : 0.0;
    }
    if (a.state_out) {
#pragma unroll
        for (int j = 0; j < 16; j += 2) {
            const float2 u = cmul(v[j], a.store_scale), w = cmul(v[j + 1], a.store_scale);
            if (flip) *(float4*)(a.state_out + (N - 16u - x0) + (14 - j)) = make_float4(w.x, w.y, u.x, u.y);
            else *(float4*)(a.state_out + x0 + j) = make_float4(u.x, u.y, w.x, w.y);
        }
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
        for (int w = 0; w < NW; ++w) sum += red[threadIdx.x][w];
        a.out[threadIdx.x] = sum;
    }
}

// NB = 0: n <= 9.
template <int NB>
constexpr int kResThreads = NB ? 1 << (NB - 4) : kResidentThreads;
template <int NB, typename CT>
__global__ __launch_bounds__(kResThreads<NB>) void resident_kernel(const ResidentArgs a) {
    __shared__ __align__(16) float2 lds[NB ? reg_lds(NB) : 512 + 32];
    __shared__ float2 tab[NB ? kTabMax : 128];
    __shared__ double red[3][16];
    if constexpr (NB != 0) reg_body<NB, CT>(a, lds, tab, false, red);
    else small_body<CT>(a, lds, (CT*)tab, red);
}

// Tables from the kernel arguments, staged in LDS.
template <int NB, typename CT>
__global__ __launch_bounds__(kResThreads<NB>) void resident_inline_kernel(const ResidentInlineArgs ia) {
    __shared__ __align__(16) float2 lds[NB ? reg_lds(NB) : 512 + 32];
    __shared__ float2 tab[kResidentInline];
    __shared__ CT cs[NB ? 1 : 512];
    __shared__ double red[3][16];
    const int layers = ia.a.p > 0 ? ia.a.p : 1;
    const int count = layers * ia.a.lut_len + ia.a.p;
    for (int i = threadIdx.x; i < count; i += kResThreads<NB>) tab[i] = ia.tab[i];
    ResidentArgs a = ia.a;
    if constexpr (NB != 0) {
        a.forms = (const MixForm*)(ia.tab + layers * ia.a.lut_len);
        reg_body<NB, CT>(a, lds, tab, true, red);
    } else {
        __syncthreads();
        a.luts = tab;
        a.forms = (const MixForm*)(tab + layers * ia.a.lut_len);
        small_body<CT>(a, lds, cs, red);
    }
}

// Many small instances, one workgroup each.
template <typename CT>
__global__ __launch_bounds__(kResidentThreads) void resident_batch_kernel(const ResidentArgs* args) {
    __shared__ __align__(16) float2 lds[reg_lds(14)];
    __shared__ float2 tab[kTabMax];
    __shared__ double red[3][16];
    const ResidentArgs a = args[blockIdx.x];
    switch (a.n) {
        case 14: return reg_body<14, CT>(a, lds, tab, false, red);
        case 13: return reg_body<13, CT>(a, lds, tab, false, red);
        case 12: return reg_body<12, CT>(a, lds, tab, false, red);
        case 11: return reg_body<11, CT>(a, lds, tab, false, red);
        case 10: return reg_body<10, CT>(a, lds, tab, false, red);
        default: return small_body<CT>(a, lds, (CT*)tab, red);
    }
}

// f(NB) for a state of n qubits.
template <typename F>
hipError_t by_size(int n, F&& f) {
    switch (n) {
        case 14: return f(std::integral_constant<int, 14>{});
        case 13: return f(std::integral_constant<int, 13>{});
        case 12: return f(std::integral_constant<int, 12>{});
        case 11: return f(std::integral_constant<int, 11>{});
        case 10: return f(std::integral_constant<int, 10>{});
        default: return n >= 1 && n <= 9 ? f(std::integral_constant<int, 0>{}) : hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_resident(int dtype, const ResidentArgs& a, hipStream_t s) {
    return by_size(a.n, [&](auto nb) {
        constexpr int NB = nb.value;
        if (dtype == 1) hipLaunchKernelGGL((resident_kernel<NB, uint8_t>), dim3(1), dim3(kResThreads<NB>), 0, s, a);
        else hipLaunchKernelGGL((resident_kernel<NB, uint16_t>), dim3(1), dim3(kResThreads<NB>), 0, s, a);
        return hipGetLastError();
    });
}

hipError_t launch_resident_inline(int dtype, const ResidentInlineArgs& a, hipStream_t s) {
    const int layers = a.a.p > 0 ? a.a.p : 1;
    if ((int64_t)layers * a.a.lut_len + a.a.p > kResidentInline) return hipErrorInvalidValue;
    return by_size(a.a.n, [&](auto nb) {
        constexpr int NB = nb.value;
        if (dtype == 1) hipLaunchKernelGGL((resident_inline_kernel<NB, uint8_t>), dim3(1), dim3(kResThreads<NB>), 0, s, a);
        else hipLaunchKernelGGL((resident_inline_kernel<NB, uint16_t>), dim3(1), dim3(kResThreads<NB>), 0, s, a);
        return hipGetLastError();
    });
}

hipError_t launch_resident_batch(int dtype, const ResidentArgs* args, int count, LaunchTo to) {
    return launch_to(to, dim3(count), dim3(kResidentThreads),
                     dtype == 1 ? resident_batch_kernel<uint8_t> : resident_batch_kernel<uint16_t>, args);
}

}  // namespace qnae
