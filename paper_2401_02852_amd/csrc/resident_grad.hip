// Whole gradients of small states (n <= 13) in one workgroup: forward, readout,
// lam = W psi, then the reverse pass on both states (formulas: adjoint.hip), psi
// refreshed from checkpoints.
//
// From n = 10 on both states live in registers, 16 amplitudes of each a thread,
// in the layouts of resident.h. What bounds it is the depth of a layer, four
// barriers and two LDS trips, and the FP32 rate of one CU at one or two waves per
// SIMD. With the states in LDS, a pass per three qubits and one for the phase, and exact
// (cos, sin) butterflies one gradient of eight layers took 86, 98, 117 and 175 us a
// call (n = 10, 11, 12, 13), this takes 78, 83, 97 and 133 (exact butterflies in
// registers: 89, 95, 110 and 146; tangent forms in LDS: 91, 100, 120 and 179). 100 of
// n = 12 with 16-bit costs 94 -> 82 us. Pair sums go to FP64 after 32 FP32 terms.
// Phase tables: all rows in LDS if they fit, else, with 256 threads or more, the
// next row is loaded while a layer is mixed (16 gathers a thread from a
// row in global memory touch up to 64 lines each), else rows where they are.
// Below n = 10 (at most half a wave at 16 amplitudes a thread) the states
// stay in LDS.
#include "resident.h"

namespace qnae {
namespace {

using namespace tile;

constexpr int kResidentGradThreads = 512;  // what n = 13 takes (n = 9, eight layers: 1024 threads 79 us, 512 71)
constexpr int kGradWaves = kResidentGradThreads / 64;

// ---------------------------------------------------------------------------
// n <= 9
// ---------------------------------------------------------------------------

// LDS slot of element x: one pad slot per 16, so that threads that hold runs
// of four or eight elements fall in different banks.
__device__ __forceinline__ uint32_t gslot(uint32_t x) { return x + (x >> 4); }

// NB consecutive bits from g0 of the resident states at once: a task holds the
// 2^NB elements of one coset of p (and of l), and for each bit first sums
// Im<l|X_j|p> (REV), then applies a' = c a - i s b. Three bits a pass touch
// LDS a third as often as one, and need a third of the barriers.
template <int NB, bool REV>
__device__ __forceinline__ float resident_pass(float2* l, float2* p, uint32_t N, int g0, float c, float s) {
    constexpr int K = 1 << NB;
    float acc = 0.f;
    for (uint32_t task = threadIdx.x; task < (N >> NB); task += kResidentGradThreads) {
        const uint32_t b = ((task >> g0) << (g0 + NB)) | (task & ((1u << g0) - 1u));
        float2 pv[K], lv[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const uint32_t at = gslot(b | ((uint32_t)i << g0));
            pv[i] = p[at];
            if (REV) lv[i] = l[at];
        }
        auto rotate = [&](float2& x, float2& y) {
            const float2 u = x, w = y;
            x = make_float2(fmaf(c, u.x, s * w.y), fmaf(c, u.y, -s * w.x));
            y = make_float2(fmaf(c, w.x, s * u.y), fmaf(c, w.y, -s * u.x));
        };
#pragma unroll
        for (int q = 0; q < NB; ++q) {
#pragma unroll
            for (int i = 0; i < K; ++i) {
                if (i & (1 << q)) continue;
                const int k = i | (1 << q);
                if (REV) {
                    acc = fmaf(lv[i].x, pv[k].y, acc);
                    acc = fmaf(-lv[i].y, pv[k].x, acc);
                    acc = fmaf(lv[k].x, pv[i].y, acc);
                    acc = fmaf(-lv[k].y, pv[i].x, acc);
                    rotate(lv[i], lv[k]);
                }
                rotate(pv[i], pv[k]);
            }
        }
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const uint32_t at = gslot(b | ((uint32_t)i << g0));
            p[at] = pv[i];
            if (REV) l[at] = lv[i];
        }
    }
    __syncthreads();
    return acc;
}

// Every bit of a layer's mixer.
template <bool REV>
__device__ __forceinline__ float resident_layer(float2* l, float2* p, uint32_t N, int n, float c, float s) {
    float acc = 0.f;
    int g = 0;
    for (; g + 3 <= n; g += 3) acc += resident_pass<3, REV>(l, p, N, g, c, s);
    if (n - g == 2) acc += resident_pass<2, REV>(l, p, N, g, c, s);
    else if (n - g == 1) acc += resident_pass<1, REV>(l, p, N, g, c, s);
    return acc;
}

// Sum over the workgroup: wave sums, then the wave totals in wave order.
__device__ __forceinline__ double block_sum(double v, double* red) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    __syncthreads();
    if ((threadIdx.x & 63u) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double sum = 0.0;
    for (int w = 0; w < kResidentGradThreads / 64; ++w) sum += red[w];
    return sum;
}

template <typename CT>
__device__ __forceinline__ void small_body(const ResidentGradArgs& a, float2* ls, float2* ps, double* red) {
    constexpr uint32_t NT = kResidentGradThreads;
    const int n = a.n;
    const uint32_t N = 1u << n;
    const uint32_t tid = threadIdx.x;
    const CT* cost = (const CT*)a.cost;
    const uint32_t last = (uint32_t)a.lut_len - 1u;
    const float amp = __builtin_ldexpf(1.0f, -n) == 0.f ? 0.f : sqrtf(__builtin_ldexpf(1.0f, -n));
    // forward
    for (int l = 0; l < a.p; ++l) {
        const float2* lut = a.luts + (size_t)l * a.lut_len;
        for (uint32_t x = tid; x < N; x += NT) {
            const float2 e = lut[min((uint32_t)cost[x], last)];
            ps[gslot(x)] = l == 0 ? make_float2(amp * e.x, amp * e.y) : cmul(ps[gslot(x)], e);
        }
        __syncthreads();
        const float2 cs = a.cs[l];
        resident_layer<false>(nullptr, ps, N, n, cs.x, cs.y);
        if ((l + 1) % a.every == 0 && l + 1 < a.p) {
            float2* ck = a.ckpt + (size_t)((l + 1) / a.every - 1) * N;
            for (uint32_t x = tid; x < N; x += NT) ck[x] = ps[gslot(x)];
        }
    }
    if (a.p == 0)
        for (uint32_t x = tid; x < N; x += NT) ps[gslot(x)] = make_float2(amp, 0.f);
    __syncthreads();
    // readout and lam = W psi
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (uint32_t x = tid; x < N; x += NT) {
        const float2 v = ps[gslot(x)];
        const uint32_t c = cost[x];
        const float pr = fmaf(v.x, v.x, v.y * v.y);
        s2 += pr;
        s1 += (double)c * pr;
        s0 += c == 0u ? pr : 0.0;
        const float w = (float)a.w_energy * (float)c + (c == 0u ? (float)a.w_psucc : 0.f);
        ls[gslot(x)] = make_float2(w * v.x, w * v.y);
    }
    s0 = block_sum(s0, red);
    s1 = block_sum(s1, red);
    s2 = block_sum(s2, red);
    if (tid == 0) {
        a.out[0] = s0;
        a.out[1] = s1;
        a.out[2] = s2;
    }
    __syncthreads();
    // reverse
    for (int l = a.p - 1; l >= 0; --l) {
        const float2 cs = a.cs[l];
        const float accb = resident_layer<true>(ls, ps, N, n, cs.x, -cs.y);
        const float2* lut = a.luts + (size_t)l * a.lut_len;
        float accg = 0.f;
        for (uint32_t x = tid; x < N; x += NT) {
            const uint32_t c = cost[x];
            const float2 lv = ls[gslot(x)], pv = ps[gslot(x)];
            accg = fmaf((float)c, fmaf(lv.x, pv.y, -lv.y * pv.x), accg);
            const float2 e = lut[min(c, last)];
            const float2 ec = make_float2(e.x, -e.y);
            ls[gslot(x)] = cmul(lv, ec);
            ps[gslot(x)] = cmul(pv, ec);
        }
        const double db = block_sum((double)accb, red);
        const double dg = block_sum((double)accg, red);
        if (tid == 0) {
            a.out[3 + l] = 2.0 * dg;
            a.out[3 + a.p + l] = 2.0 * db;
        }
        if (l % a.every == 0 && l > 0) {
            const float2* ck = a.ckpt + (size_t)(l / a.every - 1) * N;
            for (uint32_t x = tid; x < N; x += NT) ps[gslot(x)] = ck[x];
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// n = 10 .. 13
// ---------------------------------------------------------------------------

// One layer's R = c I - i s X per qubit. With |s| <= |c| as c (I - i t X), t = s / c: two
// FMAs per amplitude and qubit instead of two and two products, the factor
// f = c^n applied once at the end; the pair terms taken after k qubits carry
// |c|^-2k, which the running weight (r = c^2 each) takes back. f and r come from t in
// FP64, so a layer is unitary to one rounding.
struct GradMix {
    float c, s, t, r, f;
    bool tan;
};
template <int NB>
__device__ __forceinline__ GradMix grad_mix(float c, float s) {
    GradMix m{c, s, 0.f, 1.f, 1.f, fabsf(s) <= fabsf(c)};
    if (m.tan) {
        m.t = s / c;
        const double r = 1.0 / (1.0 + (double)m.t * m.t);
        double f = NB & 1 ? copysign(sqrt(r), (double)c) : 1.0;
#pragma unroll
        for (int k = 0; k < NB / 2; ++k) f *= r;
        m.r = (float)r;
        m.f = (float)f;
    }
    return m;
}

// a' = c a - i s b on register bit S.
template <int S>
__device__ __forceinline__ void rot(float2 (&v)[16], float c, float s) {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        if (j & (1 << S)) continue;
        const float2 u = v[j], w = v[j | (1 << S)];
        v[j] = make_float2(fmaf(c, u.x, s * w.y), fmaf(c, u.y, -s * w.x));
        v[j | (1 << S)] = make_float2(fmaf(c, w.x, s * u.y), fmaf(c, w.y, -s * u.x));
    }
}
// Im of sum over pairs on register bit S of conj(l_a) p_b + conj(l_b) p_a.
template <int S>
__device__ __forceinline__ float pairs(const float2 (&l)[16], const float2 (&p)[16]) {
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const float2 a = l[j], b = p[j ^ (1 << S)];
        acc = fmaf(a.x, b.y, acc);
        acc = fmaf(-a.y, b.x, acc);
    }
    return acc;
}
__device__ __forceinline__ float2 lane_other(float2 x) {
    return make_float2(__int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x.x), kLaneXor1, 0xf, 0xf, true)),
                       __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x.y), kLaneXor1, 0xf, 0xf, true)));
}

// One layer's mixer on p (REV: on l and p, returning the pair sums of all qubits).
// between(): called after the first barrier.
template <int NB, bool REV, bool TAN, typename F>
__device__ __forceinline__ double mix_form(const RegPlaces<NB>& at, float2* ldl, float2* ldp, float2 (&l)[16],
                                           float2 (&p)[16], const GradMix& m, F&& between) {
    double acc = 0.0;
    float w = 1.f;
    auto add = [&](float q) {
        // complete here: sunk below the next transpose, the sums would hold the
        // values from before the butterflies in registers
        asm volatile("" : "+v"(q));
        acc += (double)(TAN ? w * q : q);
        if (TAN) w *= m.r;
    };
    auto bit = [&](auto sb) {
        constexpr int S = sb.value;
        if (REV) {
            add(pairs<S>(l, p));
            if constexpr (TAN) bfly<16, S>(l, m.t);
            else rot<S>(l, m.c, m.s);
        }
        if constexpr (TAN) bfly<16, S>(p, m.t);
        else rot<S>(p, m.c, m.s);
    };
    auto bits = [&] {
        bit(std::integral_constant<int, 0>{});
        bit(std::integral_constant<int, 1>{});
        bit(std::integral_constant<int, 2>{});
        bit(std::integral_constant<int, 3>{});
    };
    bits();
    r_swap16(p);
    s_swap(p);
    if (REV) {
        r_swap16(l);
        s_swap(l);
    }
    bit(std::integral_constant<int, 2>{});
    bit(std::integral_constant<int, 3>{});
    __syncthreads();
    between();
    at.put_a2(ldp, p);
    if (REV) at.put_a2(ldl, l);
    __syncthreads();
    at.get_b(ldp, p);
    if (REV) at.get_b(ldl, l);
    bits();
    if constexpr (NB >= 11) {
        r_swap16(p);
        if constexpr (NB >= 12) s_swap(p);
        if (REV) {
            r_swap16(l);
            if constexpr (NB >= 12) s_swap(l);
        }
        bit(std::integral_constant<int, 2>{});
    }
    if constexpr (NB >= 12) bit(std::integral_constant<int, 3>{});
    if constexpr (NB >= 13) {
        float q = 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const float2 po = lane_other(p[j]);
            if (REV) {
                const float2 lo = lane_other(l[j]);
                q = fmaf(l[j].x, po.y, q);
                q = fmaf(-l[j].y, po.x, q);
                l[j] = TAN ? make_float2(fmaf(m.t, lo.y, l[j].x), fmaf(-m.t, lo.x, l[j].y))
                           : make_float2(fmaf(m.c, l[j].x, m.s * lo.y), fmaf(m.c, l[j].y, -m.s * lo.x));
            }
            p[j] = TAN ? make_float2(fmaf(m.t, po.y, p[j].x), fmaf(-m.t, po.x, p[j].y))
                       : make_float2(fmaf(m.c, p[j].x, m.s * po.y), fmaf(m.c, p[j].y, -m.s * po.x));
        }
        if (REV) add(q);
    }
    __syncthreads();
    at.put_b2(ldp, p);
    if (REV) at.put_b2(ldl, l);
    __syncthreads();
    at.get_a(ldp, p);
    if (REV) at.get_a(ldl, l);
    if (TAN) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            p[j] = make_float2(m.f * p[j].x, m.f * p[j].y);
            if (REV) l[j] = make_float2(m.f * l[j].x, m.f * l[j].y);
        }
    }
    return acc;
}
template <int NB, bool REV, typename F>
__device__ __forceinline__ double mix_layer(const RegPlaces<NB>& at, float2* ldl, float2* ldp, float2 (&l)[16],
                                            float2 (&p)[16], float c, float s, F&& between) {
    const GradMix m = grad_mix<NB>(c, s);
    return m.tan ? mix_form<NB, REV, true>(at, ldl, ldp, l, p, m, between)
                 : mix_form<NB, REV, false>(at, ldl, ldp, l, p, m, between);
}

constexpr int kGradTab = 2560;  // phase table entries kept in LDS
template <int NB, typename CT>
__device__ __forceinline__ void reg_body(const ResidentGradArgs& a, float2* ldl, float2* ldp, float2* tab,
                                         double (*red)[3][kGradWaves]) {
    constexpr uint32_t N = 1u << NB;
    constexpr int NT = kRegThreads<NB>, NW = NT / 64;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // 1: every row in tab, 2: the row in use, 0: none
    const int mode = rows_fit(a.p, a.lut_len, kGradTab) ? 1 : NT >= 256 && a.lut_len <= kGradTab ? 2 : 0;
    const int begin = mode == 1 ? a.p * a.lut_len : mode == 2 ? a.lut_len : 0;
    for (int i = threadIdx.x; i < begin; i += kResidentGradThreads) tab[i] = a.luts[i];
    __syncthreads();
    if (wave >= (uint32_t)NW) {  // a smaller state's spare waves keep the barriers company
        for (int l = 0; l < 8 * a.p; ++l) __syncthreads();
        __syncthreads();
        __syncthreads();
        return;
    }
    const RegPlaces<NB> at(lane, wave);
    const uint32_t x0 = at.x0;
    uint32_t c[4 * sizeof(CT)];
    load_costs<NB, CT>(c, (const CT*)a.cost, x0, false);
    const uint32_t last = (uint32_t)a.lut_len - 1u;
    auto with_row = [&](int l, auto&& f) {
        if (mode == 0) f(a.luts + (size_t)l * a.lut_len);
        else f((const float2*)tab + (mode == 1 ? l * a.lut_len : 0));
    };
    constexpr int R = NT >= 256 ? kGradTab / NT : 1;
    float2 next[R];
    bool fetched = false;
    auto fetch = [&](int l) {  // row l on its way, if rows come one at a time
        fetched = mode == 2 && l >= 0 && l < a.p;
        if (NT < 256 || !fetched) return;
        const float2* const row = a.luts + (size_t)l * a.lut_len;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int at_i = (int)(wave * 64u + lane) + i * NT;
            next[i] = row[at_i < a.lut_len ? at_i : a.lut_len - 1];
        }
    };
    auto keep = [&] {
        if (NT < 256 || !fetched) return;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int at_i = (int)(wave * 64u + lane) + i * NT;
            if (at_i < a.lut_len) tab[at_i] = next[i];
        }
    };
    const float amp = sqrtf(__builtin_ldexpf(1.0f, -NB));
    float2 l[16], p[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) l[j] = p[j] = make_float2(amp, 0.f);
    for (int q = 0; q < a.p; ++q) {
        with_row(q, [&](const float2* row) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const float2 e = row[min(cost_of<CT>(c, j), last)];
                p[j] = q == 0 ? make_float2(amp * e.x, amp * e.y) : cmul(p[j], e);
            }
        });
        fetch(q + 1);
        const float2 cs = a.cs[q];
        mix_layer<NB, false>(at, ldl, ldp, l, p, cs.x, cs.y, keep);
        if ((q + 1) % a.every == 0 && q + 1 < a.p) {
            float4* const ck = (float4*)(a.ckpt + (size_t)((q + 1) / a.every - 1) * N + x0);
#pragma unroll
            for (int j = 0; j < 8; ++j) ck[j] = make_float4(p[2 * j].x, p[2 * j].y, p[2 * j + 1].x, p[2 * j + 1].y);
        }
    }
    // readout and lam = W psi
    double r[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const uint32_t cx = cost_of<CT>(c, j);
        const double pr = (double)fmaf(p[j].x, p[j].x, p[j].y * p[j].y);
        r[0] += cx == 0u ? pr : 0.0;
        r[1] += (double)cx * pr;
        r[2] += pr;
        const float w = (float)a.w_energy * (float)cx + (cx == 0u ? (float)a.w_psucc : 0.f);
        l[j] = make_float2(w * p[j].x, w * p[j].y);
    }
    auto wave_sum = [&](double (*to)[kGradWaves], int count) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (k >= count) continue;
            for (int off = 32; off > 0; off >>= 1) r[k] += __shfl_xor(r[k], off);
            if (lane == 0) to[k][wave] = r[k];
        }
    };
    auto total = [&](const double* from) {
        double sum = 0.0;
        for (int w = 0; w < NW; ++w) sum += from[w];
        return sum;
    };
    wave_sum(red[2], 3);
    __syncthreads();
    if (threadIdx.x < 3) a.out[threadIdx.x] = total(red[2][threadIdx.x]);
    // reverse; a layer's sums leave after the next barriers
    auto leave = [&](int q) {
        if (threadIdx.x < 2) a.out[3 + threadIdx.x * a.p + q] = 2.0 * total(red[q & 1][threadIdx.x]);
    };
    for (int q = a.p - 1; q >= 0; --q) {
        fetch(q < a.p - 1 ? q : -1);  // the last row is still there
        const float2 cs = a.cs[q];
        r[1] = mix_layer<NB, true>(at, ldl, ldp, l, p, cs.x, -cs.y, keep);
        if (q < a.p - 1) leave(q + 1);
        r[0] = 0.0;
        with_row(q, [&](const float2* row) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const uint32_t cx = cost_of<CT>(c, j);
                r[0] += (double)((float)cx * fmaf(l[j].x, p[j].y, -l[j].y * p[j].x));
                const float2 e = row[min(cx, last)];
                const float2 ec = make_float2(e.x, -e.y);
                l[j] = cmul(l[j], ec);
                p[j] = cmul(p[j], ec);
            }
        });
        wave_sum(red[q & 1], 2);
        if (q % a.every == 0 && q > 0) {
            const float4* const ck = (const float4*)(a.ckpt + (size_t)(q / a.every - 1) * N + x0);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float4 u = ck[j];
                p[2 * j] = make_float2(u.x, u.y);
                p[2 * j + 1] = make_float2(u.z, u.w);
            }
        }
    }
    __syncthreads();
    if (a.p > 0) leave(0);
}

// One workgroup per gradient.
template <typename CT>
__global__ __launch_bounds__(kResidentGradThreads) void resident_grad_batch_kernel(const ResidentGradArgs* args) {
    __shared__ __align__(16) float2 ldl[reg_lds(13)];
    __shared__ __align__(16) float2 ldp[reg_lds(13)];
    __shared__ float2 tab[kGradTab];
    __shared__ double red[3][3][kGradWaves];
    const ResidentGradArgs a = args[blockIdx.x];
    switch (a.n) {
        case 13: return reg_body<13, CT>(a, ldl, ldp, tab, red);
        case 12: return reg_body<12, CT>(a, ldl, ldp, tab, red);
        case 11: return reg_body<11, CT>(a, ldl, ldp, tab, red);
        case 10: return reg_body<10, CT>(a, ldl, ldp, tab, red);
        default: return small_body<CT>(a, ldl, ldp, red[0][0]);
    }
}

}  // namespace

hipError_t launch_resident_grad_batch(int dtype, const ResidentGradArgs* args, int count, hipStream_t s) {
    if (dtype == 1)
        hipLaunchKernelGGL(resident_grad_batch_kernel<uint8_t>, dim3((uint32_t)count), dim3(kResidentGradThreads), 0, s,
                           args);
    else
        hipLaunchKernelGGL(resident_grad_batch_kernel<uint16_t>, dim3((uint32_t)count), dim3(kResidentGradThreads), 0, s,
                           args);
    return hipGetLastError();
}

}  // namespace qnae
