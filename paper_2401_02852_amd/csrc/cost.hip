// Cost diagonal kernel: C(x) = number of NAE-violated clauses, for every basis
// state x (Section 3.2, eq. knaesatobj; Appendix A.2, eq. demorgannae).
//
// Bit-sliced: a thread counts W runs of 32 consecutive states, a wave 64 W runs:
// state bits 0..4 in a run, 5..10 the lane, 11.. the thread's run, the rest
// the wave. Counters are NP bit planes per run (vertical counters).
//
// What bounds it is integer ALU work, so clauses are cut down to what a wave
// can see before any of its lanes counts: 64 clauses at a time, a lane per
// clause, the literals on the wave's own bits decide whether the clause can be
// violated there at all (with h of them 2^(1-h) can). Survivors go to two
// lists in LDS: clauses with a variable below 5 carry a 32-state violation
// pattern per polarity; the others are constant over a run and only count.
// Clauses that are constant over the whole wave are counted by the ballot. One
// pass over the first list then costs about 5 operations per clause and run
// (2 to form the pattern, 2.5 in a carry-save adder tree, and the lane
// compare, shared by the W runs), over the second about 1.5.
// Measured against every lane testing every clause with scalar loads: see
// launch_cost.
#include <type_traits>

#include "internal.h"
#include "tile.h"

namespace qnae {
namespace {

constexpr int kCostThreads = 256, kCostWaves = kCostThreads / 64;
constexpr int kCostChunk = 192;  // clauses filtered into the lists at a time: counts of a run fit a byte

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}

// Position of state s of a run in the planes: bit 8 (s & 3) + (s >> 2), so that
// transposing 8x8 bit blocks leaves four consecutive states in each word. The
// index bits rotate by two: swaps of index bits (0,2), (1,3), (2,4), (3,4).
template <int I, int J>
__device__ __forceinline__ uint32_t swap_index_bits(uint32_t x) {
    constexpr uint32_t set[5] = {0xAAAAAAAAu, 0xCCCCCCCCu, 0xF0F0F0F0u, 0xFF00FF00u, 0xFFFF0000u};
    constexpr uint32_t m = set[I] & ~set[J];  // bit I set, bit J clear
    constexpr int d = (1 << J) - (1 << I);
    const uint32_t t = ((x >> d) ^ x) & m;
    return x ^ t ^ (t << d);
}
__device__ __forceinline__ uint32_t to_planes(uint32_t x) {
    return swap_index_bits<3, 4>(swap_index_bits<2, 4>(swap_index_bits<1, 3>(swap_index_bits<0, 2>(x))));
}

// 8x8 transposes of the bit blocks of eight planes: byte q of word r becomes
// the counter of state 4 r + q.
__device__ __forceinline__ void transpose8(uint32_t (&p)[8]) {
    auto step = [&](int d, uint32_t m) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i & d) continue;
            const uint32_t a = p[i], b = p[i | d];
            p[i] = (a & m) | ((b << d) & ~m);
            p[i | d] = ((a >> d) & m) | (b & ~m);
        }
    };
    step(4, 0x0f0f0f0fu);
    step(2, 0x33333333u);
    step(1, 0x55555555u);
}

// Vertical counters of one run.
template <int NP>
struct Counter {
    uint32_t p[NP];
    // + carry 2^b0 (ripple)
    __device__ __forceinline__ void add_at(int b0, uint32_t carry) {
#pragma unroll
        for (int b = 0; b < NP; ++b) {
            if (b < b0) continue;
            const uint32_t t = p[b] & carry;
            p[b] ^= carry;
            carry = t;
        }
    }
    // + x + y at plane b; returns the carry out (weight 2^(b+1))
    __device__ __forceinline__ uint32_t csa(int b, uint32_t x, uint32_t y) {
        const uint32_t carry = maj3(p[b], x, y);
        p[b] = xor3(p[b], x, y);
        return carry;
    }
    __device__ __forceinline__ void add4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
        const uint32_t x = csa(0, a, b), y = csa(0, c, d);
        add_at(2, csa(1, x, y));
    }
    // + eight patterns; returns the carry of weight 8
    __device__ __forceinline__ uint32_t add8(const uint32_t (&v)[8]) {
        const uint32_t a = csa(0, v[0], v[1]), b = csa(0, v[2], v[3]), c = csa(0, v[4], v[5]), d = csa(0, v[6], v[7]);
        const uint32_t e = csa(1, a, b), f = csa(1, c, d);
        return csa(2, e, f);
    }
    // + n to every state
    __device__ __forceinline__ void add_all(uint32_t n) {
        uint32_t carry = 0u;
#pragma unroll
        for (int b = 0; b < NP; ++b) {
            const uint32_t bit = 0u - ((n >> b) & 1u);
            const uint32_t c = maj3(p[b], bit, carry);
            p[b] = xor3(p[b], bit, carry);
            carry = c;
        }
    }
};

// Wave `wv` of one diagonal: states [wv 2048 W, (wv + 1) 2048 W).
template <int NP, bool U16, int W>
__device__ __forceinline__ void cost_wave(const CostArgs& a, uint64_t wv) {
    static_assert(W == 1 || W == 4, "a thread counts one or four runs");
    constexpr int LB = W == 4 ? 13 : 11;  // state bits within a wave
    // Entries (pattern where every literal is false, where every one is true, their
    // signs on bits 5..10 and run masks, variables on bits 5..10): the first list
    // from the front, in multiples of four, the second from the back.
    __shared__ uint4 lists[kCostWaves][kCostChunk + 4];
    __shared__ uint32_t blk;
    uint32_t zeros = 0;
    const uint32_t lane = threadIdx.x & 63u;
    uint4* const list = lists[__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))];
    const uint64_t x0 = wv << LB;
    if (a.n >= LB ? (wv >> (a.n - LB)) == 0ull : wv == 0ull) {
        const uint32_t xlo = (uint32_t)x0, xhi = (uint32_t)(x0 >> 32);
        Counter<NP> cnt[W];
        uint32_t runs[W];  // clauses counted as integers, per run
#pragma unroll
        for (int w = 0; w < W; ++w) {
            runs[w] = 0u;
#pragma unroll
            for (int b = 0; b < NP; ++b) cnt[w].p[b] = 0u;
        }
        uint32_t whole = 0u;  // clauses violated on the whole wave
        for (int c0 = 0; c0 < a.num_clauses; c0 += kCostChunk) {
            const int c1 = min(a.num_clauses, c0 + kCostChunk);
            uint32_t nfront = 0u, nback = 0u;
            for (int c = c0; c < c1; c += 64) {
                uint32_t zt = 0u, ft = 0u, signs = 0u, vars = 0u;
                bool low = false, fixed = false;  // a variable below 5; none below the wave's bits
                if (c + (int)lane < c1) {
                    const ClauseRec r = a.clauses[c + lane];
                    const uint32_t mlo = r.mask_hi_lo & ~((1u << LB) - 1u);
                    const uint32_t dlo = (xlo ^ r.pat_lo) & mlo, dhi = (xhi ^ r.pat_hi) & r.mask_hi_hi;
                    const uint32_t in = (r.mask_hi_lo >> 5) & ((1u << (LB - 5)) - 1u), sg = r.pat_lo >> 5;
                    if ((dlo | dhi) == 0u) zt = r.zero_tab;
                    if (dlo == mlo && dhi == r.mask_hi_hi) ft = r.full_tab;
                    low = r.zero_tab != ~0u;
                    vars = in & 63u;
                    uint32_t nw = 1u, aw = 1u;  // runs on whose own bits every literal is false, true
                    if (W == 4) {
                        nw = aw = 0u;
#pragma unroll
                        for (uint32_t w = 0; w < 4; ++w) {
                            const uint32_t d = (w ^ (sg >> 6)) & (in >> 6);
                            nw |= d == 0u ? 1u << w : 0u;
                            aw |= d == (in >> 6) ? 1u << w : 0u;
                        }
                    }
                    signs = (sg & 63u) | (nw << 16) | (aw << 20);
                    if (low) {
                        zt = to_planes(zt);
                        ft = to_planes(ft);
                    } else {  // constant over a run: a byte per run
                        zt = zt ? (nw * 0x00204081u) & 0x01010101u : 0u;
                        ft = ft ? (aw * 0x00204081u) & 0x01010101u : 0u;
                        fixed = in == 0u;
                    }
                }
                const bool alive = (zt | ft) != 0u;
                whole += (uint32_t)__popcll(__ballot(alive && fixed));
                const bool tof = alive && low, tob = alive && !low && !fixed;
                const uint64_t bf = __ballot(tof), bb = __ballot(tob);
                const uint64_t below = (1ull << lane) - 1ull;
                const uint4 e = make_uint4(zt, ft, signs, vars);
                if (tof) list[nfront + (uint32_t)__popcll(bf & below)] = e;
                if (tob) list[kCostChunk + 3u - nback - (uint32_t)__popcll(bb & below)] = e;
                nfront += (uint32_t)__popcll(bf);
                nback += (uint32_t)__popcll(bb);
            }
            // entries that never match fill the first list to a multiple of four
            if (lane < (4u - (nfront & 3u) & 3u)) list[nfront + lane] = make_uint4(0u, 0u, 0u, 0u);
            tile::wave_lds_sync();
            const uint32_t steps = (nfront + 3u) & ~3u;
            // Patterns of entry i over the thread's runs.
            auto viol = [&](uint32_t i, uint32_t(&v)[W]) {
                const uint4 e = list[i];
                const uint32_t d = __builtin_amdgcn_bitop3_b32(lane, e.z, e.w, 0x28);  // (lane ^ z) & w
                const uint32_t z = d == 0u ? e.x : 0u, f = d == e.w ? e.y : 0u;
                if (W == 1) {
                    v[0] = z | f;
                } else {
                    const int s = __builtin_amdgcn_readfirstlane((int)e.z);
#pragma unroll
                    for (int w = 0; w < W; ++w) {
                        const uint32_t sn = (uint32_t)((s << (15 - w)) >> 31), sa = (uint32_t)((s << (11 - w)) >> 31);
                        v[w] = (z & sn) | (f & sa);
                    }
                }
            };
            auto eight = [&](uint32_t i, uint32_t(&carry)[W]) {
                uint32_t v[W][8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    uint32_t t[W];
                    viol(i + k, t);
#pragma unroll
                    for (int w = 0; w < W; ++w) v[w][k] = t[w];
                }
#pragma unroll
                for (int w = 0; w < W; ++w) carry[w] = cnt[w].add8(v[w]);
            };
            uint32_t i = 0;
            for (; i + 16u <= steps; i += 16u) {
                uint32_t x[W], y[W];
                eight(i, x);
                eight(i + 8u, y);
#pragma unroll
                for (int w = 0; w < W; ++w) cnt[w].add_at(4, cnt[w].csa(3, x[w], y[w]));
            }
            for (; i < steps; i += 4u) {
                uint32_t v[4][W];
#pragma unroll
                for (int k = 0; k < 4; ++k) viol(i + k, v[k]);
#pragma unroll
                for (int w = 0; w < W; ++w) cnt[w].add4(v[0][w], v[1][w], v[2][w], v[3][w]);
            }
            uint32_t bytes = 0u;
            for (uint32_t k = 0; k < nback; ++k) {
                const uint4 e = list[kCostChunk + 3u - k];
                const uint32_t d = __builtin_amdgcn_bitop3_b32(lane, e.z, e.w, 0x28);
                bytes += (d == 0u ? e.x : 0u) + (d == e.w ? e.y : 0u);
            }
#pragma unroll
            for (int w = 0; w < W; ++w) runs[w] += (bytes >> (8 * w)) & 0xffu;
            tile::wave_lds_sync();  // the lists are read before the next chunk's entries go in
        }
        const uint32_t valid = a.n >= 5 ? 0xffffffffu : to_planes((1u << (1u << a.n)) - 1u);
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint64_t x = x0 | (uint64_t)w << 11 | (uint64_t)lane << 5;
            if (x >> a.n) continue;  // (n below the wave's bits)
            cnt[w].add_all(whole + runs[w]);
            uint32_t any = 0u;
#pragma unroll
            for (int b = 0; b < NP; ++b) any |= cnt[w].p[b];
            zeros += (uint32_t)__popc(~any & valid);
            uint32_t lo[8];
#pragma unroll
            for (int b = 0; b < 8; ++b) lo[b] = b < NP ? cnt[w].p[b] : 0u;
            transpose8(lo);
            if (!U16) {
                uint8_t* const out = (uint8_t*)a.cost + x;
                if (a.n >= 5) {
                    ((uint4*)out)[0] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
                    ((uint4*)out)[1] = make_uint4(lo[4], lo[5], lo[6], lo[7]);
                } else {
                    for (uint32_t j = 0; j < (1u << a.n); ++j) out[j] = (uint8_t)(lo[j >> 2] >> (8 * (j & 3)));
                }
            } else {
                uint32_t hi[8];
#pragma unroll
                for (int b = 0; b < 8; ++b) hi[b] = b + 8 < NP ? cnt[w].p[b + 8] : 0u;
                transpose8(hi);
                uint32_t word[16];
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    word[2 * r] = __builtin_amdgcn_perm(hi[r], lo[r], 0x05010400u);
                    word[2 * r + 1] = __builtin_amdgcn_perm(hi[r], lo[r], 0x07030602u);
                }
                uint16_t* const out = (uint16_t*)a.cost + x;
                if (a.n >= 5) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        ((uint4*)out)[q] = make_uint4(word[4 * q], word[4 * q + 1], word[4 * q + 2], word[4 * q + 3]);
                } else {
                    for (uint32_t j = 0; j < (1u << a.n); ++j) out[j] = (uint16_t)(word[j >> 1] >> (16 * (j & 1)));
                }
            }
        }
    }
    if (a.zeros) {
        if (threadIdx.x == 0) blk = 0u;
        __syncthreads();
        // wave-level sum first, then one LDS atomic per wave
        uint32_t z = zeros;
        for (int off = 32; off > 0; off >>= 1) z += __shfl_xor(z, off);
        if ((threadIdx.x & 63) == 0 && z) atomicAdd(&blk, z);
        __syncthreads();
        if (threadIdx.x == 0 && blk) atomicAdd(a.zeros, (unsigned long long)blk);
    }
}

template <int NP, bool U16, int W>
__global__ __launch_bounds__(kCostThreads) void cost_kernel(const CostArgs a) {
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    cost_wave<NP, U16, W>(a, (uint64_t)blockIdx.x * kCostWaves + wave);
}

// Many diagonals at once: instance i owns blocks first[i] .. first[i+1]-1.
template <int NP, bool U16, int W>
__global__ __launch_bounds__(kCostThreads) void cost_batch_kernel(const CostArgs* args, const uint32_t* first,
                                                                  int count) {
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    const CostArgs a = args[lo];
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    cost_wave<NP, U16, W>(a, (uint64_t)(blockIdx.x - first[lo]) * kCostWaves + wave);
}

// What precedes a run in one launch: its tables from pinned host memory to the
// device (a copy command of their own took a 3-4 us kernel and a launch gap),
// and, with a cost, whether the diagonal is flip-symmetric: 16 bytes of the
// lower half against the 16 bytes at the mirrored place, reversed. Bound by
// the one read of the diagonal; a difference anywhere ends every workgroup's
// loop early.
__device__ __forceinline__ uint32_t flip_word(uint32_t w, bool u16) {
    return u16 ? (w >> 16) | (w << 16) : __builtin_bswap32(w);
}

constexpr int kProThreads = 256, kProUnroll = 4;

// Does a piece that thread `id` of `stride` looks at differ from its mirror
// image? found(): has another workgroup found one (asked when there is more
// to read)?
template <bool U16, typename F>
__device__ __forceinline__ bool flip_differs(const uint4* cost, uint64_t quads, uint64_t id, uint64_t stride,
                                             F&& found) {
    const uint64_t half = quads / 2;  // piece i faces quads - 1 - i
    uint32_t diff = 0u;
    for (uint64_t i = id; i < half; i += kProUnroll * stride) {
        uint4 x[kProUnroll], y[kProUnroll];
#pragma unroll
        for (int u = 0; u < kProUnroll; ++u) {
            const uint64_t j = i + u * stride < half ? i + u * stride : i;
            x[u] = cost[j];
            y[u] = cost[quads - 1 - j];
        }
#pragma unroll
        for (int u = 0; u < kProUnroll; ++u)
            diff |= (x[u].x ^ flip_word(y[u].w, U16)) | (x[u].y ^ flip_word(y[u].z, U16)) |
                    (x[u].z ^ flip_word(y[u].y, U16)) | (x[u].w ^ flip_word(y[u].x, U16));
        if (diff != 0u || (i + kProUnroll * stride < half && found())) break;
    }
    return diff != 0u;
}

template <bool U16>
__global__ __launch_bounds__(kProThreads) void prologue_kernel(const PrologueArgs a) {
    const uint64_t id = (uint64_t)blockIdx.x * kProThreads + threadIdx.x, stride = (uint64_t)gridDim.x * kProThreads;
    for (uint64_t i = id; i < a.copies; i += stride) a.dst[i] = a.src[i];
    if (!a.cost) return;
    const bool diff = flip_differs<U16>(a.cost, a.quads, id, stride, [&] {
        return __hip_atomic_load(a.word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 16 != 0u;
    });
    // One counter: workgroups done, and 2^16 for each that found a difference.
    const uint32_t mine = __syncthreads_or(diff) ? 0x10001u : 1u;
    if (threadIdx.x == 0) {
        const uint32_t v = mine + __hip_atomic_fetch_add(a.word, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((v & 0xffffu) == gridDim.x) {
            __hip_atomic_store(a.word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(a.answer, 2u * a.ticket + (v >> 16 ? 1u : 0u), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// Job blockIdx.y, its pieces over the blocks of a row; counted as above, a
// counter per job (thousands of additions to one word took 100 us). The last
// workgroup of a job writes its flag to the host, the last of all the ticket,
// after every flag. (A flag written by every workgroup that found a difference,
// 64 fenced stores to the host a job, cost a batch of 16 3-SAT instances at
// n = 20 60 us.)
__global__ __launch_bounds__(kProThreads) void flip_batch_kernel(FlipJob* jobs, uint32_t* flags, uint32_t* word,
                                                                 uint32_t ticket, uint32_t* answer) {
    const FlipJob j = jobs[blockIdx.y];
    const uint64_t id = (uint64_t)blockIdx.x * kProThreads + threadIdx.x, stride = (uint64_t)gridDim.x * kProThreads;
    auto none = [] { return false; };
    const bool diff = j.u16 ? flip_differs<true>(j.cost, j.quads, id, stride, none)
                            : flip_differs<false>(j.cost, j.quads, id, stride, none);
    const uint32_t mine = __syncthreads_or(diff) ? 0x10001u : 1u;
    if (threadIdx.x == 0) {
        const uint32_t w =
            mine + __hip_atomic_fetch_add(&jobs[blockIdx.y].done, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((w & 0xffffu) != gridDim.x) return;
        if (w >> 16) {
            __hip_atomic_store(&flags[blockIdx.y], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __threadfence_system();
        }
        const uint32_t v = 1u + __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v == gridDim.y) {
            __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __threadfence_system();
            __hip_atomic_store(answer, ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

template <int NP, bool U16, int W>
hipError_t launch_np(const CostArgs& a, hipStream_t s) {
    hipLaunchKernelGGL((cost_kernel<NP, U16, W>), dim3(cost_blocks(a.n, W)), dim3(kCostThreads), 0, s, a);
    return hipGetLastError();
}
template <int NP, bool U16, int W>
hipError_t launch_batch_np(const CostArgs* args, const uint32_t* first, int count, uint32_t blocks, hipStream_t s) {
    hipLaunchKernelGGL((cost_batch_kernel<NP, U16, W>), dim3(blocks), dim3(kCostThreads), 0, s, args, first, count);
    return hipGetLastError();
}

// Calls f.run<NP, U16, W>() with enough planes for counts up to `clauses`.
template <typename F>
hipError_t cost_dispatch(int dtype, int clauses, int words, F&& f) {
    const int need = 32 - __builtin_clz((unsigned)clauses | 1u);
    auto by_words = [&](auto np, auto u16) {
        return words == 4 ? f(np, u16, std::integral_constant<int, 4>{}) : f(np, u16, std::integral_constant<int, 1>{});
    };
    if (dtype == 1) {
        if (need <= 6) return by_words(std::integral_constant<int, 6>{}, std::false_type{});
        return by_words(std::integral_constant<int, 8>{}, std::false_type{});
    }
    if (need <= 12) return by_words(std::integral_constant<int, 12>{}, std::true_type{});
    return by_words(std::integral_constant<int, 16>{}, std::true_type{});
}

}  // namespace

hipError_t launch_cost(const CostArgs& a, int dtype, hipStream_t s) {
    return cost_dispatch(dtype, a.num_clauses, cost_words(1ull << a.n), [&](auto np, auto u16, auto w) {
        return launch_np<np.value, u16.value, w.value>(a, s);
    });
}

hipError_t launch_prologue(const PrologueArgs& a, int dtype, hipStream_t s) {
    if (a.cost && a.quads < 2) return hipErrorInvalidValue;
    constexpr uint64_t kPer = (uint64_t)kProThreads * kProUnroll;
    const uint64_t check = a.cost ? (a.quads / 2 + kPer - 1) / kPer : 1;
    const uint64_t copy = (a.copies + kProThreads - 1) / kProThreads;
    const uint64_t want = check > copy ? check : copy;
    const dim3 grid((uint32_t)(want < 1024 ? want : 1024)), block(kProThreads);
    if (dtype == 1) hipLaunchKernelGGL(prologue_kernel<false>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(prologue_kernel<true>, grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_flip_batch(FlipJob* jobs, int count, uint32_t max_quads, uint32_t* flags, uint32_t* word,
                             uint32_t ticket, uint32_t* answer, hipStream_t s) {
    if (count < 1 || count > 65535 || max_quads < 2) return hipErrorInvalidValue;
    constexpr uint32_t kPer = kProThreads * kProUnroll;
    const uint32_t want = (max_quads / 2 + kPer - 1) / kPer;
    hipLaunchKernelGGL(flip_batch_kernel, dim3(want < 64 ? want : 64, (uint32_t)count), dim3(kProThreads), 0, s, jobs,
                       flags, word, ticket, answer);
    return hipGetLastError();
}

hipError_t launch_cost_batch(const CostArgs* args, const uint32_t* first, int count, uint32_t blocks, int dtype,
                             int max_clauses, int words, hipStream_t s) {
    return cost_dispatch(dtype, max_clauses, words, [&](auto np, auto u16, auto w) {
        return launch_batch_np<np.value, u16.value, w.value>(args, first, count, blocks, s);
    });
}

}  // namespace qnae
