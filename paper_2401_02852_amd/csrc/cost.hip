// Cost diagonal kernel: C(x) = number of NAE-violated clauses, for every basis
// state x (Section 3.2, eq. knaesatobj; Appendix A.2, eq. demorgannae).
//
// Bit-sliced: each thread owns an aligned run of 32 consecutive states. For one
// clause, its violation pattern over the run is a 32-bit word: the part of the
// clause on variables >= 5 is constant over the run (one compare against the
// thread's index), and the part on variables 0..4 is a per-clause table built
// on the host. The per-state counters are kept as NP bit-planes (a vertical
// counter); clauses go in eight at a time through a carry-save adder tree, so
// one clause costs about 9 integer operations per 32 states (clauses on
// variables >= 5 only are constant over the run and are counted as one
// integer instead). At the end the planes are transposed into bytes (uint8)
// or half-words (uint16) and written with 16-byte stores.
#include "internal.h"

namespace qnae {
namespace {

// Thread `tid` of one diagonal: states [32 tid, 32 tid + 32).
template <int NP, bool WIDE, bool U16>
__device__ __forceinline__ void cost_chunk(const CostArgs& a, uint64_t tid) {
    const uint64_t nthreads = a.n >= 5 ? (1ull << (a.n - 5)) : 1ull;
    uint32_t zeros = 0;
    if (tid < nthreads) {
        const uint64_t xbase = tid << 5;
        const uint32_t xlo = (uint32_t)xbase, xhi = (uint32_t)(xbase >> 32);
        uint32_t plane[NP];
#pragma unroll
        for (int b = 0; b < NP; ++b) plane[b] = 0u;
        // Violation word of clause i over the 32 states.
        auto viol = [&](int i) -> uint32_t {
            const ClauseRec r = a.clauses[i];
            const uint32_t hlo = (xlo ^ r.pat_lo) & r.mask_hi_lo;
            bool none, all;
            if (WIDE) {
                const uint32_t hhi = (xhi ^ r.pat_hi) & r.mask_hi_hi;
                none = (hlo | hhi) == 0u;
                all = (hlo == r.mask_hi_lo) && (hhi == r.mask_hi_hi);
            } else {
                none = hlo == 0u;
                all = hlo == r.mask_hi_lo;
            }
            return (none ? r.zero_tab : 0u) | (all ? r.full_tab : 0u);
        };
        // Adds carry * 2^b0 to the counter (ripple through the planes above).
        auto add_at = [&](int b0, uint32_t carry) {
#pragma unroll
            for (int b = 0; b < NP; ++b) {
                if (b < b0) continue;
                const uint32_t t = plane[b] & carry;
                plane[b] ^= carry;
                carry = t;
            }
        };
        // Full adder per bit: x + p + q = x' + 2 carry.
        auto csa = [](uint32_t& x, uint32_t p, uint32_t q) -> uint32_t {
            const uint32_t t = x ^ p;
            const uint32_t carry = (t & q) | (~t & x);
            x = t ^ q;
            return carry;
        };
        // Eight clauses at a time through a carry-save tree (7 full adders
        // into the planes of weight 1, 2 and 4, one ripple from weight 8):
        // the counter value after the block is exactly the sum it had plus
        // the eight violation bits, per state.
        int i = 0;
        for (; i + 8 <= a.num_low; i += 8) {
            const uint32_t c2a = csa(plane[0], viol(i), viol(i + 1));
            const uint32_t c2b = csa(plane[0], viol(i + 2), viol(i + 3));
            const uint32_t c2c = csa(plane[0], viol(i + 4), viol(i + 5));
            const uint32_t c2d = csa(plane[0], viol(i + 6), viol(i + 7));
            const uint32_t c4a = csa(plane[1], c2a, c2b);
            const uint32_t c4b = csa(plane[1], c2c, c2d);
            add_at(3, csa(plane[2], c4a, c4b));
        }
        for (; i < a.num_low; ++i) add_at(0, viol(i));
        // The other clauses only have variables >= 5: each is violated on all
        // 32 states of the run or on none, so they are counted as one integer
        // (about 5 operations per clause instead of 9) and the count is added
        // to every state's counter once, as a ripple-carry over the planes.
        uint32_t cnt = 0u;
        for (; i < a.num_clauses; ++i) cnt += viol(i) & 1u;
        uint32_t carry = 0u;
#pragma unroll
        for (int b = 0; b < NP; ++b) {
            const uint32_t cb = 0u - ((cnt >> b) & 1u);
            const uint32_t t = plane[b] ^ cb;
            const uint32_t nc = (plane[b] & cb) | (t & carry);
            plane[b] = t ^ carry;
            carry = nc;
        }
        const uint32_t valid = a.n >= 5 ? 0xffffffffu : ((1u << (1u << a.n)) - 1u);
        uint32_t any = 0u;
#pragma unroll
        for (int b = 0; b < NP; ++b) any |= plane[b];
        zeros = (uint32_t)__popc(~any & valid);

        if (!U16) {
            // 32 bytes: byte j = sum_b bit j of plane b, shifted to bit b.
            uint32_t word[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                uint32_t wv = 0u;
#pragma unroll
                for (int b = 0; b < NP; ++b) {
                    const uint32_t nib = (plane[b] >> (4 * q)) & 0xfu;
                    wv |= ((nib * 0x00204081u) & 0x01010101u) << b;
                }
                word[q] = wv;
            }
            uint8_t* out = (uint8_t*)a.cost + xbase;
            if (a.n >= 5) {
                ((uint4*)out)[0] = make_uint4(word[0], word[1], word[2], word[3]);
                ((uint4*)out)[1] = make_uint4(word[4], word[5], word[6], word[7]);
            } else {
                for (uint32_t j = 0; j < (1u << a.n); ++j) out[j] = (uint8_t)(word[j >> 2] >> (8 * (j & 3)));
            }
        } else {
            // 64 bytes: half-word j = sum_b bit j of plane b, shifted to bit b.
            uint32_t word[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                uint32_t wv = 0u;
#pragma unroll
                for (int b = 0; b < NP; ++b) {
                    const uint32_t pair = (plane[b] >> (2 * q)) & 3u;
                    wv |= ((pair * 0x8001u) & 0x10001u) << b;
                }
                word[q] = wv;
            }
            uint16_t* out = (uint16_t*)a.cost + xbase;
            if (a.n >= 5) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    ((uint4*)out)[q] = make_uint4(word[4 * q], word[4 * q + 1], word[4 * q + 2], word[4 * q + 3]);
            } else {
                for (uint32_t j = 0; j < (1u << a.n); ++j) out[j] = (uint16_t)(word[j >> 1] >> (16 * (j & 1)));
            }
        }
    }
    if (a.zeros) {
        __shared__ uint32_t blk;
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

template <int NP, bool WIDE, bool U16>
__global__ __launch_bounds__(256) void cost_kernel(const CostArgs a) {
    cost_chunk<NP, WIDE, U16>(a, (uint64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// Many diagonals at once: instance i owns blocks first[i] .. first[i+1]-1.
template <int NP, bool WIDE, bool U16>
__global__ __launch_bounds__(256) void cost_batch_kernel(const CostArgs* args, const uint32_t* first, int count) {
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    const CostArgs a = args[lo];
    cost_chunk<NP, WIDE, U16>(a, (uint64_t)(blockIdx.x - first[lo]) * blockDim.x + threadIdx.x);
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

// Job blockIdx.y, its pieces over the blocks of a row. The last workgroup of
// all writes the ticket, after every flag. Ended workgroups are counted per
// job first: thousands of additions to one word took 100 us.
__global__ __launch_bounds__(kProThreads) void flip_batch_kernel(FlipJob* jobs, uint32_t* flags, uint32_t* word,
                                                                 uint32_t ticket, uint32_t* answer) {
    const FlipJob j = jobs[blockIdx.y];
    const uint64_t id = (uint64_t)blockIdx.x * kProThreads + threadIdx.x, stride = (uint64_t)gridDim.x * kProThreads;
    auto none = [] { return false; };
    const bool diff = j.u16 ? flip_differs<true>(j.cost, j.quads, id, stride, none)
                            : flip_differs<false>(j.cost, j.quads, id, stride, none);
    const bool any = __syncthreads_or(diff) != 0;
    if (threadIdx.x == 0) {
        if (any) {
            __hip_atomic_store(&flags[blockIdx.y], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __threadfence_system();
        }
        const uint32_t w =
            1u + __hip_atomic_fetch_add(&jobs[blockIdx.y].done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (w != gridDim.x) return;
        const uint32_t v = 1u + __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v == gridDim.y) {
            __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __threadfence_system();
            __hip_atomic_store(answer, ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

template <int NP, bool U16>
hipError_t launch_np(const CostArgs& a, bool wide, hipStream_t s) {
    const uint64_t nthreads = a.n >= 5 ? (1ull << (a.n - 5)) : 1ull;
    const uint64_t blocks = (nthreads + 255) / 256;
    if (wide)
        hipLaunchKernelGGL((cost_kernel<NP, true, U16>), dim3((uint32_t)blocks), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((cost_kernel<NP, false, U16>), dim3((uint32_t)blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_cost(const CostArgs& a, int dtype, bool wide, hipStream_t s) {
    // Enough planes to count up to the number of (normalised) clauses.
    const int need = 32 - __builtin_clz((unsigned)a.num_clauses | 1u);
    if (dtype == 1) {
        if (need <= 6) return launch_np<6, false>(a, wide, s);
        return launch_np<8, false>(a, wide, s);
    }
    if (need <= 12) return launch_np<12, true>(a, wide, s);
    return launch_np<16, true>(a, wide, s);
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
                             int max_clauses, bool wide, hipStream_t s) {
    const int need = 32 - __builtin_clz((unsigned)max_clauses | 1u);
    if (dtype == 1) {
        if (wide) hipLaunchKernelGGL((cost_batch_kernel<8, true, false>), dim3(blocks), dim3(256), 0, s, args, first, count);
        else hipLaunchKernelGGL((cost_batch_kernel<8, false, false>), dim3(blocks), dim3(256), 0, s, args, first, count);
    } else if (need <= 12) {
        if (wide) hipLaunchKernelGGL((cost_batch_kernel<12, true, true>), dim3(blocks), dim3(256), 0, s, args, first, count);
        else hipLaunchKernelGGL((cost_batch_kernel<12, false, true>), dim3(blocks), dim3(256), 0, s, args, first, count);
    } else {
        if (wide) hipLaunchKernelGGL((cost_batch_kernel<16, true, true>), dim3(blocks), dim3(256), 0, s, args, first, count);
        else hipLaunchKernelGGL((cost_batch_kernel<16, false, true>), dim3(blocks), dim3(256), 0, s, args, first, count);
    }
    return hipGetLastError();
}

}  // namespace qnae
