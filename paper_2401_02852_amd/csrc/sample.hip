// Sampling bitstrings from a state (include/qnae.h, qnae_sample).
//
// Measuring the final QAOA state yields x with probability |psi(x)|^2 / norm;
// the instance running time of Section 4.2 counts such draws until one
// satisfies the instance. A draw inverts the cumulative distribution in index
// order: the outcome for a uniform u is the smallest x whose cumulative mass
// exceeds u times the total. The cumulative distribution is never stored per
// amplitude; it is kept at three levels of prefix sums from zero:
//   chunk level  C[i]: sums of chunk masses, sequential within groups of 32
//                chunks and over the groups;
//   tile level   P[t] = C[i] + (sequential sum of the tile masses before t in
//                its chunk), but at most C[i + 1]; tiles of 4096 consecutive
//                amplitudes;
//   segments     S[k]: where each 256 amplitudes start in their tile (sums of
//                16 consecutive probabilities, their block-wide exclusive scan).
// The first two are nondecreasing by construction: sequential sums of nonnegative
// terms are, FP64 addition of a fixed offset keeps order, and the bound by the next
// chunk's start takes back the unit by which (C + before) + tile can round above C +
// (before + tile). The search counts the places at or below its target and relies
// on it: its tile never starts above the target. The in-tile scan is a shuffle tree whose rounding may differ from a sequential
// sum, so a draw takes the highest segment with mass whose start is at or below
// its remainder, in it the highest lane of four amplitudes likewise and, if
// rounding carries the remainder past that lane's walk, the lane's last nonzero
// probability. Probabilities are FP32 |psi|^2, sums FP64.
//
// A draw is one wave: a 64-way search over P (three or four loads in a row
// instead of a binary search's 14 to 22), the 16 starts of the tile (one cache
// line, written by the pass that sums the tiles, 0.4% more bytes there), and one
// segment of 2 KiB. Rescanning the whole 32 KiB tile per draw had made 100 000
// draws at n = 26 move 3.2 GB: 420 us.
#include "internal.h"

namespace qnae {
namespace {

constexpr int kTile = 1 << kSampleTileBits;  // amplitudes per tile
constexpr int kPer = kTile / 256;            // per thread, consecutive

// LDS slot of probability e: one pad slot per 16 so that threads reading
// their 16 consecutive entries fall in different banks.
__device__ __forceinline__ uint32_t pad(uint32_t e) { return e + (e >> 4); }

struct TileScan {
    double excl;   // sum of the lower threads' sums (block-wide exclusive scan)
    double total;  // sum of the four wave totals in wave order
};

// Stages the probabilities of tile `tile` (amplitudes tile*4096 ..) in LDS and
// scans the per-thread sums. 256 threads.
__device__ TileScan tile_scan(const float2* __restrict__ psi, uint64_t N, uint64_t tile, float* prob,
                              double* wsum) {
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint64_t base = tile * (uint64_t)kTile;
    constexpr int kLoads = kTile / 512;
    // float4s (amplitude pairs) of this tile inside the state: 2048 for every
    // tile when N >= 4096, else N / 2 >= 1 (N is even). Indices past it load
    // the last pair in range and read as zero, so all loads are unconditional
    // and in flight together.
    const uint32_t lim = (uint32_t)min<uint64_t>(N - base, (uint64_t)kTile) / 2u;
    const float4* tp = (const float4*)(psi + base);  // uniform base, 32-bit offsets
    float4 q[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        const uint32_t j = tid + 256u * i;
        q[i] = tp[j < lim ? j : lim - 1u];
        if (j >= lim) q[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        const uint32_t e = 2u * tid + 512u * i;
        prob[pad(e)] = fmaf(q[i].x, q[i].x, q[i].y * q[i].y);
        prob[pad(e + 1)] = fmaf(q[i].z, q[i].z, q[i].w * q[i].w);
    }
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) s += (double)prob[pad(kPer * tid + j)];
    double incl = s;
    for (int off = 1; off < 64; off <<= 1) {
        const double t = __shfl_up(incl, off);
        if (lane >= (uint32_t)off) incl += t;
    }
    const double prev = __shfl_up(incl, 1);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    double woff = 0.0;
    for (uint32_t w = 0; w < wave; ++w) woff += wsum[w];
    TileScan r;
    r.excl = woff + (lane ? prev : 0.0);
    r.total = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
    return r;
}

// Tile masses, and the segment starts of every tile.
constexpr int kSeg = 256, kSegs = kTile / kSeg;  // amplitudes of a segment, segments of a tile
__global__ __launch_bounds__(256) void tile_mass_kernel(const float2* __restrict__ psi, uint64_t N,
                                                         double* __restrict__ mass, double* __restrict__ seg) {
    __shared__ float prob[kTile + kTile / 16];
    __shared__ double wsum[4];
    const TileScan r = tile_scan(psi, N, blockIdx.x, prob, wsum);
    if (threadIdx.x == 0) mass[blockIdx.x] = r.total;
    constexpr uint32_t kThreadsPer = kSeg / kPer;
    if (threadIdx.x % kThreadsPer == 0) seg[(uint64_t)blockIdx.x * kSegs + threadIdx.x / kThreadsPer] = r.excl;
}

// The tile level in three launches. Thread i of the first owns tiles
// [i*chunk, (i+1)*chunk) of the kSampleChunks chunks and writes their prefix
// within the chunk, from zero, and the chunk total. T and chunk are powers of
// two, so a chunk of 16 or more splits into whole runs of 16 tiles: their
// loads are issued together, then summed in tile order. The threads spread
// over 16 workgroups, as each load instruction touches 64 chunks' lines.
constexpr int kRun = 16;

// Workgroups past those copy the uniforms in from pinned host memory.
__global__ __launch_bounds__(64) void chunk_run_kernel(const double* __restrict__ mass, double* __restrict__ pref,
                                                       double* __restrict__ chunk_total, uint32_t T, uint32_t chunk,
                                                       const double* __restrict__ u_host, double* __restrict__ u_dev,
                                                       uint32_t count) {
    if (blockIdx.x >= kSampleChunks / 64) {
        const uint32_t stride = (gridDim.x - kSampleChunks / 64) * 64u;
        for (uint32_t q = (blockIdx.x - kSampleChunks / 64) * 64u + threadIdx.x; q < count; q += stride)
            u_dev[q] = u_host[q];
        return;
    }
    const uint32_t i = blockIdx.x * 64u + threadIdx.x;
    const uint32_t lo = min(T, i * chunk), hi = min(T, lo + chunk);
    double run = 0.0;
    uint32_t t = lo;
    for (; t + kRun <= hi; t += kRun) {
        double v[kRun];
#pragma unroll
        for (int j = 0; j < kRun; ++j) v[j] = mass[t + j];
#pragma unroll
        for (int j = 0; j < kRun; ++j) {
            const double mj = v[j];
            v[j] = run;
            run += mj;
        }
#pragma unroll
        for (int j = 0; j < kRun; ++j) pref[t + j] = v[j];
    }
    for (; t < hi; ++t) {
        pref[t] = run;
        run += mass[t];
    }
    chunk_total[i] = run;
}

// The chunk and tile levels together: P[t] = C[t / chunk] + (prefix within the
// chunk), bounded by the next chunk's start, one tile per thread, and P[T] = the total. Every workgroup forms C
// for itself, 32 groups of 32 chunks: prefixes within the groups, 32 threads
// at once, then over the groups (two chains of 32 additions; one thread over
// all 1024 took 13 us and a launch of its own).
constexpr int kGroup = 32;
static_assert(kSampleChunks == kGroup * kGroup, "groups of chunks");
__global__ __launch_bounds__(256) void chunk_add_kernel(double* __restrict__ pref,
                                                        const double* __restrict__ chunk_total, uint32_t T,
                                                        uint32_t chunk_bits) {
    __shared__ double c[kSampleChunks + kGroup];  // one pad slot per group
    __shared__ double g[kGroup + 1];
    const uint32_t tid = threadIdx.x;
    for (uint32_t i = tid; i < kSampleChunks; i += 256u) c[i + i / kGroup] = chunk_total[i];
    __syncthreads();
    if (tid < kGroup) {
        double acc = 0.0;
        for (int j = 0; j < kGroup; ++j) {
            const uint32_t at = tid * (kGroup + 1) + j;
            const double v = c[at];
            c[at] = acc;
            acc += v;
        }
        g[tid + 1] = acc;
    }
    __syncthreads();
    if (tid == 0) {
        double acc = 0.0;
        g[0] = 0.0;
        for (int j = 1; j <= kGroup; ++j) {
            acc += g[j];
            g[j] = acc;
        }
    }
    __syncthreads();
    const uint32_t t = blockIdx.x * 256u + tid;
    auto start = [&](uint32_t i) { return i < kSampleChunks ? g[i / kGroup] + c[i + i / kGroup] : g[kGroup]; };
    if (t < T) {
        const uint32_t i = t >> chunk_bits;
        const double p = start(i) + pref[t], next = start(i + 1u);
        pref[t] = p < next ? p : next;
    }
    if (t == 0) pref[T] = g[kGroup];
}

// One wave per draw, four to a workgroup. The outcomes go straight to pinned
// host memory, four in one store: no copy follows the launch (of 100 000 draws
// with costs from n = 26, 309 us with copies both ways, 259 us without; two
// draws or four in turn by one wave took as long as one).
template <typename CT>
__global__ __launch_bounds__(256) void sample_kernel(const float2* __restrict__ psi, uint64_t N,
                                                     const double* __restrict__ mass, const double* __restrict__ pref,
                                                     const double* __restrict__ seg, uint32_t T,
                                                     const double* __restrict__ uniforms, uint32_t count,
                                                     const CT* __restrict__ cost, uint64_t* __restrict__ out,
                                                     int32_t* __restrict__ out_cost) {
    __shared__ uint64_t s_out[4];
    __shared__ int32_t s_cost[4];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const double total = pref[T];
    const uint32_t q = blockIdx.x * 4u + wave;
    if (q < count && !(total > 0.0)) {  // zero state: reported to the host as an error
        if (lane == 0) s_out[wave] = ~0ull;
    } else if (q < count) {
        const double target = uniforms[q] * total;
        // largest t with P[t] <= target (P[0] = 0): 64 places of the range at a time
        uint32_t lo = 0, size = T;
        while (size > 1) {
            const uint32_t step = (size + 63u) / 64u;
            const uint32_t t = lo + lane * step;
            const uint64_t le = __ballot(lane * step < size && pref[min(t, T - 1u)] <= target);
            // P is nondecreasing and place 0 at or below, but for a target of 0 * infinity
            const uint32_t k = (uint32_t)__popcll(le | 1ull) - 1u;
            size = min(step, size - k * step);
            lo += k * step;
        }
        // (the three loads go out together; the loop runs only past the last nonzero tile)
        double here = mass[lo], before = pref[lo], start = seg[(uint64_t)lo * kSegs + (lane & (kSegs - 1))];
        while (lo > 0 && !(here > 0.0)) {
            --lo;
            here = mass[lo], before = pref[lo], start = seg[(uint64_t)lo * kSegs + (lane & (kSegs - 1))];
        }
        const double r = target - before;
        // the highest segment of the tile that starts at or below r and has mass
        // (an infinite total can make r not a number: no test holds, the first place is taken)
        int k = 63 - __builtin_clzll(__ballot(lane < kSegs && start <= r) | 1ull);
        for (;; --k) {
            const double s0 = __shfl(start, k);
            const uint64_t base = (uint64_t)lo * kTile + (uint64_t)k * kSeg + 4u * lane;
            float p[4] = {0.f, 0.f, 0.f, 0.f};
            if (base + 2 <= N) {  // (N is even; small states end inside the segment)
                const float4 a = *(const float4*)(psi + base);
                p[0] = fmaf(a.x, a.x, a.y * a.y);
                p[1] = fmaf(a.z, a.z, a.w * a.w);
            }
            if (base + 4 <= N) {
                const float4 b = *(const float4*)(psi + base + 2);
                p[2] = fmaf(b.x, b.x, b.y * b.y);
                p[3] = fmaf(b.z, b.z, b.w * b.w);
            }
            const double mine = (((double)p[0] + (double)p[1]) + (double)p[2]) + (double)p[3];
            double incl = mine;
            for (int off = 1; off < 64; off <<= 1) {
                const double t = __shfl_up(incl, off);
                if (lane >= (uint32_t)off) incl += t;
            }
            const double prev = __shfl_up(incl, 1);
            const double excl = s0 + (lane ? prev : 0.0);
            const uint64_t ok = __ballot(mine > 0.0 && excl <= r);
            if (ok == 0ull && k > 0) continue;
            if (lane == 63u - (uint32_t)__builtin_clzll(ok | 1ull)) {
                double acc = excl;
                int pick = -1, last = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc += (double)p[j];
                    if (p[j] > 0.f && pick < 0) {
                        last = j;
                        if (acc > r) pick = j;
                    }
                }
                const uint64_t x = base + (uint64_t)(pick < 0 ? last : pick);  // rounding put r past this lane's walk
                s_out[wave] = x;
                if (out_cost) s_cost[wave] = cost ? (int32_t)cost[x] : -1;
            }
            break;
        }
    }
    __syncthreads();
    const uint32_t at = blockIdx.x * 4u + threadIdx.x;
    if (threadIdx.x < 4u && at < count) {
        out[at] = s_out[threadIdx.x];
        if (out_cost) out_cost[at] = s_cost[threadIdx.x];
    }
}

}  // namespace

hipError_t launch_sample_masses(const float2* psi, int n, double* mass, double* seg, hipStream_t s) {
    const uint64_t N = 1ull << n;
    hipLaunchKernelGGL(tile_mass_kernel, dim3((uint32_t)((N + kTile - 1) / kTile)), dim3(256), 0, s, psi, N, mass, seg);
    return hipGetLastError();
}

hipError_t launch_sample_prefix(int n, const double* mass, double* pref, double* chunk_scratch,
                                const double* u_host, double* u_dev, int count, hipStream_t s) {
    const uint64_t N = 1ull << n;
    const uint32_t T = (uint32_t)((N + kTile - 1) / kTile);
    static_assert(kSampleChunks % 64 == 0 && kSampleChunks % kRun == 0, "chunk launch shape");
    static_assert(kSegs == kSampleSegs, "room for the segment starts");
    const uint32_t chunk = (T + kSampleChunks - 1) / kSampleChunks;  // T is a power of two
    const uint32_t chunk_bits = (uint32_t)__builtin_ctz(chunk);
    // A uniform a thread while they last: reads of host memory take over a microsecond
    // each, and 16 in turn a thread made up most of 1000 draws
    // (n = 20, 1000 draws 54.6 -> 36.0 us, 10 000 67.1 -> 50.3, 100 000 178 -> 173).
    const uint32_t copiers = ((uint32_t)count + 63u) / 64u;
    hipLaunchKernelGGL(chunk_run_kernel, dim3(kSampleChunks / 64 + (copiers < 512u ? copiers : 512u)), dim3(64), 0, s,
                       mass, pref, chunk_scratch, T, chunk, u_host, u_dev, (uint32_t)count);
    if (hipError_t e = hipGetLastError()) return e;
    hipLaunchKernelGGL(chunk_add_kernel, dim3((T + 255) / 256), dim3(256), 0, s, pref,
                       (const double*)chunk_scratch, T, chunk_bits);
    return hipGetLastError();
}

hipError_t launch_sample_draws(const float2* psi, int n, const void* cost, int cost_dtype, const double* uniforms,
                               int count, const double* mass, const double* pref, const double* seg, uint64_t* out,
                               int32_t* out_cost, hipStream_t s) {
    const uint64_t N = 1ull << n;
    const uint32_t T = (uint32_t)((N + kTile - 1) / kTile);
    if (count <= 0) return hipSuccess;
    const dim3 grid(((uint32_t)count + 3u) / 4u), block(256);
    if (cost_dtype == 2)
        hipLaunchKernelGGL(sample_kernel<uint16_t>, grid, block, 0, s, psi, N, mass, pref, seg, T, uniforms,
                           (uint32_t)count, (const uint16_t*)cost, out, out_cost);
    else
        hipLaunchKernelGGL(sample_kernel<uint8_t>, grid, block, 0, s, psi, N, mass, pref, seg, T, uniforms,
                           (uint32_t)count, (const uint8_t*)cost, out, out_cost);
    return hipGetLastError();
}

}  // namespace qnae
