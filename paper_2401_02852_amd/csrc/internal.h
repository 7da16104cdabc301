// Internal declarations shared by the host runtime and the HIP kernels of
// libqnae.so. Not part of the public ABI (include/qnae.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qnae {

// Where a batch's launches go: to a stream, or into a graph, one node behind the
// other. (Graphs are built node by node: while a stream is being captured the runtime
// refuses other threads' synchronisations and allocations, or they end the capture.)
struct GraphChain {
    hipGraph_t graph = nullptr;
    hipGraphNode_t last = nullptr;
};
struct LaunchTo {
    hipStream_t stream = nullptr;
    GraphChain* chain = nullptr;
    LaunchTo(hipStream_t s) : stream(s) {}
    LaunchTo(GraphChain* c) : chain(c) {}
};
template <typename T>
struct Exactly {
    using type = T;
};
template <typename... P>
hipError_t launch_to(LaunchTo to, dim3 grid, dim3 block, void (*kernel)(P...), typename Exactly<P>::type... args) {
    void* params[] = {(void*)&args...};
    if (!to.chain) return hipLaunchKernel((const void*)kernel, grid, block, params, 0, to.stream);
    hipKernelNodeParams k{};
    k.func = (void*)kernel;
    k.gridDim = grid;
    k.blockDim = block;
    k.kernelParams = params;
    GraphChain& c = *to.chain;
    hipGraphNode_t node = nullptr;
    if (hipError_t e = hipGraphAddKernelNode(&node, c.graph, c.last ? &c.last : nullptr, c.last ? 1 : 0, &k)) return e;
    c.last = node;
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Cost diagonal (violated clause count per basis state)
// ---------------------------------------------------------------------------

// One clause after host normalisation. With M = the set of variables the
// clause touches and P = the variables whose literal is negated, the clause is
// violated at x exactly when ((x ^ P) & M) is 0 (all literals false) or M (all
// true; NAE) or only when it is 0 (k-SAT: full_tab is empty). The low 5 bits
// are folded into two 32-bit tables over the position j of x inside an aligned
// run of 32 states: zero_tab bit j says ((j ^ P) & M & 31) == 0, full_tab bit
// j says it equals M & 31.
struct ClauseRec {
    uint32_t mask_hi_lo, mask_hi_hi;  // M with bits 0..4 cleared (low / high word)
    uint32_t pat_lo, pat_hi;          // P
    uint32_t zero_tab, full_tab;
};

struct CostArgs {
    const ClauseRec* clauses;
    int32_t num_clauses;
    int32_t n;
    void* cost;                 // uint8 or uint16 [2^n]
    unsigned long long* zeros;  // optional counter of states with cost 0
};

// C(x) for x < 2^a.n.
hipError_t launch_cost(const CostArgs& a, int dtype, hipStream_t s);
// Runs of 32 states a thread counts, for this many states in one launch: four
// share the work per clause, once that leaves enough waves to fill the chip
// (one run and four, us per call: n = 23, k = 3 20.5 and 22.9, k = 5 26.4 and
// 34.1; n = 24 24.0 and 23.9, 32.6 and 36.3; n = 25 30.8 and 28.3, 44.2 and 45.0;
// n = 26 43.4 and 37, 67 and 63.5).
inline int cost_words(uint64_t states) { return states >= (1ull << 25) ? 4 : 1; }
// 256-thread blocks of a diagonal of 2^n states.
inline uint32_t cost_blocks(int n, int words) {
    const int bits = words == 4 ? 15 : 13;  // states of a block
    return n > bits ? 1u << (n - bits) : 1u;
}
// Many diagonals of one cost type: instance i owns blocks first[i] ..
// first[i+1]-1, cost_blocks(n, words) of them. max_clauses bounds every
// instance's clause count.
hipError_t launch_cost_batch(const CostArgs* args, const uint32_t* first, int count, uint32_t blocks, int dtype,
                             int max_clauses, int words, hipStream_t s);

// Launch ahead of a run: copies `copies` 16-byte pieces from src (pinned host
// memory) to dst and, with a cost (of `quads` >= 2 16-byte pieces), checks the
// diagonal for flip symmetry, cost[x] == cost[2^n - 1 - x] for every x. word:
// a device word that is zero before and after; the last workgroup writes
// 2 * ticket + (0 symmetric, 1 not) to *answer (pinned).
struct PrologueArgs {
    uint4* dst;
    const uint4* src;
    uint64_t copies;
    const uint4* cost;
    uint64_t quads;
    uint32_t* word;
    uint32_t* answer;
    uint32_t ticket;
};
hipError_t launch_prologue(const PrologueArgs& a, int dtype, hipStream_t s);

// The same check of many diagonals: flags[i] (pinned, zero before) is set to 1
// when job i's is not symmetric, then the ticket is written to *answer
// (pinned). word as above.
struct FlipJob {
    const uint4* cost;
    uint32_t quads;  // 16-byte pieces of the diagonal, >= 2
    uint32_t u16;
    uint32_t done;  // workgroups of this job that have ended, and 2^16 for each that found a difference; 0 before
    uint32_t pad[3];
};
hipError_t launch_flip_batch(FlipJob* jobs, int count, uint32_t max_quads, uint32_t* flags, uint32_t* word,
                             uint32_t ticket, uint32_t* answer, hipStream_t s);

// A phase table row: out[c] = (re + i im) exp(sign i g c), c = 0 .. m; |g| <= 3.2, as
// the phase is formed from the rounded product g c.
struct PhaseRow {
    double g, re, im, sign;
    float2* out;
    int32_t m, pad;
};
hipError_t launch_phase_rows(const PhaseRow* rows, int count, int max_m, hipStream_t s);

// ---------------------------------------------------------------------------
// State sweeps
// ---------------------------------------------------------------------------

// Mixer of one layer in the form used on the device. With t = tan(beta) when
// |tan(beta)| <= 1:  R(beta) = cos(beta) (I - i t X); otherwise, with
// t = -cot(beta):    R(beta) = (-i sin(beta)) X (I - i t X).
// Each butterfly therefore costs two FMAs per amplitude. The scalar factor is
// folded into the next phase table (or the readout). The X of the cot form
// (`flip`) is not applied: X on every qubit of the layer is a relabelling
// x -> NOT x of the stored state, so the runtime tracks the parity of flipped
// layers and reads the cost at the complemented index where it matters
// (phase and readout), undoing the relabelling only if the final state is
// returned.
struct MixForm {
    float t;
    int flip;
};

// Sweep kinds: which steps a sweep performs.
enum SweepKind {
    SK_FIRST = 0,     // phase table 0 as initial state, mix, store
    SK_MIDDLE = 1,    // load, mix, store
    SK_BOUNDARY = 2,  // load, mix (layer l), phase (l + 1), mix (l + 1), store
    SK_FINAL = 3,     // load, mix, readout partials (optional store)
    SK_P0 = 4,        // phase table 0 as state, readout (p = 0)
};

struct SweepArgs {
    float2* psi;           // state written (and read, unless psi_in is set)
    const float2* psi_in;  // state read by the load (== psi for in-place sweeps)
    const void* cost;
    const float2* lut;     // phase table of this sweep (lut_len entries)
    double* partials;      // 3 doubles per block for readout kinds
    int32_t n;
    int32_t nw;            // n - TB: block-index bits
    uint64_t tile_bits;    // global bits spanned by a tile
    uint8_t pos[16];       // tile bit i -> bit pos[i] of x (pos[0..3] = 0..3)
    uint64_t wmask;        // bits of x outside the tile (filled by the tile index)
    int32_t lut_len;
    uint32_t pre_mask;     // tile bits mixed before the phase
    uint32_t post_mask;    // tile bits mixed after the phase
    float pre_t, post_t;
    float2 store_scale;    // readout kinds with store: final scalar factor
    int32_t store;         // readout kinds: also store the state
    int32_t cflip;         // read the cost at the complemented index
    // Half-state sweeps (NAE global-flip symmetry): the state and cost hold
    // only x < 2^(n-1); the amplitude of x with bit n-1 set is the one at
    // its complement. With half set, tile bit vbit (pos[vbit] = n-1) is the
    // virtual bit: flipping it maps a stored index y to mir - y, mir =
    // 2^(n-1) - 1. Without a virtual bit (vbit < 0) a half sweep is a plain
    // sweep over n-1 bits.
    int32_t half;
    int32_t vbit;          // -1 or TB - 1
    int32_t expand;        // readout kinds with store, half: also store the upper half (psi holds 2^n)
    uint64_t mir;
    // Checkpointing boundary sweep (gradient forward pass): the state right
    // after the pre mixing, which completes a layer, times ckpt_scale (that
    // layer's mixer factor), in natural order (element x at x ^ (2^n - 1)
    // when cflip) to ckpt.
    float2* ckpt;
    float2 ckpt_scale;
};

hipError_t launch_sweep(int tb, int dtype, int kind, const SweepArgs& a, hipStream_t s);
// A boundary sweep that also stores a checkpoint (a.ckpt), 13-bit tiles.
hipError_t launch_sweep_ckpt(int dtype, const SweepArgs& a, hipStream_t s);

// One sweep step over `count` states at once. Instance i owns blocks
// first[i] .. first[i+1]-1 (first has count+1 entries, first[count] =
// blocks), one per tile of its own geometry; args[i].partials receives 3
// doubles per tile for readout kinds. Every instance uses tiles of tb bits
// (12, 13 or 14). virt: every instance's group holds the virtual bit
// (args[i].vbit >= 0), or none does. l1: sweep_l1 of every instance.
hipError_t launch_sweep_batch(int tb, int dtype, int kind, const SweepArgs* args, const uint32_t* first, int count,
                              uint32_t blocks, LaunchTo to, bool virt, int l1);
// Does a launch of this kind over a group with these mix masks pass its tiles
// through register layouts 2 and 3? 1 yes, 2 no. (A launch that holds one that does
// passes every tile through it.)
int sweep_l1(int tb, int kind, uint32_t pre_mask, uint32_t post_mask);
hipError_t launch_reverse(float2* psi, uint64_t N, LaunchTo to);

// Do `rows` phase table rows of `len` entries fit `room` entries? (In 64 bits: a
// call may have up to 100000 rows of 65536.)
__host__ __device__ constexpr bool rows_fit(int32_t rows, int32_t len, int32_t room) {
    return (int64_t)rows * len <= room;
}

// Whole circuit for n <= 14 in one workgroup (resident.hip).
struct ResidentArgs {
    const float2* state_in;  // optional initial state (true scale); |+> when null
    const void* cost;
    const float2* luts;    // p (or 1 when p = 0) tables of lut_len entries
    const MixForm* forms;  // p entries (device)
    float2* state_out;     // optional final state (scaled by store_scale)
    double* out;           // 3 doubles (unscaled sums)
    float2 store_scale;
    int32_t n, p, lut_len;
};

hipError_t launch_resident(int dtype, const ResidentArgs& a, hipStream_t s);

// The same with the tables in the kernel arguments (no copy ahead of the
// launch): p phase tables of lut_len entries (one when p = 0), then the p
// mixer forms, each stored in one float2 slot; a.luts and a.forms unused.
constexpr int kResidentInline = 448;
struct ResidentInlineArgs {
    ResidentArgs a;
    float2 tab[kResidentInline];
};
hipError_t launch_resident_inline(int dtype, const ResidentInlineArgs& a, hipStream_t s);

// ---------------------------------------------------------------------------
// Adjoint (gradient) sweeps: the reverse pass carries the adjoint state lam
// and the forward state psi together and applies the inverse of each layer to
// both (psi is uncomputed). The inverse mixers use the forward sweeps'
// butterflies (I - i t X) with |t| <= 1: the layer's scalar factor is folded
// into its inverse phase table, the X on every qubit of the cotangent form is
// a relabelling (index x holds element x ^ (2^n - 1)), and the inner products
// taken between butterflies carry the factor the butterflies left out.
// Tiles as in the forward sweeps, TB = 13.
// ---------------------------------------------------------------------------

enum AdjointKind {
    AK_MIDDLE = 0,    // inverse mixer of one group (b-layer i)
    AK_BOUNDARY = 1,  // inverse mixer (i), inverse phase (i), inverse mixer (i + 1) of one group
    AK_END = 2,       // inverse mixer (i), inverse phase (i): last op of a reverse segment
};

struct AdjointArgs {
    float2* lam;
    float2* psi;
    const void* cost;
    const float2* lut;     // F exp(+i gamma c), c = 0 .. lut_len - 1, F the layer's mixer factor
    double* partials;      // 3 per tile: Im<lam|X|psi> (pre group), Im<lam|C|psi>, Im<lam|X|psi> (post group)
    int32_t n, nw, lut_len;
    uint64_t tile_bits, wmask;
    uint8_t pos[16];
    uint32_t pre_mask, post_mask;
    // Butterfly own' = own - i t partner. Before each butterfly the pair term
    // is added with weight w, then w *= r (r = |one qubit's factor|^2): w
    // starts at r^k for k qubits of the layer mixed by earlier sweeps.
    float pre_t, pre_r, pre_w, post_t, post_r, post_w;
    uint64_t cost_flip;  // 0 or 2^n - 1: the phase of element x reads cost[x ^ cost_flip]
    int32_t psi_flip;    // psi of element x sits at x ^ (2^n - 1) (relabelled against lam)
    // Half state (flip-symmetric cost): both states hold x < 2^(n-1). virt:
    // the group mixes bit n-1 as tile bit 12, which maps a stored index y to
    // mir - y, mir = 2^(n-1) - 1; other groups run as full sweeps over n-1
    // bits. Relabelling is the identity there (psi_flip = cost_flip = 0).
    int32_t virt;
    uint64_t mir;
    int32_t store_psi;
    float w_psucc, w_energy;  // weigh: lam = (w_psucc [C = 0] + w_energy C) psi instead of a load
};

constexpr int kAdjointTileBits = 13;
// weigh: the middle kind forms lam from psi (first sweep of the reverse pass,
// no relabelling) instead of loading it.
hipError_t launch_adjoint(int dtype, int kind, const AdjointArgs& a, hipStream_t s, bool weigh = false);


// Whole gradient for n <= 13 in one workgroup (resident_grad.hip): forward
// (checkpoints of psi every `every` layers in ckpt), readout, then the reverse pass with psi refreshed at checkpoints.
struct ResidentGradArgs {
    const void* cost;
    const float2* luts;    // p forward tables exp(-i gamma_l c)
    const float2* cs;      // p (cos beta_l, sin beta_l)
    float2* ckpt;          // (p - 1) / every states of 2^n
    double* out;           // pinned host memory: 3 readout sums, then dgamma[p], then dbeta[p]
    double w_psucc, w_energy;
    int32_t n, p, lut_len, every;
};
// One workgroup per entry of args (count entries, all of one cost type).
hipError_t launch_resident_grad_batch(int dtype, const ResidentGradArgs* args, int count, hipStream_t s);
hipError_t launch_resident_batch(int dtype, const ResidentArgs* args, int count, LaunchTo to);

// Sum of 3-double block partials into out[3], FP64.
hipError_t launch_final_reduce(const double* partials, int64_t blocks, double* out, hipStream_t s);
// Instance i: sum of blocks[i] triples at partials[i] -> outs[i][0..2].
hipError_t launch_final_reduce_batch(const double* const* partials, const uint32_t* blocks, double* const* outs,
                                     int count, LaunchTo to);

// Sum i of `count`: `blocks` triples at partials + 3 blocks i -> out[3 i ..].
hipError_t launch_final_reduce_rows(const double* partials, int64_t blocks, double* out, int count, hipStream_t s);

// ---------------------------------------------------------------------------
// Sampling outcomes of a state (sample.hip)
// ---------------------------------------------------------------------------

constexpr int kSampleTileBits = 12;
constexpr int kSampleChunks = 1024;  // tile-prefix chunks
constexpr int kSampleSegs = 16;      // segments of a tile
// Tile masses of psi (2^n complex64; ceil(2^n / 4096) doubles) and segment starts
// (kSampleSegs per tile).
hipError_t launch_sample_masses(const float2* psi, int n, double* mass, double* seg, hipStream_t s);
// Their prefix sums: pref (one more than mass), chunk (kSampleChunks doubles of
// scratch); also copies `count` uniforms from pinned u_host to u_dev.
hipError_t launch_sample_prefix(int n, const double* mass, double* pref, double* chunk, const double* u_host,
                                double* u_dev, int count, hipStream_t s);
// `count` outcomes for the given uniforms in [0, 1) from those, to pinned host
// memory. out[q] = ~0 marks a zero state. out_cost, if not null, receives C at
// each outcome (or -1 without a cost diagonal).
hipError_t launch_sample_draws(const float2* psi, int n, const void* cost, int cost_dtype, const double* uniforms,
                               int count, const double* mass, const double* pref, const double* seg, uint64_t* out,
                               int32_t* out_cost, hipStream_t s);

}  // namespace qnae
