// qnae_qaoa_grad: gradient of w_psucc p_succ + w_energy E[C] by a hand-written
// adjoint pass (include/qnae.h). See adjoint.hip for the formulas.
//
// n <= 13: one workgroup does the forward pass, the readout and the reverse
// pass, with both states in registers from n = 10 on, in LDS below
// (resident_grad.hip). Larger n: the forward pass runs as one sweep
// plan that also stores the state after every `every` layers (checkpoints:
// the ends of segments); then for each segment from the last, reverse sweeps
// take lam (the first one forms lam = W psi_p) and that segment's checkpoint
// (psi, uncomputed in place) through the inverse layers, summing the inner
// products per tile. With a flip-symmetric cost psi and lam are symmetric too
// and both passes keep x < 2^(n-1) only; every sum over the stored elements
// is then half of the whole one.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <utility>
#include <vector>

#include "host.h"

using namespace qnae_host;
using qnae::MixForm;
using qnae::SweepArgs;

namespace {

// g modulo 2 pi, for phases exp(i g c) with whole c that are formed from the product
// g c: its rounding turns them by up to g c 2^-53, which shows in FP32 from g c = 1e8
// on. The library's sine and cosine reduce their argument exactly.
double reduced(double g) {
    return std::fabs(g) <= 3.2 ? g : std::atan2(std::sin(g), std::cos(g));
}

// The gradients of the jobs `pick` (n <= 13), one launch per cost type. Uploaded:
// a record per phase table row, the (cos, sin) of the mixers and the kernel
// arguments; the tables are built on the device, the results come back
// through pinned memory that the kernels write.
int resident_grads(qnae_ctx* ctx, const qnae_grad_job* jobs, const std::vector<int>& pick, double w_psucc,
                   double w_energy, int every, qnae_result* out, hipStream_t s) {
    DrainOnExit drain{s};
    Blob B, C, T;  // uploaded; checkpoints; tables
    size_t rows = 0;
    int max_m = 0;
    std::vector<int> group[2];
    for (int i : pick) {
        rows += (size_t)jobs[i].p;
        max_m = std::max(max_m, jobs[i].m);
        group[jobs[i].cost_dtype == QNAE_U16 ? 1 : 0].push_back(i);
    }
    const size_t row_at = B.take(sizeof(qnae::PhaseRow) * rows);
    const size_t cs_at = B.take(sizeof(float2) * rows);
    size_t args_at[2];
    for (int g = 0; g < 2; ++g) args_at[g] = B.take(sizeof(qnae::ResidentGradArgs) * group[g].size());
    B.take(16);
    const size_t out_at = B.take(sizeof(double) * (3 * pick.size() + 2 * rows));  // pinned only
    for (int i : pick) {
        const int nck = jobs[i].p > 1 ? (jobs[i].p - 1) / every : 0;
        C.take(sizeof(float2) * ((size_t)1 << jobs[i].n) * (size_t)std::max(nck, 1));
        T.take(sizeof(float2) * (size_t)std::max(jobs[i].p, 1) * (size_t)(jobs[i].m + 1));
    }
    HIP_TRY(ctx->h_blob.reserve(B.size));
    HIP_TRY(ctx->g_blob.reserve(B.size));
    HIP_TRY(ctx->g_states.reserve(C.size));
    HIP_TRY(ctx->g_tables.reserve(T.size));
    char* const h = (char*)ctx->h_blob.ptr;
    char* const d = (char*)ctx->g_blob.ptr;
    qnae::PhaseRow* const hr = (qnae::PhaseRow*)(h + row_at);
    float2* const hc = (float2*)(h + cs_at);
    double* const ho = (double*)(h + out_at);
    Blob ck, tab;
    size_t row = 0, at[2] = {0, 0}, res = 0;
    for (int i : pick) {
        const qnae_grad_job& j = jobs[i];
        const int nck = j.p > 1 ? (j.p - 1) / every : 0;
        const size_t N = (size_t)1 << j.n, ck_at = ck.take(sizeof(float2) * N * (size_t)std::max(nck, 1));
        const size_t tab_at = tab.take(sizeof(float2) * (size_t)std::max(j.p, 1) * (size_t)(j.m + 1));
        float2* const tables = (float2*)((char*)ctx->g_tables.ptr + tab_at);
        const int g = j.cost_dtype == QNAE_U16 ? 1 : 0;
        qnae::ResidentGradArgs& a = ((qnae::ResidentGradArgs*)(h + args_at[g]))[at[g]++];
        a.cost = j.cost_dev;
        a.luts = tables;
        a.cs = (const float2*)(d + cs_at) + row;
        a.ckpt = (float2*)((char*)ctx->g_states.ptr + ck_at);
        a.out = ho + res;
        a.w_psucc = w_psucc;
        a.w_energy = w_energy;
        a.n = j.n;
        a.p = j.p;
        a.lut_len = j.m + 1;
        a.every = every;
        res += 3 + 2 * (size_t)j.p;
        for (int l = 0; l < j.p; ++l, ++row) {
            hr[row] = {reduced(j.gammas[l]), 1.0, 0.0, -1.0, tables + (size_t)l * (size_t)(j.m + 1), j.m, 0};
            hc[row] = make_float2((float)std::cos(j.betas[l]), (float)std::sin(j.betas[l]));
        }
    }
    if (int rc = prologue(ctx, d, h, args_at[1] + sizeof(qnae::ResidentGradArgs) * group[1].size(), nullptr, QNAE_U8, 0,
                          s))
        return rc;
    HIP_TRY(qnae::launch_phase_rows((const qnae::PhaseRow*)(d + row_at), (int)rows, max_m, s));
    for (int g = 0; g < 2; ++g) {
        if (group[g].empty()) continue;
        double bytes = 0.0;
        for (int i : group[g]) bytes += std::ldexp(3.0 * jobs[i].p, jobs[i].n);
        HIP_TRY(timed(ctx, K_RESIDENT, bytes, s, [&] {
            return qnae::launch_resident_grad_batch(g ? QNAE_U16 : QNAE_U8,
                                                    (const qnae::ResidentGradArgs*)(d + args_at[g]),
                                                    (int)group[g].size(), s);
        }));
    }
    HIP_TRY(finish(drain));
    const double* r = ho;
    for (int i : pick) {
        const qnae_grad_job& j = jobs[i];
        out[i].p_success = r[0];
        out[i].expected_cost = r[1];
        out[i].norm = r[2];
        for (int l = 0; l < j.p; ++l) {
            j.dgammas[l] = r[3 + l];
            j.dbetas[l] = r[3 + j.p + l];
        }
        r += 3 + 2 * (size_t)j.p;
    }
    return QNAE_OK;
}

}  // namespace

extern "C" {

int qnae_qaoa_grad(qnae_ctx* ctx, const void* cost_dev, int32_t cost_dtype, int32_t n, int32_t m,
                   const double* gammas, const double* betas, int32_t p, double w_psucc, double w_energy,
                   int32_t checkpoint_every, double* dgammas, double* dbetas, qnae_result* out, void* stream) try {
    if (int rc = check_run_args(n, m, cost_dtype, cost_dev, gammas, betas, p)) return rc;
    if (!out) return fail(QNAE_EINVAL, "null result pointer");
    if (p > 0 && (!dgammas || !dbetas)) return fail(QNAE_EINVAL, "null gradient arrays with p=%d", p);
    if (checkpoint_every < 0) return fail(QNAE_EINVAL, "checkpoint_every=%d < 0", checkpoint_every);
    if (!std::isfinite(w_psucc) || !std::isfinite(w_energy)) return fail(QNAE_EINVAL, "non-finite weights");
    // a segment longer than p layers is one segment (and p + every stays in range)
    const int every = checkpoint_every > 0 ? std::min(checkpoint_every, std::max(p, 1)) : 4;
    if (int rc = enter(ctx, (hipStream_t)stream)) return rc;
    hipStream_t s = (hipStream_t)stream;
    const int lut_len = m + 1;

    if (n <= 13) {
        const qnae_grad_job job{cost_dev, cost_dtype, n, m, p, gammas, betas, dgammas, dbetas};
        return resident_grads(ctx, &job, {0}, w_psucc, w_energy, every, out, s);
    }

    // ---- tiled path ----------------------------------------------------------
    DrainOnExit drain{s};
    const int TB = qnae::kAdjointTileBits;
    const int nseg = p > 0 ? (p + every - 1) / every : 1;
    const std::vector<Group> groups = make_groups(n, TB, ctx->min_low_run, ctx->page_bit, 0);
    // The forward pass is one plan over all p layers, in place in the last
    // checkpoint's buffer; the boundary sweep that completes the last layer
    // of segment j < nseg - 1 also stores checkpoint j.
    const int T = p > 0 ? p : 1;
    std::vector<float2> ftab((size_t)T * lut_len), btab((size_t)T * lut_len);
    std::vector<MixForm> forms(T);
    const std::complex<double> final_scale = build_tables(n, m, gammas, betas, p, ftab.data(), forms.data());
    SweepPlan F;
    plan_sweeps(F, n, m, p, cost_dtype, TB, ctx->min_low_run, ctx->page_bit, 0, true, forms.data(), final_scale);
    std::vector<int> ckpt_of(F.ops.size(), -1);  // checkpoint stored by each forward sweep
    int stored = 0;
    for (size_t q = 0; q < F.ops.size(); ++q) {
        const Op& op = F.ops[q];
        if (op.kind != qnae::SK_BOUNDARY || op.pre_layer < 0) continue;
        const int done_layers = op.lut_layer;  // its pre mixing completes layer lut_layer - 1
        if (done_layers % every == 0 && done_layers < p) {
            ckpt_of[q] = done_layers / every - 1;
            ++stored;
        }
    }
    if (stored != nseg - 1)
        return fail(QNAE_EINVAL, "n=%d: %zu qubit groups, the forward pass needs at least two", n, groups.size());

    // Reverse segments: b-layer i of segment j is forward layer b - 1 - i.
    struct Seg {
        int a, b;
        size_t blut_at;
        std::vector<AdjOp> aops;
        std::vector<Layer> inv;  // inverse mixer of b-layer i: exp(+i beta X) per qubit
    };
    std::vector<Seg> segs(nseg);
    int total_aops = 0;
    for (int j = 0; j < nseg; ++j) {
        Seg& S = segs[j];
        S.a = j * every;
        S.b = p > 0 ? std::min(p, S.a + every) : 0;
        const int L = S.b - S.a;
        // the inverse phase exp(+i gamma c) times the scalar factor the
        // inverse mixer's butterflies left out
        S.blut_at = (size_t)S.a * lut_len;
        S.inv.resize(L);
        for (int i = 0; i < L; ++i) {
            S.inv[i] = mixer_form(-betas[S.b - 1 - i], n);
            phase_row(gammas[S.b - 1 - i], m, S.inv[i].scale, +1, btab.data() + S.blut_at + (size_t)i * lut_len);
        }
        if (L > 0) S.aops = make_adjoint_plan((int)groups.size(), L);
        total_aops += (int)S.aops.size();
    }
    // The reverse pass opens with a sweep that mixes one group and forms lam.
    if (!segs[nseg - 1].aops.empty() && segs[nseg - 1].aops[0].kind != qnae::AK_MIDDLE)
        return fail(QNAE_EINVAL, "n=%d: %zu qubit groups, the reverse pass needs at least two", n, groups.size());
    Blob B;
    const size_t flut_at = B.take(sizeof(float2) * ftab.size());
    const size_t blut_at = B.take(sizeof(float2) * btab.size());
    B.take(16);
    const size_t res_at = B.take(sizeof(double) * 3 * (total_aops + 1));  // pinned only
    HIP_TRY(ctx->h_blob.reserve(B.size));
    HIP_TRY(ctx->g_blob.reserve(B.size));
    char* h = (char*)ctx->h_blob.ptr;
    char* d = (char*)ctx->g_blob.ptr;
    std::memcpy(h + flut_at, ftab.data(), sizeof(float2) * ftab.size());
    std::memcpy(h + blut_at, btab.data(), sizeof(float2) * btab.size());
    const bool check = p > 0 && n >= kFlipMinN, early = check && n <= kFlipEarlyMaxN;
    // Elements of a state's buffer: with the first sweep launched on the whole
    // state ahead of the answer, whole states, used up to the lower half.
    size_t room = (size_t)1 << n;
    // checkpoints 0 .. nseg-1 (state after each segment), then lam
    auto reserve = [&]() -> hipError_t {
        if (hipError_t e = ctx->g_states.reserve(sizeof(float2) * room * (size_t)(nseg + 1))) return e;
        return ctx->g_partials.reserve(sizeof(double) * 3 * (room >> TB) * (size_t)(total_aops + 1));
    };
    if (!check || early) HIP_TRY(reserve());
    if (int rc = prologue(ctx, d, h, blut_at + sizeof(float2) * btab.size(), check ? cost_dev : nullptr, cost_dtype, n,
                          s))
        return rc;
    bool half = false;
    if (check && !early) {
        if (int rc = flip_answer(ctx, s, &half)) return rc;
        if (half) room >>= 1;
        HIP_TRY(reserve());
    }
    float2* ck = (float2*)ctx->g_states.ptr;
    float2* lam = ck + room * (size_t)nseg;
    double* parts = (double*)ctx->g_partials.ptr;
    const float2* d_flut = (const float2*)(d + flut_at);
    const float2* d_blut = (const float2*)(d + blut_at);

    // forward pass
    float2* const run = ck + room * (size_t)(nseg - 1);
    F.half = half;
    size_t N = room;  // stored elements of a state
    uint32_t tiles = (uint32_t)(N >> TB);
    for (size_t q = 0; q < F.ops.size(); ++q) {
        const Op& op = F.ops[q];
        if (early && q == 1) {
            if (int rc = flip_answer(ctx, s, &half)) return rc;
            F.half = half;
            N >>= half ? 1 : 0;
            tiles = (uint32_t)(N >> TB);
        }
        // row total_aops of the partial sums: the forward readout
        double* const fwd_parts = parts + 3 * (size_t)tiles * total_aops;
        SweepArgs a;
        sweep_args(F, op, run, cost_dev, d_flut, fwd_parts, &a);
        if (ckpt_of[q] < 0) {
            HIP_TRY(timed(ctx, op_profile_kind(op), op_bytes(F, op), s,
                          [&] { return qnae::launch_sweep(TB, cost_dtype, op.kind, a, s); }));
            continue;
        }
        const std::complex<double> f = mixer_form(betas[op.lut_layer - 1], n).scale;
        a.ckpt = ck + room * (size_t)ckpt_of[q];
        a.ckpt_scale = make_float2((float)f.real(), (float)f.imag());
        HIP_TRY(timed(ctx, op_profile_kind(op), op_bytes(F, op) + 8.0 * (double)N, s,
                      [&] { return qnae::launch_sweep_ckpt(cost_dtype, a, s); }));
    }
    // a symmetric state equals its all-qubit flip: relabelling is the identity
    if (!half && p > 0 && F.flips_before[p]) HIP_TRY(qnae::launch_reverse(run, N, s));
    // lam = W psi_p is formed by the first reverse sweep, which mixes one
    // group only (a layer spans at least two groups here, n > TB), from the
    // psi_p and cost it loads
    // reverse segments, last first. `relabel`: lam's index x holds element
    // x ^ (2^n - 1) (an odd number of cotangent forms so far); psi restarts
    // from a checkpoint in natural order at each segment, so within a segment
    // it is relabelled against lam by the value `relabel` had at the start.
    // done[i]: qubits of b-layer i mixed by earlier sweeps.
    int q = 0;
    std::vector<std::pair<int, const AdjOp*>> order;  // (segment, op) in launch order
    std::vector<double> gamma_weight;                 // per op: |F|^2 of its phase layer
    int relabel = 0;
    for (int j = nseg - 1; j >= 0; --j) {
        const Seg& S = segs[j];
        float2* psi = ck + room * (size_t)j;
        const int psi_flip = relabel;
        std::vector<int> done(S.inv.size(), 0);
        for (const AdjOp& op : S.aops) {
            const Group& g = groups[op.group];
            qnae::AdjointArgs a;
            std::memset(&a, 0, sizeof a);
            a.lam = lam;
            a.psi = psi;
            a.cost = cost_dev;
            a.lut = op.phase_layer >= 0 ? d_blut + S.blut_at + (size_t)op.phase_layer * lut_len : nullptr;
            a.partials = parts + 3 * (size_t)tiles * q;
            a.n = n;
            a.lut_len = lut_len;
            // half: bit n-1, when the group has it, is the virtual bit
            for (int i = 0; i < TB; ++i) {
                a.pos[i] = (uint8_t)g.pos[i];
                if (half && g.pos[i] == n - 1) a.virt = 1;
                else a.tile_bits |= 1ull << g.pos[i];
            }
            a.mir = N - 1;
            a.wmask = (N - 1) & ~a.tile_bits;
            // (its mirror covers the highest stored bit outside the tile)
            if (a.virt) a.wmask &= ~(1ull << (63 - __builtin_clzll(a.wmask)));
            a.nw = __builtin_popcountll(a.wmask);
            a.pre_mask = op.pre_layer >= 0 ? g.mask : 0u;
            a.post_mask = op.post_layer >= 0 ? g.mask : 0u;
            const int qubits = __builtin_popcount(g.mask);
            // one qubit's |factor|^2: cos^2 (tangent form) or sin^2, 1 / (1 + t^2) either way
            auto factor2 = [&](int i) {
                const double b = betas[S.b - 1 - i];
                const double c = std::cos(b), sn = std::sin(b);
                return S.inv[i].form.flip ? sn * sn : c * c;
            };
            if (op.pre_layer >= 0) {
                const int i = op.pre_layer;
                a.pre_t = S.inv[i].form.t;
                a.pre_r = (float)factor2(i);
                a.pre_w = (float)std::pow(factor2(i), done[i]);
                done[i] += qubits;
            }
            double gw = 0.0;
            if (op.phase_layer >= 0) {
                const int i = op.phase_layer;
                relabel ^= half ? 0 : S.inv[i].form.flip;
                a.cost_flip = relabel ? (uint64_t)N - 1ull : 0ull;
                gw = std::pow(factor2(i), n);
            }
            if (op.post_layer >= 0) {
                const int i = op.post_layer;
                a.post_t = S.inv[i].form.t;
                a.post_r = (float)factor2(i);
                a.post_w = (float)std::pow(factor2(i), done[i]);
                done[i] += qubits;
            }
            a.psi_flip = psi_flip;
            a.store_psi = op.kind == qnae::AK_END ? 0 : 1;
            const bool weigh = q == 0;
            a.w_psucc = (float)w_psucc;
            a.w_energy = (float)w_energy;
            const double cost_bytes = cost_dtype == QNAE_U8 ? 1.0 : 2.0;
            const double bytes = (32.0 - (a.store_psi ? 0.0 : 8.0) - (weigh ? 8.0 : 0.0) +
                                  (op.phase_layer >= 0 || weigh ? cost_bytes : 0.0)) *
                                 (double)N;
            HIP_TRY(timed(ctx, K_ADJOINT, bytes, s,
                          [&] { return qnae::launch_adjoint(cost_dtype, op.kind, a, s, weigh); }));
            order.emplace_back(j, &op);
            gamma_weight.push_back(gw);
            ++q;
        }
    }
    const double* r = (const double*)(h + res_at);  // the reduction writes pinned memory: no copy follows it
    HIP_TRY(qnae::launch_final_reduce_rows(parts, tiles, (double*)(h + res_at), total_aops + 1, s));
    HIP_TRY(finish(drain));
    const double twice = half ? 4.0 : 2.0;
    for (int l = 0; l < p; ++l) dgammas[l] = dbetas[l] = 0.0;
    for (int k = 0; k < total_aops; ++k) {
        const Seg& S = segs[order[k].first];
        const AdjOp& op = *order[k].second;
        if (op.pre_layer >= 0) dbetas[S.b - 1 - op.pre_layer] += twice * r[3 * k];
        if (op.phase_layer >= 0) dgammas[S.b - 1 - op.phase_layer] += twice * gamma_weight[k] * r[3 * k + 1];
        if (op.post_layer >= 0) dbetas[S.b - 1 - op.post_layer] += twice * r[3 * k + 2];
    }
    const double sc = std::norm(final_scale) * (half ? 2.0 : 1.0);
    out->p_success = r[3 * total_aops] * sc;
    out->expected_cost = r[3 * total_aops + 1] * sc;
    out->norm = r[3 * total_aops + 2] * sc;
    return QNAE_OK;
} catch (...) {
    return host_exception();
}

int qnae_qaoa_grad_batched(qnae_ctx* ctx, const qnae_grad_job* jobs, int32_t count, double w_psucc, double w_energy,
                           int32_t checkpoint_every, qnae_result* out, void* stream) try {
    if (count < 0 || (count > 0 && (!jobs || !out))) return fail(QNAE_EINVAL, "bad job array (count=%d)", count);
    if (checkpoint_every < 0) return fail(QNAE_EINVAL, "checkpoint_every=%d < 0", checkpoint_every);
    if (!std::isfinite(w_psucc) || !std::isfinite(w_energy)) return fail(QNAE_EINVAL, "non-finite weights");
    for (int i = 0; i < count; ++i) {
        const qnae_grad_job& j = jobs[i];
        int rc = check_run_args(j.n, j.m, j.cost_dtype, j.cost_dev, j.gammas, j.betas, j.p);
        if (!rc && j.p > 0 && (!j.dgammas || !j.dbetas)) rc = fail(QNAE_EINVAL, "null gradient arrays");
        if (rc) return fail(rc, "job %d: %s", i, std::string(last_error()).c_str());
    }
    if (count == 0) return QNAE_OK;
    const int every = checkpoint_every > 0 ? checkpoint_every : 4;
    if (int rc = enter(ctx, (hipStream_t)stream)) return rc;
    hipStream_t s = (hipStream_t)stream;
    std::vector<int> small;
    for (int i = 0; i < count; ++i)
        if (jobs[i].n <= 13) small.push_back(i);
    if (!small.empty())
        if (int rc = resident_grads(ctx, jobs, small, w_psucc, w_energy, every, out, s)) return rc;
    // Large jobs: the tiled adjoint, one after another.
    for (int i = 0; i < count; ++i) {
        const qnae_grad_job& j = jobs[i];
        if (j.n <= 13) continue;
        if (int rc = qnae_qaoa_grad(ctx, j.cost_dev, j.cost_dtype, j.n, j.m, j.gammas, j.betas, j.p, w_psucc, w_energy,
                                    checkpoint_every, j.dgammas, j.dbetas, &out[i], stream))
            return fail(rc, "job %d: %s", i, std::string(last_error()).c_str());
    }
    return QNAE_OK;
} catch (...) {
    return host_exception();
}

}  // extern "C"
