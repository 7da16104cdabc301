// The launch ahead of a run: table upload and, where asked for, the check of
// the cost diagonal for flip symmetry (Section 2.2: every NAE instance has it).
#include <algorithm>
#include <cmath>
#include <vector>

#include "host.h"

namespace qnae_host {

static constexpr size_t kFlipFlagsAt = 64;  // pinned: the ticket, then a flag per checked instance, then the jobs

int prologue(qnae_ctx* ctx, void* dst, const void* src, size_t bytes, const void* cost, int dtype, int n,
             hipStream_t s, bool profiled) {
    qnae::PrologueArgs a;
    a.dst = (uint4*)dst;
    a.src = (const uint4*)src;
    a.copies = (bytes + 15) / 16;
    a.cost = (const uint4*)cost;
    const uint64_t cost_bytes = cost ? (uint64_t)(dtype == QNAE_U8 ? 1 : 2) << n : 0;
    a.quads = cost_bytes / 16;
    a.word = (uint32_t*)((char*)ctx->small.ptr + kSmallFlipAt);
    a.answer = (uint32_t*)((char*)ctx->h_small.ptr + kSmallFlipAt);
    a.ticket = 0;
    if (cost) {
        a.ticket = next_ticket(&ctx->flip_ticket);
        *(volatile uint32_t*)a.answer = 0u;
    }
    auto launch = [&] { return qnae::launch_prologue(a, dtype, s); };
    HIP_TRY(profiled ? timed(ctx, K_PROLOGUE, (double)cost_bytes + (double)bytes, s, launch) : launch());
    return QNAE_OK;
}

// Waits until *word >> shift is `ticket`: watches it for a while, then (long
// work ahead of the check) waits for the stream.
static int wait_ticket(const volatile uint32_t* word, int shift, uint32_t ticket, hipStream_t s) {
    for (int spin = 0; spin < (1 << 20) && *word >> shift != ticket; ++spin) {
    }
    if (*word >> shift != ticket) HIP_TRY(hipStreamSynchronize(s));
    if (*word >> shift != ticket) return fail(QNAE_EHIP, "the flip check left no answer");
    return QNAE_OK;
}

int flip_answer(qnae_ctx* ctx, hipStream_t s, bool* symmetric) {
    const volatile uint32_t* const answer = (const volatile uint32_t*)((char*)ctx->h_small.ptr + kSmallFlipAt);
    if (int rc = wait_ticket(answer, 1, ctx->flip_ticket, s)) return rc;
    *symmetric = (*answer & 1u) == 0u;
    return QNAE_OK;
}

int flip_batch_begin(qnae_ctx* ctx, const qnae_instance* inst, int count, const std::vector<int>& half, hipStream_t s,
                     FlipBatch* f) {
    std::vector<int>& jobs = f->jobs;
    jobs.clear();
    uint64_t amps = 0;
    for (int i = 0; i < count; ++i) {
        if (half[i] || inst[i].n <= kResidentMaxN || inst[i].p == 0) continue;
        jobs.push_back(i);
        amps += 1ull << inst[i].n;
    }
    if (amps < kFlipBatchAmps || jobs.size() > 65535) {
        jobs.clear();
        return QNAE_OK;
    }
    const size_t jobs_at = (kFlipFlagsAt + sizeof(uint32_t) * jobs.size() + 15) / 16 * 16;
    const size_t jobs_bytes = sizeof(qnae::FlipJob) * jobs.size();
    static_assert(sizeof(qnae::FlipJob) % 16 == 0, "jobs travel in 16-byte pieces");
    HIP_TRY(ctx->h_flip.reserve(jobs_at + jobs_bytes));
    HIP_TRY(ctx->f_jobs.reserve(jobs_bytes));
    char* const h = (char*)ctx->h_flip.ptr;
    volatile uint32_t* const answer = (volatile uint32_t*)h;
    uint32_t* const flags = (uint32_t*)(h + kFlipFlagsAt);
    qnae::FlipJob* const fj = (qnae::FlipJob*)(h + jobs_at);
    uint32_t most = 0;
    double bytes = 0.0;
    for (size_t q = 0; q < jobs.size(); ++q) {
        const qnae_instance& x = inst[jobs[q]];
        const bool u16 = x.cost_dtype == QNAE_U16;
        flags[q] = 0u;
        fj[q] = {(const uint4*)x.cost_dev, (uint32_t)(((uint64_t)(u16 ? 2 : 1) << x.n) / 16), u16 ? 1u : 0u, 0u, {}};
        most = std::max(most, fj[q].quads);
        bytes += 16.0 * fj[q].quads;
    }
    const uint32_t ticket = f->ticket = next_ticket(&ctx->flip_ticket);
    *answer = 0u;
    if (int rc = prologue(ctx, ctx->f_jobs.ptr, fj, jobs_bytes, nullptr, QNAE_U8, 0, s)) return rc;
    uint32_t* const word = (uint32_t*)((char*)ctx->small.ptr + kSmallFlipAt);
    HIP_TRY(timed(ctx, K_PROLOGUE, bytes, s, [&] {
        return qnae::launch_flip_batch((qnae::FlipJob*)ctx->f_jobs.ptr, (int)jobs.size(), most, flags, word,
                                       ticket, (uint32_t*)h, s);
    }));
    return QNAE_OK;
}

int flip_batch_end(qnae_ctx* ctx, const FlipBatch& f, std::vector<int>& half, hipStream_t s) {
    if (f.jobs.empty()) return QNAE_OK;
    const volatile uint32_t* const answer = (const volatile uint32_t*)ctx->h_flip.ptr;
    const volatile uint32_t* const flags = (const volatile uint32_t*)((const char*)ctx->h_flip.ptr + kFlipFlagsAt);
    if (int rc = wait_ticket(answer, 0, f.ticket, s)) return rc;
    for (size_t q = 0; q < f.jobs.size(); ++q)
        if (flags[q] == 0u) half[f.jobs[q]] = 2;
    return QNAE_OK;
}

}  // namespace qnae_host
