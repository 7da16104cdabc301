// The launch ahead of a run: table upload and, where asked for, the check of
// the cost diagonal for flip symmetry (Section 2.2: every NAE instance has it).
#include <cmath>

#include "host.h"

namespace qnae_host {

int prologue(qnae_ctx* ctx, void* dst, const void* src, size_t bytes, const void* cost, int dtype, int n,
             hipStream_t s) {
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
        a.ticket = ++ctx->flip_ticket & 0x7fffffffu;
        *(volatile uint32_t*)a.answer = 2u * (a.ticket ^ 1u);  // another ticket's
    }
    HIP_TRY(timed(ctx, K_PROLOGUE, (double)cost_bytes + (double)bytes, s,
                  [&] { return qnae::launch_prologue(a, dtype, s); }));
    return QNAE_OK;
}

int flip_answer(qnae_ctx* ctx, hipStream_t s, bool* symmetric) {
    const volatile uint32_t* const answer = (const volatile uint32_t*)((char*)ctx->h_small.ptr + kSmallFlipAt);
    const uint32_t ticket = ctx->flip_ticket & 0x7fffffffu;
    for (int spin = 0; spin < (1 << 20) && *answer >> 1 != ticket; ++spin) {
    }
    if (*answer >> 1 != ticket) HIP_TRY(hipStreamSynchronize(s));  // long work ahead of the check
    const uint32_t v = *answer;
    if (v >> 1 != ticket) return fail(QNAE_EHIP, "the flip check left no answer");
    *symmetric = (v & 1u) == 0u;
    return QNAE_OK;
}

}  // namespace qnae_host
