// The library's host code over a stand-in for the HIP runtime and the kernel
// launchers (no GPU): buffers are host memory, a launch only counts as work in
// flight until something waits for it, and any one call can be made to fail.
// Flip checks answer as g_symmetric says.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../paper_2401_02852_amd/csrc/host.h"

#define CHECK(cond)                                        \
    do {                                                   \
        if (!(cond)) {                                     \
            std::printf("line %d: %s\n", __LINE__, #cond); \
            std::exit(1);                                  \
        }                                                  \
    } while (0)

namespace {
int g_fail_at = 0;   // the call that fails, counted from 1 (0: none)
int g_calls = 0;     // calls that can fail, so far
int g_in_flight = 0; // launches and copies since the last wait
bool g_symmetric = false;
double g_time = 0.0;          // ms that the sweeps launched so far take
double g_sweep_ms[2][15];     // per sweep: whole or half state, tile bits
std::vector<uint32_t> g_tickets;

hipError_t step(hipError_t error) { return ++g_calls == g_fail_at ? error : hipSuccess; }
hipError_t launched() {
    if (hipError_t e = step(hipErrorLaunchFailure)) return e;
    ++g_in_flight;
    return hipSuccess;
}
hipError_t waited() {
    g_in_flight = 0;
    return hipSuccess;
}
hipError_t allocated(void** p, size_t bytes) {
    if (hipError_t e = step(hipErrorOutOfMemory)) return e;
    *p = std::malloc(bytes ? bytes : 1);
    return hipSuccess;
}
}  // namespace

extern "C" {
hipError_t hipDeviceSynchronize() { return waited(); }
hipError_t hipStreamSynchronize(hipStream_t) { return waited(); }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "injected"; }
hipError_t hipMalloc(void** p, size_t bytes) { return allocated(p, bytes); }
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) { return allocated(p, bytes); }
hipError_t hipFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipHostFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) { return std::memset(p, v, n), hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return launched(); }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return launched(); }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t)std::malloc(sizeof(double)), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return std::free((void*)e), hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
    return *ms = (float)(*(double*)b - *(double*)a), hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { return *(double*)e = g_time, step(hipErrorUnknown); }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = (hipStream_t)std::malloc(1), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { return std::free((void*)s), hipSuccess; }
hipError_t hipGraphCreate(hipGraph_t* g, unsigned) {
    if (hipError_t e = step(hipErrorOutOfMemory)) return e;
    return *g = (hipGraph_t)std::malloc(1), hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    if (hipError_t e = step(hipErrorOutOfMemory)) return e;
    return *x = (hipGraphExec_t)std::malloc(1), hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { return std::free((void*)g), hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { return std::free((void*)x), hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return launched(); }
}

namespace qnae {
hipError_t launch_cost(const CostArgs&, int, hipStream_t) { return launched(); }
hipError_t launch_cost_batch(const CostArgs*, const uint32_t*, int, uint32_t, int, int, int, hipStream_t) {
    return launched();
}
hipError_t launch_prologue(const PrologueArgs& a, int, hipStream_t) {
    if (hipError_t e = launched()) return e;
    if (a.cost) {
        g_tickets.push_back(a.ticket);
        *a.answer = 2u * a.ticket + (g_symmetric ? 0u : 1u);
    }
    return hipSuccess;
}
hipError_t launch_flip_batch(FlipJob*, int count, uint32_t, uint32_t* flags, uint32_t*, uint32_t ticket,
                             uint32_t* answer, hipStream_t) {
    if (hipError_t e = launched()) return e;
    g_tickets.push_back(ticket);
    for (int i = 0; i < count; ++i) flags[i] = g_symmetric ? 0u : 1u;
    *answer = ticket;
    return hipSuccess;
}
hipError_t launch_phase_rows(const PhaseRow*, int, int, hipStream_t) { return launched(); }
hipError_t launch_sweep(int tb, int, int, const SweepArgs& a, hipStream_t) {
    g_time += g_sweep_ms[a.half ? 1 : 0][tb];
    return launched();
}
hipError_t launch_sweep_ckpt(int, const SweepArgs&, hipStream_t) { return launched(); }
hipError_t launch_sweep_batch(int, int, int, const SweepArgs*, const uint32_t*, int, uint32_t, LaunchTo, bool, int) {
    return launched();
}
int sweep_l1(int, int, uint32_t, uint32_t) { return 1; }
hipError_t launch_reverse(float2*, uint64_t, LaunchTo) { return launched(); }
hipError_t launch_resident(int, const ResidentArgs&, hipStream_t) { return launched(); }
hipError_t launch_resident_inline(int, const ResidentInlineArgs&, hipStream_t) { return launched(); }
hipError_t launch_resident_batch(int, const ResidentArgs*, int, LaunchTo) { return launched(); }
hipError_t launch_resident_grad_batch(int, const ResidentGradArgs*, int, hipStream_t) { return launched(); }
hipError_t launch_adjoint(int, int, const AdjointArgs&, hipStream_t, bool) { return launched(); }
hipError_t launch_final_reduce(const double*, int64_t, double*, hipStream_t) { return launched(); }
hipError_t launch_final_reduce_batch(const double* const*, const uint32_t*, double* const*, int, LaunchTo) {
    return launched();
}
hipError_t launch_final_reduce_rows(const double*, int64_t, double*, int, hipStream_t) { return launched(); }
hipError_t launch_sample_masses(const float2*, int, double*, double*, hipStream_t) { return launched(); }
hipError_t launch_sample_prefix(int, const double*, double*, double*, const double*, double*, int, hipStream_t) {
    return launched();
}
hipError_t launch_sample_draws(const float2*, int, const void*, int, const double*, int, const double*, const double*,
                               const double*, uint64_t*, int32_t*, hipStream_t) {
    return launched();
}
}  // namespace qnae

namespace qnae_host {
int noalloc_setup(qnae_ctx*) { return QNAE_OK; }
}  // namespace qnae_host

namespace {

const double g_angles[3] = {0.3, 0.2, 0.9};
void* const g_cost = (void*)(uintptr_t)0x1000;  // never read here

std::vector<qnae_instance> batch(int count, int n) {
    return std::vector<qnae_instance>((size_t)count, {g_cost, QNAE_U8, n, 40, 3, g_angles, g_angles, nullptr, 0});
}

// Successive checks, single and batched in any order, never share a ticket.
void tickets() {
    qnae_ctx* ctx = nullptr;
    CHECK(qnae_create(&ctx, 0) == QNAE_OK);
    auto jobs = batch(8, 20);
    std::vector<qnae_result> out(8);
    g_tickets.clear();
    for (int i = 0; i < 12; ++i) {
        if (i % 3 == 2) CHECK(qnae_qaoa_run(ctx, g_cost, QNAE_U8, 20, 40, g_angles, g_angles, 3, nullptr, out.data(), nullptr) == QNAE_OK);
        else CHECK(qnae_qaoa_run_batched(ctx, jobs.data(), 8, out.data(), nullptr) == QNAE_OK);
    }
    CHECK(g_tickets.size() == 12);
    for (size_t i = 0; i < g_tickets.size(); ++i) {
        CHECK(g_tickets[i] != 0u);
        for (size_t j = 0; j < i; ++j) CHECK(g_tickets[i] != g_tickets[j]);
    }
    ctx->flip_ticket = 0x7ffffffeu;  // and past the end of their range
    g_tickets.clear();
    for (int i = 0; i < 3; ++i) CHECK(qnae_qaoa_run_batched(ctx, jobs.data(), 8, out.data(), nullptr) == QNAE_OK);
    CHECK(g_tickets[0] == 0x7fffffffu && g_tickets[1] == 1u && g_tickets[2] == 2u);
    CHECK(qnae_qaoa_run(ctx, g_cost, QNAE_U8, 24, 40, g_angles, g_angles, 3, nullptr, out.data(), nullptr) == QNAE_OK);
    CHECK(qnae_destroy(ctx) == QNAE_OK);
}

// Every call of `fn` that ends in an error has waited for what it had launched,
// whichever step failed; then the same call succeeds.
template <typename F>
void drains(const char* what, F&& fn) {
    for (bool symmetric : {false, true}) {
        g_symmetric = symmetric;
        for (int at = 1;; ++at) {
            CHECK(at < 500);
            qnae_ctx* ctx = nullptr;
            CHECK(qnae_create(&ctx, 0) == QNAE_OK);
            g_calls = 0;
            g_in_flight = 0;
            g_fail_at = at;
            const int rc = fn(ctx);
            const bool failed = g_calls >= at;
            g_fail_at = 0;
            if ((rc != QNAE_OK) != failed || g_in_flight != 0) {
                std::printf("%s, step %d: status %d, %d launches in flight\n", what, at, rc, g_in_flight);
                std::exit(1);
            }
            CHECK(fn(ctx) == QNAE_OK && g_in_flight == 0);
            CHECK(qnae_destroy(ctx) == QNAE_OK);
            if (!failed) break;
        }
    }
}

void error_exits() {
    double dg[3], db[3];
    qnae_result out[16];
    for (int n : {12, 16, 20, 23})
        for (int m : {40, 255})
            drains("run", [&](qnae_ctx* ctx) {
                return qnae_qaoa_run(ctx, g_cost, QNAE_U8, n, m, g_angles, g_angles, 3, nullptr, out, nullptr);
            });
    for (int n : {12, 16, 20, 23})
        drains("gradient", [&](qnae_ctx* ctx) {
            return qnae_qaoa_grad(ctx, g_cost, QNAE_U8, n, 40, g_angles, g_angles, 3, 1.0, 0.0, 2, dg, db, out, nullptr);
        });
    for (int n : {12, 18, 20})
        drains("batch", [&](qnae_ctx* ctx) {
            auto jobs = batch(8, n);
            jobs[0].n = 14;
            jobs[7].n = 20;
            return qnae_qaoa_run_batched(ctx, jobs.data(), 8, out, nullptr);
        });
    drains("sample", [&](qnae_ctx* ctx) {
        const double u[4] = {0.1, 0.5, 0.7, 0.9};
        uint64_t x[4];
        return qnae_sample(ctx, g_cost, 16, nullptr, QNAE_U8, u, 4, x, nullptr, nullptr);
    });
}

// The tile shape is ranked on whole-state and half-state runs together where
// diagonals with and without the symmetry share it, on whole-state ones below.
void autotune() {
    qnae_ctx* ctx = nullptr;
    CHECK(qnae_create(&ctx, 0) == QNAE_OK);
    const double whole[3] = {100.0, 60.0, 50.0}, half[3] = {10.0, 11.0, 40.0};
    for (int i = 0; i < 3; ++i) {
        g_sweep_ms[0][12 + i] = whole[i];
        g_sweep_ms[1][12 + i] = half[i];
    }
    qnae_tune t;
    CHECK(qnae_autotune(ctx, 20, QNAE_U8, 2, &t, nullptr) == QNAE_OK);
    CHECK(t.tile_bits == 13);  // 100 + 20, 60 + 22, 50 + 80
    // two groups, p + 1 sweeps: three and five of them timed, eleven for ten layers
    CHECK(t.ms_per_layer > 65.9 && t.ms_per_layer < 66.1);
    CHECK(qnae_autotune(ctx, 19, QNAE_U8, 2, &t, nullptr) == QNAE_OK);
    CHECK(t.tile_bits == 14 && t.ms_per_layer > 54.9 && t.ms_per_layer < 55.1);
    qnae_tune in_use;
    CHECK(qnae_get_tune(ctx, 20, QNAE_U8, &in_use) == QNAE_OK && in_use.tile_bits == 13);
    CHECK(qnae_destroy(ctx) == QNAE_OK);
}

}  // namespace

int main() {
    tickets();
    error_exits();
    autotune();
    std::printf("host paths ok\n");
    return 0;
}
