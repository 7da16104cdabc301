// Phase tables built on the device: rows scale exp(sign i g c), c = 0 .. m, in
// FP64 and rounded to FP32, as the host's phase_row builds them by angle
// addition (their entries differ by at most its 1e-13 before rounding). For
// calls with many long rows: 800 rows of 2124 entries took the host's eight
// threads and two 13.6 MB copies over PCIe about 0.7 ms, here 48-byte row
// records travel instead. Bound by the FP64 sine and cosine. Rows come with |g| <= 3.2
// (the host reduces larger ones), so that the rounding of g c stays below 3e-11.
#include "internal.h"

namespace qnae {
namespace {

constexpr int kRowThreads = 256;
__global__ __launch_bounds__(kRowThreads) void phase_rows_kernel(const PhaseRow* rows) {
    const PhaseRow r = rows[blockIdx.y];
    for (int32_t c = (int32_t)(blockIdx.x * kRowThreads + threadIdx.x); c <= r.m;
         c += (int32_t)(gridDim.x * kRowThreads)) {
        double sn, cs;
        sincos(r.g * (double)c, &sn, &cs);
        sn *= r.sign;
        r.out[c] = make_float2((float)(r.re * cs - r.im * sn), (float)(r.re * sn + r.im * cs));
    }
}

}  // namespace

hipError_t launch_phase_rows(const PhaseRow* rows, int count, int max_m, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    for (int at = 0; at < count; at += 65535) {
        const int some = count - at < 65535 ? count - at : 65535;
        const int per = (max_m + kRowThreads) / kRowThreads;
        hipLaunchKernelGGL(phase_rows_kernel, dim3((uint32_t)(per < 64 ? per : 64), (uint32_t)some), dim3(kRowThreads),
                           0, s, rows + at);
        if (hipError_t e = hipGetLastError()) return e;
    }
    return hipSuccess;
}

}  // namespace qnae
