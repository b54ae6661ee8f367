// The CFL rate slots of dg_step after a launch that failed: the library's host code (dg_host.cpp) against
// stand-ins for the HIP calls and kernels it reaches, whose "device" memory is the host's.  Every launch of
// a three-step call fails in turn (it returns an error and does nothing); the time step of the next call
// must be that of the state it is given.  The kernels' part in the slots is what their sources say: the
// reduction raises its slot to the state's rate and clears the other, a stage clears zero_rate and raises
// next_rate.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "dg_internal.h"

static int launches = 0, fail_at = -1;
static double state_rate = 1.0;
static hipError_t launch() { return launches++ == fail_at ? hipErrorLaunchFailure : hipSuccess; }

extern "C" {
hipError_t hipMalloc(void **p, size_t n) { return (*p = calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { memset(p, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t) { memset(p, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorName(hipError_t) { return "error"; }
const char *hipGetErrorString(hipError_t) { return "error"; }
}

namespace dgmi {
hipError_t stage_cell_setup(int, int, int *per_cu) { *per_cu = 2; return hipSuccess; }
hipError_t launch_zero_u64(unsigned long long *p, hipStream_t) {
    const hipError_t e = launch();
    if (e == hipSuccess) *p = 0;
    return e;
}
hipError_t launch_cfl(int, const void *, int, int, long long, double, const double *, double *rate, double *zero, hipStream_t) {
    const hipError_t e = launch();
    if (e != hipSuccess) return e;
    *rate = std::max(*rate, state_rate);
    if (zero) *zero = 0.0;
    return e;
}
hipError_t launch_stage_cell(int, int, const StageArgs &a, hipStream_t) {
    const hipError_t e = launch();
    if (e != hipSuccess) return e;
    if (a.zero_rate) *a.zero_rate = 0.0;
    if (a.next_rate) *a.next_rate = std::max(*a.next_rate, state_rate);
    return e;
}
}  // namespace dgmi

int main() {
    int bad = 0, failed = 0;
    for (fail_at = 0;; fail_at++) {
        dg_config cfg{};
        cfg.k = 1;
        cfg.gamma = 1.4;
        cfg.cfl = 0.3;
        cfg.precision = DG_FP64;
        for (int a = 0; a < 3; a++) cfg.n[a] = 8, cfg.box[a] = 1.0;
        dg_ctx *c = nullptr;
        if (dg_init(&cfg, nullptr, &c) != DG_OK) return 2;
        const size_t n = dg_state_count(c);
        double *y = static_cast<double *>(calloc(3 * n, sizeof(double)));
        launches = 0;
        state_rate = 10.0;
        const bool ok = dg_step(c, y, y + n, 0.0, 3, nullptr) == DG_OK;
        failed += !ok;
        launches = -1000;  // no more failures
        state_rate = 2.0;  // the caller goes on with a slower state
        double dt[2];
        for (double &d : dt)
            if (dg_dt(c, y, &d) != DG_OK) return 3;
        const double want = 0.3 / 3.0 / 2.0;
        if (!(dt[0] == want && dt[1] == want)) {
            printf("launch %d failed: dt %.17g, %.17g, not %.17g\n", fail_at, dt[0], dt[1], want);
            bad++;
        }
        free(y);
        dg_destroy(c);
        if (ok) break;
    }
    printf("%d failing launches, %d wrong time steps\n", failed, bad);
    return bad || failed < 10 ? 1 : 0;
}
