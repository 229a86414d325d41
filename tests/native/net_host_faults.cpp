// The host side of a network gradient with resources refused: this program
// defines the HIP calls that the library makes for it, over host memory (copies
// at once, launches that do nothing), and refuses the stream, an event or the
// pinned memory of the gradient's host copy.  Linked to liblbm.so, whose calls
// resolve here; needs no GPU.
//
// A refusal must leave the gradient as it is without these resources (one copy
// after the pass), no message of an error and no error for the next launch.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "lbm_net.h"

namespace {
enum Refused { NONE, STREAM, EVENT, PINNED };
Refused refused = NONE;
hipError_t last = hipSuccess;      // as the runtime keeps it: until it is read
int events = 0, streams = 0, pins = 0, failures = 0;

hipError_t refuse() { return last = hipErrorOutOfMemory; }

void check(bool ok, const char *what, int n) {
    if (ok) return;
    std::printf("FAILED: %s (case %d)\n", what, n);
    ++failures;
}
}  // namespace

extern "C" {
hipError_t hipGetLastError(void) {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    if (refused == STREAM) return refuse();
    return ++streams, *s = (hipStream_t)std::malloc(1), hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { return --streams, std::free(s), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    if (refused == EVENT && events == 3) return refuse();
    return ++events, *e = (hipEvent_t)std::malloc(1), hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { return --events, std::free(e), hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    if (refused == PINNED) return refuse();
    return ++pins, *p = std::malloc(n), hipSuccess;
}
hipError_t hipHostFree(void *p) { return --pins, std::free(p), hipSuccess; }
}  // extern "C"

int main() {
    lbm_net_config cfg{};
    cfg.H = 8;
    cfg.W = 16;
    cfg.batch = 1;
    cfg.cin = cfg.cout = 3;
    const int chans[4] = {32, 64, 128, 128};      // enough parameters for a copy in pieces
    for (int k = 0; k < 4; ++k) cfg.chans[k] = chans[k];
    cfg.act_bf16 = 1;
    const size_t bytes = lbm_net_workspace_bytes(&cfg), np = (size_t)lbm_net_param_count(&cfg);
    char *ws = (char *)std::aligned_alloc(256, bytes);
    std::vector<float> in((size_t)3 * 8 * 16), grad(np);
    std::vector<uint8_t> fluid((size_t)8 * 16, 1);

    for (int r = NONE; r <= PINNED; ++r) {
        lbm_net *net = nullptr;
        check(lbm_net_create(&net, &cfg, ws, bytes, nullptr) == LBM_OK, "create", r);
        std::memset(ws, 0x11, bytes);             // what every kernel "computed"
        float want;
        std::memcpy(&want, ws, 4);
        for (int call = 0; call < 3; ++call) {    // refused twice, then granted
            refused = call < 2 ? (Refused)r : NONE;
            std::fill(grad.begin(), grad.end(), 0.f);
            double loss = 0.0;
            check(lbm_net_gradient(net, in.data(), in.data(), fluid.data(), 1, &loss, grad.data()) == LBM_OK,
                  "gradient", r);
            check(std::strlen(lbm_net_last_error(net)) == 0, "no message after a call that succeeded", r);
            check(last == hipSuccess, "no error left for the next launch", r);
            size_t same = 0;
            for (float g : grad) same += g == want;
            check(same == np, "the whole gradient reaches the caller", r);
        }
        check(streams == 1 && events > 0 && pins == 1, "the resources once", r);
        lbm_net_free(net);
        check(streams == 0 && events == 0 && pins == 0, "and given back", r);
    }
    std::free(ws);
    if (failures == 0) std::printf("network host faults: ok\n");
    return failures ? 1 : 0;
}
