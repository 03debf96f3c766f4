// The device branch of the heuristic's integer square root, for its test: it
// starts from the hardware's single-precision root, which the host branch does
// not have. Built into the probe library (libppsp_probe.so), outside the search
// library and its C interface. probe_isqrt32(device, q, n, out) writes
// isqrt32(q[i]) to out[i], i < n, host arrays. Returns 0, or -1 for bad
// arguments (null arrays, n == 0 or n > 2^28), -3 when the device has no room
// for them, -7 on a HIP error.
#include "ppsp_dev.h"

namespace ppsp_rootprobe_kernels {

__global__ __launch_bounds__(256) void k_isqrt32(const uint64_t *q, uint32_t n, uint32_t *out) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = ppsp::isqrt32(q[i]);
}

}  // namespace ppsp_rootprobe_kernels

extern "C" int probe_isqrt32(int device, const uint64_t *q, uint64_t n, uint32_t *out) {
    enum { E_INVALID = -1, E_OOM = -3, E_DEVICE = -7 };
    if (!q || !out || n == 0 || n > (1ull << 28)) return E_INVALID;
    if (hipSetDevice(device) != hipSuccess) return E_DEVICE;
    uint64_t *dq = nullptr;
    uint32_t *dout = nullptr;
    if (hipMalloc((void **)&dq, n * 8) != hipSuccess) return E_OOM;
    if (hipMalloc((void **)&dout, n * 4) != hipSuccess) { (void)hipFree(dq); return E_OOM; }
    int rc = 0;
    if (hipMemcpy(dq, q, n * 8, hipMemcpyHostToDevice) != hipSuccess) rc = E_DEVICE;
    if (rc == 0) {
        ppsp_rootprobe_kernels::k_isqrt32<<<(uint32_t)((n + 255) / 256), 256>>>(dq, (uint32_t)n, dout);
        if (hipGetLastError() != hipSuccess || hipMemcpy(out, dout, n * 4, hipMemcpyDeviceToHost) != hipSuccess) rc = E_DEVICE;
    }
    (void)hipFree(dq);
    (void)hipFree(dout);
    return rc;
}
