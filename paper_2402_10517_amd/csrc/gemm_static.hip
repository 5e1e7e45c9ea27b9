// Large-batch path for callers that cannot allocate device memory: ap_gemm with its workspace in a static device array.
//
// ap_gemm takes the workspace from the caller and hands large batches to rocBLAS, whose first use
// allocates.  Code under HIP graph capture, tight serving loops and harnesses that forbid
// hipMalloc need an entry point that allocates nothing at all: the fused kernel (gemm_fused.hip) takes
// every batch above 16 here, with its copy of the activations and its partial sums in `scratch` below (one copy per
// GPU, held until the process ends).  Against dequantising into the array and a dense kernel, 4096 x 4096 b = 5 batch 33:
// 61 -> 14 us.
#include <hip/hip_runtime.h>

#include <mutex>

#include "../../include/apgemv.h"
#include "handle.h"
#include "kernels.h"

namespace apgemv {

// Workspace of one call.  In host code this name is only a stand-in for the device
// symbol: the device address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) uint8_t scratch[AP_GEMM_STATIC_MAX_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_lock;
void *g_scratch_ptr[kMaxDevices]; // device address of `scratch` on each device, 0 = not asked yet

// Address of this device's copy of `scratch` (each GPU holds its own copy at its own address).
void *scratch_on_current_device()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> guard(g_lock);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}

} // namespace

bool static_scratch_setup() { return scratch_on_current_device() != nullptr; }

} // namespace apgemv

using namespace apgemv;

extern "C" ap_status ap_gemm_static(const ap_matrix *h, int b, const void *x_dev, void *y_dev, int batch,
                                    void *stream)
{
    if (!handle_ok(h) || !x_dev || !y_dev) return AP_ERR_INVALID_ARG;
    if (b < AP_MIN_BITS || b > h->hdr.n || !(h->hdr.lut_mask & (1u << b))) return AP_ERR_BITS;
    if (batch < 1 || batch > (1 << 20)) return AP_ERR_BATCH;
    if (reinterpret_cast<uintptr_t>(x_dev) % 16 || reinterpret_cast<uintptr_t>(y_dev) % 2) return AP_ERR_INVALID_ARG;
    const size_t need = (size_t)h->hdr.M * (size_t)h->hdr.K * 2;
    if (need > (size_t)AP_GEMM_STATIC_MAX_BYTES) return AP_ERR_BUFFER_TOO_SMALL;
    if ((long long)((h->hdr.M + 15) / 16) * ((batch + 15) / 16) > 0x7fffffffLL / 64) return AP_ERR_BATCH; // no such y exists
    void *work = scratch_on_current_device();
    if (!work) return AP_ERR_HIP;

    GemvArgs a;
    a.slices = h->dev + h->hdr.slice_off;
    a.slice_bytes = h->hdr.slice_bytes;
    a.lut = reinterpret_cast<const uint16_t *>(h->dev + h->hdr.lut_off[b]);
    a.M = h->hdr.M;
    a.K = h->hdr.K;
    a.b = b;
    a.waves_per_group = 0;
    a.row_groups_per_wg = -1;
    a.mfma_min_batch = 0;
    a.variant = 0;
    a.work_bytes = AP_GEMM_STATIC_MAX_BYTES;
    // up to 16 rows on the kernels of ap_gemv; else as many batch rows at a time as the array has room for (at least 48:
    // those need no copy of x)
    for (int first = 0; first < batch;) {
        a.x = static_cast<const uint16_t *>(x_dev) + (size_t)first * a.K;
        a.y = static_cast<uint16_t *>(y_dev) + (size_t)first * a.M;
        a.batch = batch - first < kMaxFusedBatch ? batch - first : kMaxFusedBatch;
        while (a.batch > 48 && !gemm_fused_ok(a)) a.batch = a.batch > 96 ? a.batch / 2 : 48;
        a.work = a.batch > AP_MAX_BATCH ? work : nullptr;
        if (launch_gemv(a, static_cast<hipStream_t>(stream)) != hipSuccess) return AP_ERR_HIP;
        first += a.batch;
    }
    return AP_OK;
}
