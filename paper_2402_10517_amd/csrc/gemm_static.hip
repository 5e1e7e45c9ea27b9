// Large-batch path for callers that cannot allocate device memory: ap_gemm with its workspace in a static device array.
//
// ap_gemm takes the workspace from the caller and hands large batches to rocBLAS, whose first use
// allocates.  Code under HIP graph capture, tight serving loops and harnesses that forbid
// hipMalloc need an entry point that allocates nothing at all: the fused kernel (gemm_fused.hip) takes batches above 16
// here, with its copy of the activations and its partial sums in `scratch` below (one copy per GPU, held until the process
// ends).  Against dequantising into the array and the dense kernel below, 4096 x 4096 b = 5 batch 33: 61 -> 11 us.  The
// dense kernel keeps products of very few columns (static_dense_pays).
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

typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// The product over dequantised weights, where the tables of 64 rows that every workgroup of the fused kernel builds outweigh the
// columns they serve.  y[t][i] = sum_k w[i][k] * x[t][k]: one wave per tile of 16 output rows x 16 batch rows.  In
// v_mfma_f32_16x16x16_f16 lane l supplies A[l % 16][4 (l / 16) .. + 3] and B[4 (l / 16) .. + 3][l % 16]
// and receives D[4 (l / 16) .. + 3][l % 16].  Which four k a lane group contributes is free as long
// as A and B agree, so group g takes the 8 consecutive k of a 16-byte load in two instructions.
// K % 32 == 0 (guaranteed by the packed format).
__global__ __launch_bounds__(256) void dense_gemm_kernel(const uint16_t *__restrict__ w, const uint16_t *__restrict__ x,
                                                         uint16_t *__restrict__ y, int M, int K, int batch, int row_tiles,
                                                         int tiles)
{
    const int tile = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
    if (tile >= tiles) return; // whole waves
    const int rt = tile % row_tiles, bt = tile / row_tiles;
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int row = rt * 16 + r, t = bt * 16 + r;
    const u32x4 *wp = reinterpret_cast<const u32x4 *>(w + (size_t)(row < M ? row : M - 1) * K) + g;
    const u32x4 *xp = reinterpret_cast<const u32x4 *>(x + (size_t)(t < batch ? t : batch - 1) * K) + g;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < K / 8; k += 4) {
        const u32x4 a = wp[k], b = xp[k];
        const u32x2 a0 = {a[0], a[1]}, a1 = {a[2], a[3]}, b0 = {b[0], b[1]}, b1 = {b[2], b[3]};
        acc = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4, a0), __builtin_bit_cast(f16x4, b0), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4, a1), __builtin_bit_cast(f16x4, b1), acc, 0, 0, 0);
    }
    if (t < batch) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int orow = rt * 16 + 4 * g + j;
            if (orow < M) {
                const _Float16 h = (_Float16)acc[j];
                y[(size_t)t * M + orow] = __builtin_bit_cast(uint16_t, h);
            }
        }
    }
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
    a.x = static_cast<const uint16_t *>(x_dev);
    a.y = static_cast<uint16_t *>(y_dev);
    a.batch = batch;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (static_dense_pays(a)) { // M * K fits the array (above)
        a.y = static_cast<uint16_t *>(work);
        if (launch_dequantize(a, st) != hipSuccess) return AP_ERR_HIP;
        const int row_tiles = (a.M + 15) / 16, tiles = row_tiles * ((batch + 15) / 16);
        hipLaunchKernelGGL(dense_gemm_kernel, dim3((tiles + 3) / 4), dim3(256), 0, st, static_cast<const uint16_t *>(work), a.x,
                           static_cast<uint16_t *>(y_dev), a.M, a.K, batch, row_tiles, tiles);
        return hipGetLastError() == hipSuccess ? AP_OK : AP_ERR_HIP;
    }
    a.work_bytes = AP_GEMM_STATIC_MAX_BYTES;
    // up to 16 rows on the kernels of ap_gemv, unless that means two passes over a tiny matrix (64x256 b = 3 batch 16 8.9 us, fused 5.0)
    const int gemv_rows = a.K <= 256 && a.M < 512 ? AP_MAX_BATCH / 2 : AP_MAX_BATCH;
    // the others in as few passes as keep the copy of x within 16 MB, 8 MB with more than 32 row blocks, which all read it: passes
    // of 512 rows / as many as that, us: 16x256 b = 3 batch 4096 62/9, 512x4096 b = 5 batch 1024 40/27, 4096x512 batch 4096 98/70; but
    // all rows in one pass at 33 and 17 MB: 2048x8192 b = 3 batch 2048 125/165, 4096x4096 119/161
    const int steps = (a.K / 32 + 3) / 4;
    const int most = (int)((size_t)(a.M <= 32 * 64 ? 1 << 24 : 1 << 23) / ((size_t)steps * 256));
    const int passes = (batch + (most > 512 ? most : 512) - 1) / (most > 512 ? most : 512);
    const int rows = ((batch + passes - 1) / passes + 63) / 64 * 64;
    for (int first = 0; first < batch;) {
        a.x = static_cast<const uint16_t *>(x_dev) + (size_t)first * a.K;
        a.y = static_cast<uint16_t *>(y_dev) + (size_t)first * a.M;
        a.batch = batch - first < rows ? batch - first : rows;
        while (a.batch > 48 && !gemm_fused_ok(a)) a.batch = a.batch > 96 ? a.batch / 2 : 48; // (at 48 rows no copy of x)
        a.work = a.batch > gemv_rows ? work : nullptr;
        if (launch_gemv(a, st) != hipSuccess) return AP_ERR_HIP;
        first += a.batch;
    }
    return AP_OK;
}
