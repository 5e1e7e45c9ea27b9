// Internal interface between the C-ABI entry points and the HIP kernels.
#ifndef APGEMV_KERNELS_H
#define APGEMV_KERNELS_H

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

namespace apgemv {

struct GemvArgs {
    const uint8_t *slices; // device: slice 0 of the packed matrix
    size_t slice_bytes;
    const uint16_t *lut;   // device: table of bit-width b, M * 2^b binary16
    const uint16_t *x;     // device: batch * K binary16
    uint16_t *y;           // device: batch * M binary16
    int M, K, b, batch;
    int waves_per_group;   // 0 = choose from the shape
    int row_groups_per_wg; // -1 = choose from the shape; 1 = one group of 4 rows per workgroup
    int mfma_min_batch;    // 0 = default (3); batches below it use the ALU kernels; 9 = never
    int variant;           // AP_VARIANT_*: 0 = choose; 1 = never the matrix-core kernel with in-wave exchange;
                           // 3 = that kernel whenever the shape allows it (batch >= 2, K % 128 == 0);
                           // 5 = the bank-per-lane kernel at batch 1, b >= 7;
                           // 7 / 8 = two row groups per workgroup at batch 1 whenever possible / never;
                           // 9 / 10 = the 16-row-tile matrix-core kernel (batch 2..8, K % 256 == 0) with one /
                           //          two tiles per workgroup
    void *work = nullptr;  // not null = the fused large-batch kernel, with this scratch (device, 16-byte aligned)
    size_t work_bytes = 0;
};

// The fused large-batch kernel (gemm_fused.hip) takes a product straight from the packed form.
// How it divides a product: `ntiles` tiles of up to 64 batch rows, evenly filled with `nj` times 16 rows; blocks of 64 rows;
// `waves` per workgroup; `parts` of the columns, which the scratch has room for the partial sums of; `copy_bytes` of the scratch
// hold a copy of x in fragment order (none if 0).
struct FusedPlan {
    int ntiles, nj, blocks, waves, steps, parts;
    size_t copy_bytes;
};
// Column parts (workgroups that share a row block's columns): as many as give every CU one workgroup, a step or more per wave.
// Measured, 1 / 2 / 4 / 8 parts, us: 4096 x 4096 b = 5 batch 33 (64 row blocks) 18.7 / 15.5 / 13.5 / 13.3, 8192 x 8192 b = 3
// batch 64 (128) 27.9 / 23.5 / 29.9 / 38.5, 11008 x 4096 b = 3 batch 64 (172) 18.1 / 26.9 / 29.5: a second round of workgroups
// costs more than idle CUs.
inline int fused_parts_wanted(const FusedPlan &p)
{
    const int fill = (int)(256 / ((long long)p.blocks * p.ntiles));
    const int parts = fill < p.steps / p.waves ? fill : p.steps / p.waves;
    return parts > 1 ? parts : 1;
}
inline FusedPlan fused_plan(const GemvArgs &a)
{
    FusedPlan p;
    p.ntiles = (a.batch + 63) / 64;
    p.nj = ((a.batch + 15) / 16 + p.ntiles - 1) / p.ntiles;
    p.blocks = (a.M + 63) / 64;
    // 8 waves per workgroup when every workgroup has a CU of its own, else 4 (two workgroups per CU): 28672 x 8192 b = 4 batch 64
    // 65 -> 59 us with 4, 11008 x 4096 b = 4 batch 32 17.3 -> 20.3.
    p.waves = (long long)p.blocks * p.ntiles <= 256 ? 8 : 4;
    p.steps = (a.K / 32 + 3) / 4;
    const int wanted = fused_parts_wanted(p);
    const auto parts_in = [&](size_t bytes) { // as many of them as fit
        const size_t room = bytes / ((size_t)a.batch * a.M * 4);
        return room >= (size_t)wanted ? wanted : room > 1 ? (int)room : 1;
    };
    p.parts = parts_in(a.work_bytes);
    // With 64 batch rows per workgroup the copy of x pays from the third step of a wave on (at 8 bits, whose instance with the exchange
    // spills in its loop, from the second): it is a launch of 2 to 3 us, the exchange 0.1 us per step.  With the copy / without,
    // us: 1 step 4096 x 4096 batch 64 b = 3 13.9 / 12.3, b = 8 16.3 / 15.0, 1024 x 1024 b = 5 batch 300 10.1 / 7.9; 2 steps 8192 x 4096
    // batch 64 b = 3 16.4 / 15.7, b = 5 18.7 / 18.5, b = 8 22.3 / 26.0; 4 steps 8192 x 8192 b = 5 24.8 / 24.8, 11008 x 4096 b = 8
    // 25.6 / 29.6.  The steps are those of the parts that fit, not of the wanted ones.
    const bool copy = p.nj >= 4 && p.steps > (a.b == 8 ? 1 : 2) * p.waves * p.parts;
    p.copy_bytes = copy ? (size_t)p.steps * 4 * p.ntiles * p.nj * 1024 : 0;
    if (copy) p.parts = a.work_bytes > p.copy_bytes ? parts_in(a.work_bytes - p.copy_bytes) : 1;
    return p;
}
// Whether it takes the call with a.work_bytes of scratch (always for 48 rows of an aligned x): 16-byte loads of x, whose rows are
// multiples of 64 bytes; room for the copy of x; grids within 2^32 threads and 65535 tiles of 16 batch rows.
inline bool gemm_fused_ok(const GemvArgs &a)
{
    if (reinterpret_cast<uintptr_t>(a.x) % 16 || a.batch < 1 || a.batch > 1 << 19) return false;
    const FusedPlan p = fused_plan(a);
    return p.copy_bytes <= a.work_bytes && p.copy_bytes < 0xffffffffu && (long long)p.blocks * p.ntiles <= 1 << 22;
}

constexpr int kMaxMulti = 8;
struct MultiArgs { // passed by value as the kernel argument of a fused launch
    const uint8_t *slices[kMaxMulti];
    size_t slice_bytes[kMaxMulti];
    const uint16_t *lut[kMaxMulti];
    const uint16_t *x[kMaxMulti];
    uint16_t *y[kMaxMulti];
    int M[kMaxMulti];
    int group_begin[kMaxMulti]; // first workgroup of matrix i
    int count, K, batch;
};

// Work list of gemv_list_kernel, passed by value as its kernel argument (batch 1).
constexpr int kMaxListItems = 32;
struct ListItem {
    const uint8_t *slices;
    size_t slice_bytes;
    const uint16_t *lut; // table of this item's bit-width
    const uint16_t *x;
    uint16_t *y;
    int M, K, b;
    int pad;
};
struct ListArgs {
    ListItem item[kMaxListItems];
    int group_begin[kMaxListItems]; // first workgroup of item i (filled in by the launcher)
    int count;
};

hipError_t launch_gemv(const GemvArgs &a, hipStream_t stream);
// a work list on the batch-1/2 kernel: every item at batch `batch` (1 or 2); group_begin is filled in there
hipError_t launch_gemv_list(ListArgs &a, int batch, hipStream_t stream);
hipError_t launch_gemv_multi(const MultiArgs &a, int b, int total_groups, hipStream_t stream);
// the same launch on the matrix-core kernel over tiles of 16 rows (batch 2..8, K % 256 == 0)
hipError_t launch_matrix_tile_multi(const MultiArgs &a, int b, hipStream_t stream);
// a work list on that kernel: every item at bit-width b, K % 256 == 0, all rows in the same class of length
// (below / from 12288 columns); group_begin is filled in here
hipError_t launch_matrix_tile_list(ListArgs &a, int b, int batch, hipStream_t stream);
hipError_t launch_dequantize(const GemvArgs &a, hipStream_t stream);
hipError_t launch_probe_read(const void *dev_buf, size_t bytes, hipStream_t stream);
hipError_t launch_probe_issue(int kind, int passes, hipStream_t stream);
// Looks up, once per device, the device address of the static array ap_gemm_static uses as
// its workspace (the current device's copy); called where a matrix is set up on a device.
bool static_scratch_setup();

} // namespace apgemv
#endif
