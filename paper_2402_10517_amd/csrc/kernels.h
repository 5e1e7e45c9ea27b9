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
// Whether a product of ap_gemm runs on the fused kernel rather than as ap_dequantize and one rocBLAS product.  The fused kernel
// dequantises once per 64 batch rows, at b = 3 for half the cost.  The batch lines come from 14 000 calls (18 heights 64..28672, 12 row
// lengths 256..28672, 15 batches 17..512, every b), the others from 9700 more on the kernel that copies x only where that pays (32
// heights 1..2560, 31 row lengths 32..6656, 9 batches 49..384).  Dequantise + rocBLAS / fused, us:
//   batch, by b   8192x8192 batch 256 / 384 / 512  b = 3 106/46 98/65 112/86, b = 5 110/59 101/84 113/111, b = 8 115/68 108/97 118/126
//   tall, short   the dense weights stay in the last-level cache: 28672x1024 b = 8 batch 128 / 256 38/37 43/58, b = 5 batch 320 41/49,
//                 b = 3 batch 512 47/61; 28672x8192 b = 8 batch 256 255/215
//   column parts  a workspace without room for the partial sums leaves few workgroups with all columns: 64x5632 b = 8 batch 64 (1 of 5)
//                 13/22, 256x13824 b = 8 batch 256 (1 of 13) 25/46, 400x16384 b = 5 batch 384 (1 of 6) 39/50, batch 320 (5 of 7) 32/30
//   small, b = 8  a copy of x and steps that do not divide evenly among two or three parts: 300x2304 batch 64 / 192 11.8/13.1 11.7/13.9,
//                 300x2816 12.9/14.8 12.8/16.0, 256x3584 batch 192 14.0/15.6; without the copy 300x3072 batch 64 / 192 13.3/10.8 13.5/12.3,
//                 512x256 batch 256 9.0/7.0, 256x416 batch 64 15.8/7.1; one part 512x1056 batch 128 12.4/11.1; b = 7 512x1056 12.6/9.0
inline bool gemm_fused_pays(const GemvArgs &a)
{
    const FusedPlan p = fused_plan(a);
    const int M = a.M, K = a.K;
    int most = a.b == 3 ? 512 : a.b <= 5 ? 384 : 256;
    if (a.b == 3 && M >= 24576 && K <= 2048) most = 384;
    if ((a.b == 4 || a.b == 5) && M >= 12288 && K < 8192) most = M >= 24576 && K <= 2048 ? 256 : 320;
    if (a.b == 7 && M >= 24576 && K <= 1024) most = 128;
    if (a.b == 8 && M >= 12288 && K <= 1024) most = M >= 20480 ? 128 : 192;
    if (a.b == 8 && M >= 24576 && K > 1024 && K <= 2048) most = 192;
    if (a.batch > most) return false;
    const int wanted = fused_parts_wanted(p), parts = p.parts;
    if (parts < wanted && ((4 * parts <= wanted && K <= 16384) || (a.b > 3 && parts == 1))) return false;
    return !(a.b == 8 && p.copy_bytes && M <= 768 && K > 2048 && K <= (a.batch > 128 && M <= 512 ? 4096 : 3072));
}
// Whether ap_gemm_static dequantises and runs its dense kernel (gemm_static.hip) rather than the fused kernel, whose workgroups each
// build the tables of 64 rows: where these outweigh few columns, most at 8 bits.  The dense kernel's waves read 16 rows and 16 batch rows
// each for themselves, so its time grows with their product.  From 7900 calls (heights 1..4096, row lengths 32..768, batches
// 49..5000, every b); 0.5 % of them are 3 to 17 % slower than on the other kernel where that was taken before.  Dequantise + dense
// kernel / fused, us: 64 x 32 / 64 / 96 batch 200 b = 8 5.8/6.5 6.0/6.5 6.3/6.5, b = 3 5.1/5.4 5.3/5.4 5.6/5.4, b = 5 5.6/5.8 5.8/5.8
// 6.2/5.8; 1024 x 32 b = 8 batch 200 / 500 / 1500 6.4/6.8 6.9/7.0 9.5/8.2, b = 5 batch 200 1.02 to 1; 8 x 128 batch 200 b = 8 6.0/6.5,
// b = 5 5.8/5.8; 300 x 256 batch 128 b = 8 7.9/6.9.
inline bool static_dense_pays(const GemvArgs &a)
{
    const long long waves = (long long)((a.M + 15) / 16) * ((a.batch + 15) / 16);
    if (a.batch <= 48) return false;
    if (a.M <= 8) return a.K <= 256 && waves * a.K <= 1 << 16;
    if (a.b == 8) return a.K <= (a.M <= 200 ? 128 : 96) && a.M <= 1024 && waves * a.K <= 1 << 17;
    return a.K <= (a.M <= 200 ? 64 : 32) && a.M <= 768 && waves * a.K <= 1 << 16;
}

// Whether a product at batch 2 without options runs on the kernel on tiles of 16 rows rather than on the batch-1/2 kernel, in a single call as in
// a list or fused launch (which give its bits: rows of 3072 columns and more have 4 waves, from 12288 on 8, in both).  In pairs of
// centroids (b = 4, where the lookups of the ALU kernel cost most) the tile kernel is ahead from about 2^25 weights on, but where a list or a
// fused launch holds other products as well it is one launch more, 3 to 4 us.  The line lies where that is paid for: alone / with two
// of 1024 rows in one call / with the products of a 13B layer at b = 5, ALU kernel / tile kernel, us:
//   28672x8192 38 / 29, 37.1 / 32.5, 77.0 / 71.9; 16384x8192 22.0 / 16.5, 23.9 / 22.5, 63.8 / 61.2; 20480x7168 23.1 / 18.9, 24.4 / 23.9,
//   64.1 / 63.4; 12288x11264 22.3 / 17.0, 24.7 / 24.7, 63.0 / 61.5; 8192x28672 45 / 28, -, 85.8 / 69.4
//   smaller: 8192x8192 12.2 / 9.4, 14.3 / 16.5, 54.7 / 55.6; 13824x5120 14.0 / 11.4, 15.3 / 17.5, 55.3 / 56.8; 14336x8192 -, 20.6 / 22.1, 61.9 / 60.8
//   short rows: 28672x6144 26.2 / 21.8, 26.9 / 26.6, 67.0 / 66.2; 28672x5120 23.5 / 20.2, 24.3 / 24.8, 65.1 / 64.6; 32768x4096 20.4 / 17.8, 20.8 / 22.5
//   last round of tiles (% of the CUs over all rounds): 8704x16384 (71 %) 21.3 / 20.5, 25.5 / 28.9, 61.9 / 65.6; 11008x12288 (90 %) 21.8 / 18.2,
//   24.5 / 26.2, 61.1 / 63.6
inline bool batch2_tile_pays(const GemvArgs &a)
{
    const long long tiles = (a.M + 15) / 16, rounds = (tiles + 255) / 256;
    return a.b == 4 && a.K % 256 == 0 && a.K >= 7168 && (long long)a.M * a.K >= 1 << 27 && 100 * tiles >= 91 * 256 * rounds;
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
