// Bit-width and kernel-family dispatch of one ap_gemv call: one stored matrix, the kernel and the
// table are chosen per call (Section 5.2: only the first b slices and the b-bit table are touched).
#include "launchers.h"
#include "layout.h"

namespace apgemv {

// Whether the matrix-core kernel on tiles of 16 rows is the fastest for a call without tuning overrides.  Time of the kernels below
// (batch 9 and more: in two passes) over its time, at M x K and b = 3 / 5 / 8, from 9270 calls at batch 3..8 (14 heights, 23 row
// lengths) and 5500 at 9..16:
//   batch 9       1024x4096 1.30/1.23/1.09  1024x8192 1.04/0.95/-  1024x20480 0.97/0.91/0.85  512x1024 1.80/1.26/1.47  2048x20480 1.32/1.23/1.15
//   batch 16      1024x11008 1.37/1.25/1.08  1024x4192 1.27/1.02/0.93  4096x4096 1.58/1.62/1.68  28000x4192 3.59/3.16/2.36
//   batch 5       1024x4096 1.08/0.92/0.77  2048x1024 1.25/0.92/0.94  2048x4192 1.13/0.95/0.78  2048x8224 1.16/0.95/0.79
//                 3072x1024 1.32/0.96/1.01  3072x4096 1.60/1.38/1.18  5120x2208 1.38/1.22/0.95  28000x2208 2.52/2.02/1.50
//   batch 3, 4    3072x4096 1.14/1.01/0.95  3072x8192 1.06/0.92/0.88  3072x11008 1.31/1.36/1.04  3072x16384 1.15/1.27/0.95
//                 4096x4096 1.24/1.08/1.04  4096x8192 1.19/1.06/1.02  4096x11008 1.88/1.69/1.47  4096x12416 1.32/1.48/0.98
//                 5120x4096 0.96/0.86/0.83  5120x8192 0.94/0.80/0.78  5120x11008 1.33/1.32/1.05  5120x13824 1.10/1.30/0.86
//                 6144x4096 1.07/0.94/0.94  6144x8192 1.02/0.89/0.88  6144x11008 1.50/1.52/1.16  6144x13824 1.45/1.52/1.12
//                 8192x4096 1.18/1.16/1.28  8192x4224 1.21/1.06/1.06  8192x8192 1.21/1.09/1.20  8192x16384 1.63/1.76/1.25
//   batch 2       4096x4096 1.01/0.95/0.92  6144x11008 0.77/0.77/0.77
// Where the ALU kernel is close, three things decide: the CUs that the last round of tiles leaves idle (5120 rows are 320 tiles, 1.25
// rounds; `busy` below), the last span of the ALU kernel's rows (whole at 8192 and 16384 columns; at b >= 7 it gains again beyond 6
// spans), and whether the row ends inside 128 columns (the last octet is then mostly padding, and the other kernel is the ALU kernel
// at every height).  From another 11000 calls at batch 4, 6, 8 (24 heights 3072..12200, 34 row lengths), batch 4, b = 7: 5100 / 6300 /
// 7600 x 8224 1.02/1.24/1.37  x 11808 0.90/1.04/1.17  x 15808 0.70/0.85/0.92  x 18432 0.98/1.20/1.28, 8600 / 10600 x 15808 0.76/0.90;
// b = 8: 5700 / 6300 x 13056 1.06/1.14, 6700 / 7600 x 8192 0.89/1.01; b = 3: 5100 / 5400 x 8192 0.92/1.01, 8600 / 9800 x 7200 0.89/1.0;
// batch 8, b = 8: 5100 / 6300 x 2208 0.93/1.08  x 7200 0.83/0.98  x 10400 0.98/1.21, 5700 x 2016 0.85.  b = 4 always wins there
// (1.0 to 2.4).  What is left of calls slower than without this kernel: 1.3 % of them by 3 to 12 %.
static bool tile_pays(const GemvArgs &a)
{
    const int groups = padded_rows(a.M) / kRowsPerGroup, b = a.b, K = a.K;
    if (a.batch >= 9)
        return groups >= 512 || (groups >= 256 && b <= 5 && K <= 12288 && (b <= 4 || K <= 4096 || a.batch >= 13)) ||
               (groups >= 128 && K <= 1024);
    if (a.batch < 3) return false;
    const long long tiles = (a.M + 15) / 16, rounds = (tiles + 255) / 256;
    auto busy = [&](int percent) { return 100 * tiles >= percent * 256 * rounds; }; // of the CUs, over the rounds
    const bool ragged = K % 128 != 0;
    if (a.batch >= 5) {
        if (groups < 512 || (groups < 768 && b > 3)) return false;
        if (!ragged || groups >= 2048 || b < 7) return true;
        if (K <= 2048) return K <= (b == 8 ? 1024 : 1536);
        if (b == 7) return (K <= 2560 || (K > 4096 && K <= 5376) || (K > 8192 && K <= 12800)) || busy(65);
        if (rounds == 1 && K > 4096 && K <= 8192) return busy(80);
        return (K > 8192 && K <= 11264) || busy(65);
    }
    if (groups >= 2048) {
        if (b >= 7 && K > 8192 && ragged) return groups >= 3072 || (K <= 12288 && (K <= 9472 || busy(75)));
        return K >= 8192 || K % 256 == 0 || (b == 3 && busy(78));
    }
    if (groups < 768 || K < 4096 || (K < 8192 && (K % 256 || b > 4))) return false;
    if (b == 4) return true;
    if (b == 3) return K > 8192 || busy(65);
    if (b <= 6) return K > 8192 || busy(80);
    if (K <= 8192) return busy(85);
    if (rounds == 1) return (K <= 12288 && !ragged) || (busy(80) && (K <= 12288 || !ragged));
    if (ragged) return K <= 12288 && (K <= 9472 || busy(75));
    return K <= 12288 || busy(68);
}

hipError_t launch_gemv(const GemvArgs &a, hipStream_t stream)
{
    if (a.b < 3 || a.b > 8) return hipErrorInvalidValue;
    const int B = a.b;
    if (a.work) return launch_gemm_fused(a, stream);
    // Bank-per-lane lookups at batch 1, b = 7, 8: conflict-free, but two operations per table address
    // and 8 copies of every table; measured slower than the shared-table kernel on every Llama shape
    // (b = 8: 8.2 / 17.7 / 19.6 us against 6.8 / 12.0 / 12.7 us on the 7B shapes), so only on request.
    if (a.batch == 1 && B >= 7 && a.variant == 5) return launch_quad(a, stream);
    // variant: 9 / 10 = the kernel on tiles of 16 rows with one / two tiles per workgroup at K % 256 == 0; any other tuning
    // override keeps the call away from it.
    const bool tuned = a.variant != 0 || a.row_groups_per_wg >= 0 || a.mfma_min_batch != 0 || a.waves_per_group != 0;
    const bool forced = (a.variant == 9 || a.variant == 10) && a.K % 256 == 0;
    if (a.batch > kMaxMulti) {
        if (!tuned && tile_pays(a)) return launch_matrix_tile(a, stream);
        // the other kernels take up to 8 activation rows: two passes
        GemvArgs pass = a;
        pass.batch = kMaxMulti;
        const hipError_t e = launch_gemv(pass, stream);
        if (e != hipSuccess) return e;
        pass.x = a.x + (size_t)kMaxMulti * a.K;
        pass.y = a.y + (size_t)kMaxMulti * a.M;
        pass.batch = a.batch - kMaxMulti;
        return launch_gemv(pass, stream);
    }
    if (a.batch >= 2 && (forced || (!tuned && tile_pays(a)))) return launch_matrix_tile(a, stream);
    // What is left for batch >= 2: the plain ALU kernel at batch 2 (fastest everywhere), on smaller matrices, and at batch 3, 4 on ragged
    // rows below 8192 columns (b >= 4), where the matrix-core kernel with in-wave exchange takes those of a multiple of 128 columns
    // from 2048 row groups on at b >= 6, from 4096 on at b = 4, 5 too (up to 24 % faster than the ALU kernels).  A handle with
    // an option stays away from the tile kernel; for it the rules of the exchange kernel reach further: batch 5..8 at every b, and
    // one wave per span at batch 3, 4.
    // variant: 1 = never the in-wave-exchange kernel, 3 = whenever the shape allows (tuning overrides).
    if (a.batch >= 2 && a.K % 128 == 0 && a.variant != 1) {
        const int groups = padded_rows(a.M) / kRowsPerGroup;
        const int nspans = (a.K / kChunkSlots + kSpanLanes - 1) / kSpanLanes;
        const bool one_wave_per_span = nspans <= 8;
        bool pays = false;
        if (groups >= 2048 && a.row_groups_per_wg < 0 && a.mfma_min_batch == 0) {
            if (a.batch >= 5) pays = true;
            else if (a.batch >= 3 && one_wave_per_span) pays = B >= 6 || (B >= 4 && groups >= 4096);
        }
        if (a.variant == 3 || pays)
            return launch_matrix_exchange(a, stream);
    }
    // The first matrix-core kernel (one row per lane) is reached by handles with options only: batch 3..8 at b >= 6 when the row
    // length allows it; at b <= 5 the four rows' small tables of a block share LDS banks and it is slower.  Matrices
    // with fewer than 2048 groups of rows stay on the ALU kernels: measured on 4096x4096 and 4096x11008
    // at batch 3, 4, 8 the ALU kernels are level or up to 30 % faster there (the device is not full,
    // and a call is bound by latency, not by the multiply-accumulates the matrix cores take over).
    // (mfma_min_batch: tuning override, also of the size rule; a negative value lifts the b limit too.)
    const int min_batch = a.mfma_min_batch > 0 ? a.mfma_min_batch : a.mfma_min_batch < 0 ? -a.mfma_min_batch : 3;
    const bool big_enough = a.mfma_min_batch != 0 || padded_rows(a.M) / kRowsPerGroup >= 2048;
    if (a.batch >= min_batch && a.K % 128 == 0 && big_enough && (B >= 6 || a.mfma_min_batch < 0))
        return launch_matrix_row_per_lane(a, stream);
    return launch_alu(a, stream);
}

} // namespace apgemv
