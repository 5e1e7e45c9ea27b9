// Bit-width and kernel-family dispatch of one ap_gemv call: one stored matrix, the kernel and the
// table are chosen per call (Section 5.2: only the first b slices and the b-bit table are touched).
#include "launchers.h"
#include "layout.h"

namespace apgemv {

// Whether the matrix-core kernel on tiles of 16 rows is the fastest for a call without tuning overrides.  Time of the kernels below
// over its time, at M x K, from 21 000 calls (37 heights 256..28672, 55 row lengths 256..28672, every b, batch 3, 4, 5, 8) and 5200 at batch 9, 16:
//   batch 16      b = 3/5/8   512x1120 1.71/1.90/1.75  512x7200 1.28/1.22/1.00  2048x9312 1.53/1.63/1.41
//   batch 9       512x1120 1.57/1.66/1.57  512x7200 1.08/1.02/0.87  2048x4640 1.40/1.40/1.32
//   batch 5       512x2048 1.20/1.08/1.03  512x4096 1.10/0.98/0.91  1536x4096 1.43/1.30/1.22  1536x8192 1.31/1.08/1.00
//                 1536x8224 1.24/0.99/0.98  1536x11008 1.53/1.21/1.15  3072x1024 1.35/1.10/1.17  3072x8192 1.75/1.51/1.36
//   batch 3, 4    2048x4096 1.08/1.00/0.97  3072x4096 1.16/1.09/1.11  3072x5120 1.13/0.89/0.95  3072x11008 1.50/1.55/1.24
//                 4096x4096 1.27/1.19/1.23  4096x8192 1.29/1.17/1.08  4096x8224 1.94/1.59/1.51  4352x4096 1.08/0.96/0.96
//                 5120x8192 1.11/0.94/0.94  6144x4096 1.24/1.06/1.09  7168x8192 1.39/1.19/1.15  8192x3744 1.24/1.13/0.99
//                 b = 4 2048x4096 1.18  1536x8224 1.15  3072x1024 0.94  3072x4096 1.27  4352x512 1.05
//   in us: 4096x4096 b = 8 batch 4 7.66 / 6.16, 2048x4096 b = 5 batch 8 7.14 / 5.52, 1536x11008 b = 4 batch 8 11.54 / 8.02, 14336x640 b = 7
//   batch 4 17.7 / 6.1, 4096x8224 b = 5 batch 3 16.3 / 10.3, 512x1120 b = 5 batch 16 9.4 / 5.2
// What decides where the other kernel is close: the CUs that the last round of tiles leaves idle (5120 rows are 320 tiles, 1.25 rounds;
// `busy` below), whether the last octet of a row is partly padding (`whole`, `half`), how much of the call is building the tables (short
// rows; by b), the ALU kernel's second round of spans from 8193 columns on, and its batch: it takes the same time at 5 to 8 rows, the tile
// kernel grows with them.  On ragged rows at b = 7, 8 up to 1280 row groups are one round of the ALU kernel's workgroups (5 per CU) and more
// than one of tiles (`one_alu_round`); it is then ahead the more of its last span is filled and the higher b and batch are, ALU / tile kernel:
// 4384x24288 b = 8 batch 5..8 0.92 0.88 0.87 0.83, b = 7 0.97 0.93 0.92 0.88, but 4798x26592 b = 7 batch 5 1.1; 4978x7648 b = 3 batch 4 0.88.
// At batch 9 and more the other kernel takes two passes, of which the second costs as much as the first from 13 on (two passes / tile, below
// 320 row groups at 6 to 8k columns b = 7, 8 0.92 at batch 9, 0.99 at 12, 1.09 at 13 and 16).
// Over the 21 000 calls this rule loses 0.1 to 0.8 % (by b and batch) against the better kernel of each; where it keeps to the ALU kernel for
// simplicity the tile kernel is ahead by up to 1.3 (b = 4, batch 5 to 8, 512x28672 15.6 / 12.0) and, at batch 9 and more below 64 row
// groups, 1.9 to 2.3 (182x256 b = 3).  512 rows stand for fewer: up to 1024 every tile has a CU to itself.
static bool tile_pays(const GemvArgs &a)
{
    const int groups = padded_rows(a.M) / kRowsPerGroup, b = a.b, K = a.K;
    if (a.batch >= 9) {
        if (groups >= 320) return true;
        return groups >= 64 && (a.batch >= 13 ? K <= 12288 || b <= 6 : K <= 5632 || (b <= 5 && K <= 12288));
    }
    const long long tiles = (a.M + 15) / 16, rounds = (tiles + 255) / 256;
    auto busy = [&](int percent) { return 100 * tiles >= percent * 256 * rounds; }; // of the CUs, over the rounds
    const bool whole = K % 256 == 0, half = K % 128 == 0, one_alu_round = groups <= 1280;
    if (a.batch == 2) return batch2_tile_pays(a);
    if (a.batch < 2) return false;
    if (a.batch >= 5) {
        if (groups >= 640) {
            if (half || b < 7 || K <= 5632 || rounds != 2) return true;
            if (K <= 8192 && !busy(58)) return false;
            return !one_alu_round || (K > 8192 && K <= 12800) || K % 2048 < 256 * (33 - 2 * (b + a.batch));
        }
        if (b == 3 && a.batch == 8 && groups < 512 && K > 12288 && !whole && K % 2048 >= 1024) return false;
        if (groups >= 320) return K <= 4096 || b <= 4 || (K > 8192 && whole && (b <= 6 || K <= 12288));
        if (!whole) return groups >= 64 && K <= (b == 3 ? 1536 : 512);
        return groups >= 64 && K <= (b <= 4 ? 4096 : b == 6 ? 512 : 2048);
    }
    if (b == 3) {
        if (groups >= 640) return whole || K <= 5632 || K > 8192 || rounds != 2 || !one_alu_round;
        if (groups >= 64 && K <= 512) return true;
        return whole && groups >= 64 && (K <= 2048 || (groups >= 320 && (K <= 4096 || (K > 8192 && K <= 13824))));
    }
    if (b == 4) return groups >= 1088 || (groups >= 640 && K > 2048) || (groups >= 320 && (whole ? K > 2560 : K > 9216));
    if (half && groups >= 2048) return true; // the kernel with in-wave exchange is the other one: 14336x640 b = 8 2.7, 8192x8320 b = 5 1.95
    if (K <= 512) return groups >= (b >= 7 ? 320 : 1088);
    if (K <= 2048) return whole ? groups >= (b <= 6 ? 1792 : 1088) : b == 5 && groups >= 2048 && K <= 1536;
    if (groups < 640) return false;
    if (rounds == 1) {
        if (K <= 4096) return b != 6 || groups >= 896 || whole;
        if (K <= 8192) return groups >= 896 && (whole || (b <= 6 && K > 5632));
        return b <= 6 || K <= (groups > 768 ? 12288 : 11264) || half;
    }
    if (K <= 8192) return whole ? busy(69) : b <= 6 && busy(b == 5 ? 85 : 95);
    return b <= 6 || K <= (whole || busy(68) ? 12288 : 11264) || busy(whole ? 60 : 85);
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
    // What is left for batch >= 2: the plain ALU kernel on what tile_pays refuses.  The matrix-core kernel with in-wave
    // exchange takes calls of handles with an option only: batch 5..8 at every b and, where every span has a wave, batch 3, 4 at b >= 6
    // (b = 4, 5 from 4096 row groups on), from 2048 row groups on at K % 128 == 0.
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
