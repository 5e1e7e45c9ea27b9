// Large-batch product y = x W_b^T without the dense detour (Section 6.2, "Matrix-Matrix Multiplication Performance": above a
// batch of about 16 the engine dequantises with a separate kernel and runs a dense GEMM).  Writing and reading back 2 bytes
// per weight costs more than the product itself up to a batch of a few hundred, so here the lanes that dequantise feed
// v_mfma_f32_16x16x32_f16 directly.
//
//  * A workgroup owns 64 rows (16 groups of 4) x up to 64 batch rows; its waves split the columns.  A step of a wave is 4
//    chunks (128 columns): lane (i, kg) = (l % 16, l / 16) holds the 16-byte units of row group i, chunk kg, and supplies, for
//    r = 0..3 and run t, row r of its group as operand A of one instruction (16 groups x 32 columns) per 16 batch rows.  So a
//    fragment of the activations serves 4 instructions, a dequantised one up to 4, and there is no waste in the result.
//  * The units are loaded 4 lanes to 64 contiguous bytes and change to that order through a wave-private LDS buffer (one
//    ds_write_b128 + ds_read_b128 per slice).  Loaded directly in the instruction's order every lane is a cache access of its
//    own, and the vector L1 then bounds the kernel: 28672 x 8192, b = 4, batch 64: 74 -> 59 us.
//  * Activations: up to 48 batch rows per workgroup take the same way through LDS.  With 64 (batch 49..64, 97..128, 145 and more)
//    and several steps per wave a small kernel first copies x to the workspace in fragment order, and the waves read their fragments
//    as whole lines (3 us for the copy; the exchange of 4 tiles costs as much LDS time per step as the lookups): fused_plan.
//  * Tables: 32 lanes of an LDS clock = 16 row groups x 2 lane groups, each with a bank of its own: two copies per row, the rows
//    2 rp and 2 rp + 1 of a group in the halves of one dword, entries 256 bytes apart, so that one v_perm_b32 of the index byte
//    and the lane's base makes an address (64 KB at 8 bits, 8 KB at 4 and 5).  b = 3 looks up pairs.
//  * Lookups of run t + 1 are issued before the instructions of run t, loads two runs and one step ahead: at two waves per
//    SIMD there is nobody else to hide them.  In the steady state VALU (350 instructions per step) and matrix instructions
//    (64 x 16 cycles) take turns on a SIMD; neither HBM nor LDS is the limit.
#include <type_traits>
#include "device_common.h"
#include "launchers.h"

namespace apgemv {

// Tables of 64 rows in LDS.  Bank of a dword = copy * 16 + row group.
template <int B> struct BlockTable {
    static constexpr bool kPair = (B == 3);
    static constexpr uint32_t kMask = kPair ? 0xFCu : Table<B>::addr_mask(); // index bits inside a merged byte
    static constexpr int kLow = (kMask & 1) ? 0 : (kMask & 2) ? 1 : 2;       // lowest of them
    static constexpr uint32_t kClean = (kMask >> kLow) * 0x01010101u;        // index bits of the rotated words
    static constexpr int kEntries = (int)(kMask >> kLow) + 1;                // entry slots (b = 4 uses 16 of 24)
    static constexpr int kBytes = kEntries * 256 * (kPair ? 2 : 1);
    // slot of the entry stored at position p of a row (lut_stored_pos order; pair index for B = 3)
    __device__ static constexpr uint32_t slot_of(uint32_t p)
    {
        return (kPair ? p << 2 : B == 4 ? (((p & 8u) << 3) | ((p & 7u) << 2)) : p << kLow) >> kLow;
    }
    // byte offset, from a lane's entry, of row r of its group
    __device__ static constexpr int row_off(int r) { return kPair ? (r & 1) * 128 + (r >> 1) * (kEntries * 256) : (r & 1) * 2 + (r >> 1) * 128; }
    // LDS address of the entry selected by byte J of the index word w, for a lane with base `lanebase` (< 128)
    template <int J> __device__ static __forceinline__ uint32_t addr(uint32_t w, uint32_t lanebase)
    {
        return __builtin_amdgcn_perm(lanebase, w, 0x0c0c0004u | ((uint32_t)J << 8));
    }
};

struct FusedArgs {
    const uint8_t *slices;
    size_t slice_bytes;
    const uint16_t *lut, *x; // XF: x in fragment order
    uint16_t *y;
    float *partial; // parts > 1: [part][batch row][row]
    int M, K, batch, ntiles, parts;
    int share, extra; // steps of a wave: share, one more for the first `extra` waves of a row block
};

// B bits, NJ tiles of 16 batch rows per workgroup, W waves (4 or 8).  blockIdx.y: part of the columns (the parts of a row
// block are summed by reduce_parts_kernel).
template <int B, int NJ, int W, bool XF>
__global__ __launch_bounds__(64 * W, 2) void gemm_fused_kernel(FusedArgs a)
{
    using BT = BlockTable<B>;
    const uint8_t *__restrict__ slices = a.slices;
    const size_t slice_bytes = a.slice_bytes;
    const uint16_t *__restrict__ lut = a.lut;
    const uint16_t *__restrict__ x = a.x;
    uint16_t *__restrict__ y = a.y;
    const int M = a.M, K = a.K, batch = a.batch, ntiles = a.ntiles;
    constexpr int kRows = 64, kGroups = 16, kStepChunks = 4, kNT = 16 * NJ;
    constexpr int kRedRow = 16 * 16 + 16;               // bytes of one batch row of partial sums: 16 groups x 4 rows
    constexpr int kRedBytes = W * NJ * 16 * kRedRow;
    constexpr int kBounceSlices = B <= 4 ? B : (B + 1) / 2;
    constexpr int kBounce = (!XF && NJ > kBounceSlices ? NJ : kBounceSlices) * 1024;
    constexpr int kMain = BT::kBytes + W * kBounce;
    __shared__ __attribute__((aligned(16))) uint8_t smem[kMain > kRedBytes ? kMain : kRedBytes];
    uint8_t *tab = smem;
    const int tid = threadIdx.x;
    constexpr int nth = 64 * W;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    uint8_t *bounce = smem + BT::kBytes + wave * kBounce;

    // workgroup -> (row block, batch tile): the batch tiles of a row block on one XCD (ids equal mod 8), next to each other
    const int blocks = (M + kRows - 1) / kRows;
    int rb, nt;
    const int part = blockIdx.y;
    if (ntiles == 1) {
        rb = blockIdx.x;
        nt = 0;
    } else {
        const uint32_t id = blockIdx.x, per = 8 * (uint32_t)ntiles, full = (uint32_t)blocks / 8 * per;
        if (id < full) {
            rb = id / per * 8 + id % 8;
            nt = id % per / 8;
        } else {
            const uint32_t rest = (uint32_t)blocks % 8;
            rb = blocks / 8 * 8 + (id - full) % rest;
            nt = (id - full) / rest;
        }
    }
    const int groups = (M + kRowsPerGroup - 1) / kRowsPerGroup;
    const int g0 = rb * kGroups, row0 = rb * kRows, n0 = nt * kNT;
    const int nrows = batch - n0 < kNT ? batch - n0 : kNT; // batch rows of this tile
    const int chunks = K / kChunkSlots;
    const int lastspan = (chunks - 1) / kSpanLanes;
    const int ragged = chunks - lastspan * kSpanLanes;

    const __amdgpu_buffer_rsrc_t srsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t *>(slices + (size_t)g0 * chunks * 16), 0, 0xffffffffu, kBufferRsrcWord3);
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(x + (size_t)n0 * K), 0, (uint32_t)nrows * (uint32_t)K * 2u, kBufferRsrcWord3);
    const int i = lane & 15, kg = lane >> 4; // row group and chunk in the matrix instruction's order
    const int p = lane & 3, ln = lane >> 2;  // chunk and row group / batch row in load order: 4 lanes read 64 contiguous bytes
    const int gi = g0 + ln < groups ? ln : groups - 1 - g0;
    const uint32_t soff = (uint32_t)(gi * chunks + p) * 16u;
    const uint32_t bw = (uint32_t)(4 * ln + (p ^ ((ln >> 1) & 3))) * 16u, br = (uint32_t)(4 * i + (kg ^ ((i >> 1) & 3))) * 16u;
    const uint32_t lanebase = (uint32_t)(lane & 31) << 2;
    uint32_t xoff[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) xoff[j] = 16 * j + ln < nrows ? (uint32_t)(16 * j + ln) * (uint32_t)K * 2u + (uint32_t)p * 16u : 0x80000000u;

    const __amdgpu_buffer_rsrc_t xfrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(x + (size_t)nt * NJ * 512), 0, 0xffffffffu, kBufferRsrcWord3);
    u32x4 Q[B], X[2][NJ];
    auto load_q = [&](int st) {
        const int left = chunks - st * kStepChunks;
        const uint32_t off = p < left ? soff : soff - (uint32_t)(p - (left - 1)) * 16u;
        const uint32_t sst = (uint32_t)st * (kStepChunks * 16u);
#pragma unroll
        for (int s = 0; s < B; ++s) Q[s] = __builtin_amdgcn_raw_buffer_load_b128(srsrc, off, sst + (uint32_t)s * (uint32_t)slice_bytes, 0);
    };
    auto load_x = [&](int st, int t) {
        if constexpr (XF) {
            const uint32_t xs = (uint32_t)((st * 4 + t) * ntiles * NJ) * 1024u;
#pragma unroll
            for (int j = 0; j < NJ; ++j) X[t & 1][j] = __builtin_amdgcn_raw_buffer_load_b128(xfrsrc, (uint32_t)lane * 16u, xs + j * 1024u, 0);
            return;
        }
        const int span = st / (kSpanLanes / kStepChunks);
        const int nl = span == lastspan ? ragged : kSpanLanes;
        const uint32_t xs = (uint32_t)span * (kSpanCols * 2u) + (uint32_t)(st % (kSpanLanes / kStepChunks)) * (kStepChunks * 16u) + (uint32_t)(t * 16 * nl);
        const bool in = p < chunks - st * kStepChunks;
#pragma unroll
        for (int j = 0; j < NJ; ++j) X[t & 1][j] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, in ? xoff[j] : 0x80000000u, xs, 0);
    };

    float4_t acc[NJ][kRowsPerGroup];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < kRowsPerGroup; ++r) acc[j][r] = float4_t{0.f, 0.f, 0.f, 0.f};

    // the waves split the row's steps evenly (by the host's division: two 64-bit ones here were 0.3 us ahead of the first load); a
    // wave may get none (short rows)
    const int slot = part * W + wave;
    int st = slot * a.share + (slot < a.extra ? slot : a.extra);
    int st1 = st + a.share + (slot < a.extra ? 1 : 0);
    asm("" : "+s"(st), "+s"(st1)); // opaque: as products of the arguments they cost the NJ = 4 loops up to 57 spilled registers
    const bool any = st < st1;
    // Unconditional (a wave without steps loads some step and drops it): past a branch the compiler cannot tell these loads from
    // the tables' and waits for all of them before the first table entry is written (4096 x 4096 b = 3..8 batch 17, 64: 1 to 4 %).
    auto load_first = [&]() {
        const int first = any ? st : 0;
        load_q(first);
        load_x(first, 0);
        load_x(first, 1);
    };

    // ---- tables: bank = copy * 16 + group; all loads go out before the slice loads
    if constexpr (BT::kPair) {
        // thread (bank, row r, parity of the entry): 32 pair entries from the row's 8 centroids
        static_assert(nth >= 256, "4 rows x 32 banks x 2 parities");
        const int bank = tid & 31, r = (tid >> 5) & 3, e0 = (tid >> 7) & 1;
        const int row = row0 + (bank & 15) * 4 + r;
        const u32x4 c = *reinterpret_cast<const u32x4 *>(lut + (size_t)(row < M ? row : M - 1) * 8);
        load_first();
        uint32_t ev[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) ev[k] = e0 ? c[k] >> 16 : c[k] & 0xffffu;
        uint8_t *dst = tab + e0 * 256 + bank * 4 + (r & 1) * 128 + (r >> 1) * (BT::kEntries * 256);
        const int m0 = nth == 512 ? (tid >> 8) * 16 : 0; // wave-uniform
        auto fill = [&](auto first) {
#pragma unroll
            for (int m = decltype(first)::value; m < decltype(first)::value + (nth == 512 ? 16 : 32); ++m) {
                const int even = pair3_even(2 * m), odd = pair3_odd(2 * m); // the thread's parity is bit 0 of the even code
                const uint32_t hi = (odd & 1) ? c[odd >> 1] & 0xffff0000u : c[odd >> 1] << 16;
                *reinterpret_cast<uint32_t *>(dst + m * 512) = ev[even >> 1] | hi;
            }
        };
        if (m0 == 0) fill(std::integral_constant<int, 0>{});
        else fill(std::integral_constant<int, 16>{});
    } else {
        // Thread (row group, row pair, piece of 8 entries) loads for both copies: 4 lanes read 64 contiguous bytes of a row, and of
        // every two neighbours one writes its entries to the first copy first, the other to the second, which spreads a store over the
        // banks of both.  A thread per bank instead loaded every piece twice and each lane from a row of its own: 4096 x 4096
        // batch 17 b = 8 12.2 -> 11.6 us, b = 6 10.8 -> 10.4, level at b = 4, 5.
        constexpr int kPieces = (2 << B) / 16;
        constexpr int kTasks = 32 * kPieces, kPer = (kTasks + nth - 1) / nth;
        constexpr int kLanes = kPieces < 4 ? kPieces : 4; // neighbouring lanes of a row
        u32x4 lo[kPer], hi[kPer];
#pragma unroll
        for (int m = 0; m < kPer; ++m) {
            const int k = tid + m * nth < kTasks ? tid + m * nth : kTasks - 1;
            const int g = (k / kLanes) & 15, rp = (k / (kLanes * 16)) & 1, pc = k / (kLanes * 32) * kLanes + k % kLanes;
            const int ra = row0 + g * 4 + rp * 2, rlo = ra < M ? ra : M - 1, rhi = ra + 1 < M ? ra + 1 : M - 1;
            lo[m] = reinterpret_cast<const u32x4 *>(lut + ((size_t)rlo << B))[pc];
            hi[m] = reinterpret_cast<const u32x4 *>(lut + ((size_t)rhi << B))[pc];
        }
        load_first();
#pragma unroll
        for (int m = 0; m < kPer; ++m) {
            const int k = tid + m * nth;
            const int g = (k / kLanes) & 15, rp = (k / (kLanes * 16)) & 1, pc = k / (kLanes * 32) * kLanes + k % kLanes;
            if (kTasks % nth == 0 || k < kTasks) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    uint8_t *dst = tab + rp * 128 + ((c ^ (k & 1)) * 16 + g) * 4;
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        *reinterpret_cast<uint32_t *>(dst + BT::slot_of(8 * pc + e) * 256) =
                            (e & 1) ? (lo[m][e >> 1] >> 16) | (hi[m][e >> 1] & 0xffff0000u) : (lo[m][e >> 1] & 0xffffu) | (hi[m][e >> 1] << 16);
                }
            }
        }
    }
    __syncthreads();

    // a wave's private exchange of 16-byte pieces from load order to the matrix instruction's order
    auto exchange = [&](auto &v, int first, int n) {
#pragma unroll
        for (int k = 0; k < n; ++k) *reinterpret_cast<u32x4 *>(bounce + k * 1024 + bw) = v[first + k];
        wave_lds_fence();
#pragma unroll
        for (int k = 0; k < n; ++k) v[first + k] = *reinterpret_cast<const u32x4 *>(bounce + k * 1024 + br);
        wave_lds_fence();
    };
    auto exchange_q = [&]() {
        exchange(Q, 0, kBounceSlices);
        if constexpr (B > kBounceSlices) exchange(Q, kBounceSlices, B - kBounceSlices);
    };
    uint32_t Wd[kRowsPerGroup][8]; // index words of the current step
    u32x4 P[kRowsPerGroup];        // packed centroid pairs of the current run
    auto merge = [&]() {
#pragma unroll
        for (int r = 0; r < kRowsPerGroup; ++r) {
            uint32_t q[B];
#pragma unroll
            for (int s = 0; s < B; ++s) q[s] = Q[s][r];
            merge_words<B, BT::kLow>(q, Wd[r]);
            if constexpr (B < 8) {
#pragma unroll
                for (int u = 0; u < 8; u += BT::kPair ? 2 : 1) Wd[r][u] &= BT::kClean;
            }
        }
    };
    constexpr int kH = BT::kPair ? 1 : 2;
    uint32_t R[kRowsPerGroup][kH][4]; // table entries of the next run
    auto lookup = [&](int t) {
#pragma unroll
        for (int r = 0; r < kRowsPerGroup; ++r) {
            const uint8_t *tr = tab + BT::row_off(r);
#pragma unroll
            for (int h = 0; h < kH; ++h) {
                const uint32_t v = Wd[r][2 * t + h];
                const uint32_t ad[4] = {BT::template addr<0>(v, lanebase), BT::template addr<1>(v, lanebase),
                                        BT::template addr<2>(v, lanebase), BT::template addr<3>(v, lanebase)};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if constexpr (BT::kPair) R[r][h][j] = *reinterpret_cast<const uint32_t *>(tr + ad[j]);
                    else R[r][h][j] = *reinterpret_cast<const uint16_t *>(tr + ad[j]);
                }
            }
        }
    };
    auto pack = [&]() {
#pragma unroll
        for (int r = 0; r < kRowsPerGroup; ++r)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (BT::kPair) P[r][j] = R[r][0][j];
                else P[r][j] = R[r][0][j] | (R[r][1][j] << 16);
            }
    };
    auto products = [&](int t) {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < kRowsPerGroup; ++r)
                acc[j][r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, P[r]), __builtin_bit_cast(half8_t, X[t & 1][j]),
                                                                   acc[j][r], 0, 0, 0);
    };
    if (any) {
        exchange_q();
        merge();
        if (st + 1 < st1) load_q(st + 1);
        lookup(0);
        if constexpr (!XF) exchange(X[0], 0, NJ);
        pack();
    }
    for (; st + 1 < st1; ++st) {
        const int next2 = st + 2 < st1 ? st + 2 : st + 1; // the pass before the last step loads that step's units again
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (t == 2) exchange_q();
            if (t == 3) {
                merge();
                load_q(next2);
            }
            lookup((t + 1) & 3);
            products(t);
            load_x(t < 2 ? st : st + 1, (t + 2) & 3);
            if constexpr (!XF) exchange(X[(t + 1) & 1], 0, NJ);
            pack();
        }
    }
    // The wave's last step, which prepares nothing for a next one: with up to 4096 columns it is the only one, and looking up a step that
    // does not follow took 1.3 to 1.6 us of 11 to 13 (4096 x 4096, batch 17 and 33, b = 5).  Chunks past the row (a ragged step)
    // count for nothing.
    if (any) {
        const uint32_t keep = kg < chunks - st * kStepChunks ? 0xffffffffu : 0u;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
#pragma unroll
            for (int r = 0; r < kRowsPerGroup; ++r) P[r] &= u32x4{keep, keep, keep, keep};
            if (t < 3) lookup(t + 1);
            products(t);
            if (t < 2) load_x(st, t + 2);
            if (t < 3) {
                if constexpr (!XF) exchange(X[(t + 1) & 1], 0, NJ);
                pack();
            }
        }
    }

    // ---- waves are added in fixed order: element q of acc[j][r] is row group 4 kg + q (row r of it), batch row 16 j + i
    const bool wide = M % 4 == 0 && reinterpret_cast<uintptr_t>(y) % 8 == 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4_t *>(smem + ((wave * NJ + j) * 16 + i) * kRedRow + (4 * kg + q) * 16) =
                float4_t{acc[j][0][q], acc[j][1][q], acc[j][2][q], acc[j][3][q]};
    __syncthreads();
    for (int o = tid; o < 256 * NJ; o += nth) {
        const int n = o >> 4, g = o & 15;
        float4_t s = *reinterpret_cast<const float4_t *>(smem + n * kRedRow + g * 16);
#pragma unroll
        for (int w = 1; w < W; ++w) s += *reinterpret_cast<const float4_t *>(smem + (w * NJ * 16 + n) * kRedRow + g * 16);
        const int row = row0 + 4 * g;
        if (n < nrows && row < M && a.parts > 1) {
            float *dst = a.partial + ((size_t)part * batch + n0 + n) * M + row;
            if (M % 4 == 0) *reinterpret_cast<float4_t *>(dst) = s;
            else
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (row + r < M) dst[r] = s[r];
        } else if (n < nrows && row < M) {
            uint16_t *dst = y + (size_t)(n0 + n) * M + row;
            uint16_t hv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) hv[r] = __builtin_bit_cast(uint16_t, __float2half_rn(s[r]));
            if (wide) *reinterpret_cast<u32x2 *>(dst) = u32x2{hv[0] | ((uint32_t)hv[1] << 16), hv[2] | ((uint32_t)hv[3] << 16)};
            else
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (row + r < M) dst[r] = hv[r];
        }
    }
}


// x (batch x K) in the order of the matrix instruction's B operand: 1 KB per (step of 4 chunks, run, 16 batch rows), zeros
// for batch rows and chunks that do not exist.  A wave per step and tile of batch rows writes whole lines.
__global__ __launch_bounds__(256) void fragment_x_kernel(const uint16_t *__restrict__ x, u32x4 *__restrict__ xf, int K, int batch, int tiles)
{
    const int chunks = K / kChunkSlots, steps = (chunks + 3) / 4;
    const int st = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, tile = blockIdx.y;
    if (st >= steps) return;
    const int n = tile * 16 + (lane & 15), c = st * 4 + (lane >> 4);
    const int span = c / kSpanLanes, rem = chunks - span * kSpanLanes, nl = rem < kSpanLanes ? rem : kSpanLanes;
    const uint16_t *src = x + (size_t)n * K + (size_t)span * kSpanCols + (c % kSpanLanes) * 8;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        u32x4 v = {0, 0, 0, 0};
        if (n < batch && c < chunks) v = *reinterpret_cast<const u32x4 *>(src + t * 8 * nl);
        xf[((size_t)(st * 4 + t) * tiles + tile) * 64 + lane] = v;
    }
}

// y = sum of the parts, in order (n = batch * M values each).  All latency: a part's values come from beyond this XCD's L2, so the
// loads of up to 8 parts go out together.  One after the other / together, us (batch 32, b = 4): 2 parts 8192 x 4096 3.84 / 3.84, 3 parts
// 5440 x 4096 3.80 / 3.80, 4 parts 4096 x 4096 3.76 / 2.28, 8 parts 2048 x 8192 3.56 / 2.46.
__global__ __launch_bounds__(256) void reduce_parts_kernel(const float *__restrict__ partial, uint16_t *__restrict__ y, size_t n, int parts)
{
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= n) return;
    constexpr int kBurst = 8;
    if (n % 4 == 0) {
        float4_t s = {0.f, 0.f, 0.f, 0.f};
        for (int p0 = 0; p0 < parts; p0 += kBurst) {
            float4_t v[kBurst];
#pragma unroll
            for (int p = 0; p < kBurst; ++p) v[p] = *reinterpret_cast<const float4_t *>(partial + (size_t)(p0 + p < parts ? p0 + p : p0) * n + i);
#pragma unroll
            for (int p = 0; p < kBurst; ++p)
                if (p0 + p < parts) s = p0 + p ? s + v[p] : v[p];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) y[i + e] = __builtin_bit_cast(uint16_t, __float2half_rn(s[e]));
    } else {
        for (int e = 0; e < 4 && i + e < n; ++e) {
            float s = partial[i + e];
            for (int p = 1; p < parts; ++p) s += partial[p * n + i + e];
            y[i + e] = __builtin_bit_cast(uint16_t, __float2half_rn(s));
        }
    }
}

template <int B, int NJ, int W, bool XF> static hipError_t launch_fused_w(FusedArgs &a, const FusedPlan &p, uint8_t *work, hipStream_t stream)
{
    if (XF) {
        const int tiles = p.ntiles * NJ;
        hipLaunchKernelGGL(fragment_x_kernel, dim3((p.steps + 3) / 4, tiles), dim3(256), 0, stream, a.x, reinterpret_cast<u32x4 *>(work), a.K,
                           a.batch, tiles);
        a.x = reinterpret_cast<const uint16_t *>(work);
        work += p.copy_bytes;
    }
    a.partial = reinterpret_cast<float *>(work);
    hipLaunchKernelGGL((gemm_fused_kernel<B, NJ, W, XF>), dim3(p.blocks * p.ntiles, a.parts), dim3(64 * W), 0, stream, a);
    if (a.parts > 1) {
        const size_t n = (size_t)a.M * a.batch;
        hipLaunchKernelGGL(reduce_parts_kernel, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, stream, a.partial, a.y, n, a.parts);
    }
    return hipGetLastError();
}

template <int B, int NJ> static hipError_t launch_fused_nj(FusedArgs &a, const FusedPlan &p, uint8_t *work, hipStream_t stream)
{
    if constexpr (NJ == 4) {
        if (p.copy_bytes) return p.waves == 8 ? launch_fused_w<B, NJ, 8, true>(a, p, work, stream) : launch_fused_w<B, NJ, 4, true>(a, p, work, stream);
    }
    return p.waves == 8 ? launch_fused_w<B, NJ, 8, false>(a, p, work, stream) : launch_fused_w<B, NJ, 4, false>(a, p, work, stream);
}

template <int B> static hipError_t launch_fused_b(FusedArgs &a, const FusedPlan &p, uint8_t *work, hipStream_t stream)
{
    switch (p.nj) {
    case 1:
    case 2: return launch_fused_nj<B, 2>(a, p, work, stream);
    case 3: return launch_fused_nj<B, 3>(a, p, work, stream);
    }
    return launch_fused_nj<B, 4>(a, p, work, stream);
}

hipError_t launch_gemm_fused(const GemvArgs &g, hipStream_t stream)
{
    if (!gemm_fused_ok(g)) return hipErrorInvalidValue;
    const FusedPlan p = fused_plan(g);
    const int slots = p.parts * p.waves;
    FusedArgs a = {g.slices, g.slice_bytes, g.lut, g.x, g.y, nullptr, g.M, g.K, g.batch, p.ntiles, p.parts, p.steps / slots, p.steps % slots};
    uint8_t *w = static_cast<uint8_t *>(g.work);
    switch (g.b) {
    case 3: return launch_fused_b<3>(a, p, w, stream);
    case 4: return launch_fused_b<4>(a, p, w, stream);
    case 5: return launch_fused_b<5>(a, p, w, stream);
    case 6: return launch_fused_b<6>(a, p, w, stream);
    case 7: return launch_fused_b<7>(a, p, w, stream);
    case 8: return launch_fused_b<8>(a, p, w, stream);
    }
    return hipErrorInvalidValue;
}

} // namespace apgemv
