// Small-batch kernel (batch 2..16) that feeds v_mfma_f32_16x16x32_f16 from the dequantising lanes
// (Section 6.2 "Matrix-Matrix Multiplication Performance": the paper's kernel runs batches on the
// ordinary ALUs and slows down by up to 2x at batch 8).
//
// In that instruction lane l supplies A[l % 16][8 (l / 16) .. + 7] and B[8 (l / 16) .. + 7][l % 16] and
// receives D[4 (l / 16) .. + 3][l % 16].  With A = weights and B = activations this fixes who owns
// what: lane (i, kg) = (l % 16, l / 16) dequantises row i of a tile of 16 rows, 8 columns per
// instruction; the multiply-accumulate cost does not depend on the batch.
//   * A wave works on octets of chunks (8 chunks = 256 columns of the tile's 16 rows): two quads of
//     chunks, lane group kg taking chunk kg of the first and chunk 4 + kg of the second.
//   * Every load of slices reads whole 128-byte lines in lane order: 2 row groups x 8 chunks x 4 rows (lane 32 p + 4 c + r: group p,
//     chunk c, row r), two loads per slice and tile.  The words go to the lanes that dequantise them (lane 16 kg + 4 g + r: group g, row
//     r; chunk 4 h + kg of quad h) through 1 KB of LDS per wave, two slices at a time: two ds_write2st64_b32 and two ds_read2st64_b32.
//     A permlane16_swap (12 clocks of its SIMD) and two ds_bpermute (6 of the LDS each) per slice before that, us: 28672 x 8192 batch 8
//     b = 4/5/7 31.8/39.9/46.8 -> 31.1/38.4/45.4, 4099 x 2208 b = 7 batch 5 7.24 -> 6.92, 4096 x 4096 b = 8 batch 8 7.36 -> 7.12.
//     Loaded directly in the order of use, every 4 lanes touch another cache line and a line is requested again while it is still in
//     flight; 64-byte pieces of all 4 row groups, which need no swap, are 10 to 15 % slower for that reason too.
//   * The activations of a run go into the matrix instruction as they are loaded: lane 16 kg + 2 n + h loads the 16 bytes of batch
//     row n, chunk 4 h + kg, so column 2 n + h of operand B belongs to batch row n and quad h.  Both quads of an octet multiply with
//     that one register: of either product the columns of its own quad count, the others are dropped, and a final sum adds the two
//     columns of a batch row.  A load in this order costs the vector L1 33 clocks instead of 17 (16 bytes of four neighbouring lanes are
//     64 contiguous ones there, here 32), but it replaces 4 ds_bpermute per run, and the LDS was the busiest unit: it alone took 29 of
//     37 us that 28672 x 8192, b = 5, batch 8 needs without its loads.  With the exchange / without, us: 8192 x 28672 b = 3 batch 8
//     26.0 / 23.2, 28672 x 8192 b = 4 batch 4 32.9 / 26.5, b = 5 batch 8 42.7 / 41.0, b = 8 53.2 / 51.3, 4096 x 4096 b = 4 batch 4
//     5.4 / 4.95.  Batch rows that do not exist read zeros (their buffer offset is out of range: no memory traffic).
//   * Batch 9..16 (WIDE): two such registers, rows 0..7 and 8..15, and twice the matrix instructions (11008 x 4096 b = 4 batch 16
//     14.7 / 13.05, 28672 x 8192 b = 3 38.8 / 33.8).
//   * One instruction takes one run of 8 consecutive columns: their indices are the bytes of the
//     merged words of the run's even and odd slots, the activations the lane's 16 bytes of that run.
//   * The LDS serves 32 lanes per clock, here 16 rows x 2 lane groups, so every (row, lane group
//     parity) gets a bank of its own: each row's table is stored twice, entry v of row i for lane
//     groups of parity c is the low half of the dword at (v << s) | (c << 6) | (i << 2); no two lanes
//     of a clock share a bank.  For b <= 7, s = 8 and v = the index byte shifted down to its lowest
//     used bit (the index words are rotated that much further and masked, once per 4 lookups), so
//     that one v_perm_b32 per lookup builds the address from the word's byte and the lane's base; for
//     b = 8 that would need 64 KB per tile, so s = 7 and v_dot4_u32_u8 multiplies the wanted byte by 128, the
//     others by 0 and adds the lane's base (a byte select and a shift-or before: 28672 x 8192 batch 8 54.2 -> 51.1 us,
//     decoder layer batch 4 54.3 -> 51.6).  The 3-bit path keeps its 64-entry table of centroid pairs, one pair
//     per dword.  The 4-bit path looks pairs up as well: slice 3 is rotated to rotation 0 so that a
//     merged byte is the 8-bit index of a column pair (8 selects and 4 rotates per 32 weights instead
//     of 14 and 7, no clean-up), a row's 256 pair entries are built in LDS from its 16 stored
//     centroids, two copies, entry p of row i at (p << 7) | (c << 6) | (i << 2) (v_dot4_u32_u8 here too; no pack before the
//     matrix instruction).  Here that pays (same box,
//     alternating runs at batch 8: 28672 x 8192 46 -> 39 us, 8192 x 8192 16 -> 13.5, 8192 x 28672
//     46 -> 36), once the table build is cheap (below); in the batch-1 kernel, where all 64 lanes gather
//     from one row's 256 dwords, the bank conflicts eat the gain.
// Rows that are not a multiple of 256 columns end with an octet of fewer chunks (RAG: chunks that do not exist load the last
// one again, their centroids are masked to zero before the matrix instruction and their activations read as zeros; one fast
// operation per pair of columns).
#include <type_traits>
#include "device_common.h"
#include "launchers.h"

namespace apgemv {

template <int B> struct TileTable {
    static constexpr bool kPair = (B == 3);
    // 4 bits: a 256-entry table of centroid pairs per row, two copies like the other tables: entry p of row i
    // for lane groups of parity c at (p << 7) | (c << 6) | (i << 2)
    static constexpr bool kPair4 = (B == 4);
    static constexpr uint32_t kMask = kPair ? 0xFCu : Table<B>::addr_mask(); // index bits inside a merged byte
    static constexpr int kLow = (kMask & 1) ? 0 : (kMask & 2) ? 1 : 2;       // lowest of them
    static constexpr bool kPerm = (B <= 7 && B != 4);                        // address by v_perm_b32, else by v_dot4_u32_u8
    static constexpr int kExtra = kPerm ? kLow : 0;                          // extra rotation of the index words
    static constexpr uint32_t kClean = (kMask >> kExtra) * 0x01010101u;      // index bits of the rotated words
    static constexpr int kShift = kPerm ? 8 : 7;                             // entry value -> address
    static constexpr int kTileBytes = kPair4 ? 256 * 128 : (int)((kMask >> kLow) + 1) << (kPerm ? 8 : 7); // 16 rows x 2 copies x 4 bytes per entry (x 2 unused)
    // value in a (rotated) index byte of the entry stored at position p of a row (lut_stored_pos order; pair index for B = 3)
    __device__ static constexpr uint32_t byte_of(uint32_t p)
    {
        return (kPair ? p << 2 : B == 4 ? (((p & 8u) << 3) | ((p & 7u) << 2)) : p << kLow) >> kExtra;
    }
    // LDS address of the entry selected by byte J of the index word w, for a lane with base `rowbase` (< 128)
    template <int J> __device__ static __forceinline__ uint32_t addr(uint32_t w, uint32_t rowbase)
    {
        if constexpr (kPerm) return __builtin_amdgcn_perm(rowbase, w, 0x0c0c0004u | ((uint32_t)J << 8));
        else return __builtin_amdgcn_udot4(w, 128u << (8 * J), rowbase, false);
    }
};

// The waves split a row's pairs of octets evenly: wave w starts at npairs * w / nwaves.  The quotient comes from a product with
// 2^32 / nwaves + 1 (exact: npairs < 2^23, nwaves <= 8); a 64-bit division took 300 scalar instructions, ahead of the first load.
static inline uint32_t wave_reciprocal(int nwaves) { return nwaves > 1 ? 0xffffffffu / (uint32_t)nwaves + 1 : 0; }
__device__ __forceinline__ int first_pair(int npairs, int w, uint32_t reciprocal)
{
    const uint32_t a = (uint32_t)npairs * (uint32_t)w;
    return (int)(reciprocal ? __umulhi(a, reciprocal) : a);
}

constexpr int kExchangeBytes = 1024; // LDS per wave, given at the launch

// `wg` = index of the workgroup within its matrix (R tiles each).  RAG: K is not a multiple of 256 (the last octet holds fewer than 8
// chunks; lanes of chunks that do not exist multiply zeros by zeros).  WIDE: batch 9..16.  SKIP: loads that are dropped ask for no
// memory, REFILL: one set of activation registers (both: launch_tile_r).
template <int B, int R, int MAXT, bool RAG, bool WIDE, bool SKIP, bool REFILL>
__device__ __forceinline__ void gemv_tile_body(const uint8_t *__restrict__ slices, size_t slice_bytes, const uint16_t *__restrict__ lut,
                                               const uint16_t *__restrict__ x, uint16_t *__restrict__ y, int M, int K, int batch,
                                               int wg, uint32_t reciprocal)
{
    using TT = TileTable<B>;
    constexpr int kTileRows = 16, kTileGroups = kTileRows / kRowsPerGroup;
    // the tables during the main loop, then the waves' partial sums [wave][tile][row][batch row]
    constexpr int kTabBytes = R * TT::kTileBytes, kCols = WIDE ? 16 : 8, kRedBytes = (MAXT / 64) * R * kTileRows * kCols * 4;
    __shared__ __attribute__((aligned(16))) uint8_t smem[kTabBytes > kRedBytes ? kTabBytes : kRedBytes];
    uint8_t *tab = smem;
    __shared__ __attribute__((aligned(16))) uint16_t nat[TT::kPair ? R * kTileRows * 10 : TT::kPair4 ? R * kTileRows * 18 : 8]; // the rows as stored (pair paths)
    extern __shared__ __attribute__((aligned(16))) uint32_t bounce_all[]; // kExchangeBytes per wave
    float(*red)[R][kTileRows][kCols] = reinterpret_cast<float(*)[R][kTileRows][kCols]>(smem);

    const int tid = threadIdx.x, nth = blockDim.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nwaves = nth >> 6;
    const int i = lane & 15;  // row of a tile this lane dequantises; output column (batch row, quad) it receives
    const int kg = lane >> 4; // its 8 columns of every instruction; its chunk of every quad of chunks
    const int groups = (M + kRowsPerGroup - 1) / kRowsPerGroup;
    const int g0 = wg * (R * kTileGroups);
    const int row0 = g0 * kRowsPerGroup;
    const int chunks = K / kChunkSlots;
    const int nspans = (chunks + kSpanLanes - 1) / kSpanLanes;

    // ---- per-lane offsets of the slice loads: lane 32 p + 4 c + r loads row r of row group 2 half + p of
    // the tile, chunk c of the octet
    const int lp = lane >> 5, lc = (lane >> 2) & 7, lr = lane & 3;
    const uint32_t group_bytes = (uint32_t)chunks * 16u, lane_part = (uint32_t)lc * 16u + (uint32_t)lr * 4u;
    const uint32_t soff_first = (uint32_t)lp * group_bytes + lane_part, soff_last = (uint32_t)(groups - 1 - g0) * group_bytes + lane_part;
    auto soff_lane = [&](int tile, int half) { // groups past the matrix: the last one again (never stored)
        const uint32_t off = soff_first + (uint32_t)(tile * kTileGroups + 2 * half) * group_bytes;
        return off < soff_last ? off : soff_last;
    };
    // Dword in the wave's exchange memory of the word of row r, row group g, quad h, lane group k: 32 lanes a clock are on 32 banks both
    // when a load is written (one g; all h, k, r) and when a quad is read (one h, two k; all g, r).
    auto place = [](int h, int k, int g, int r) {
        return r | (k & 1) << 2 | ((k >> 1) ^ (g & 1)) << 3 | (h ^ (g >> 1)) << 4 | (k >> 1) << 5 | h << 6;
    };
    uint32_t *bounce = bounce_all + wave * 256;
    int put0 = place(lc >> 2, lc & 3, lp, lr), get0 = place(0, kg, i >> 2, i & 3);
    // activations: lane 16 kg + 2 n + h loads batch row n (WIDE: and n + 8), chunk 4 h + kg of the octet; the descriptor ends with the last
    // batch row, and lanes of rows past the batch carry an offset beyond it (batch * K * 2 < 2^31; valid lanes stay below the end
    // with any scalar offset).
    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(x), 0, (uint32_t)batch * (uint32_t)K * 2u, kBufferRsrcWord3);
    constexpr int kXSets = WIDE ? 2 : 1;
    constexpr int kNoMemory = 0x38f; // of sched_barrier: what may move across, all but loads and stores of memory
    const int xn = i >> 1, xc = 4 * (i & 1) + kg;
    uint32_t xoff_lane[kXSets];
#pragma unroll
    for (int q = 0; q < kXSets; ++q)
        xoff_lane[q] = xn + 8 * q < batch ? (uint32_t)(xn + 8 * q) * (uint32_t)K * 2u + (uint32_t)xc * 16u : 0x80000000u;
    const uint32_t rowbase = ((uint32_t)i << 2) | ((uint32_t)(kg & 1) << 6);

    int lanes = xc | lc << 8; // the chunks that this lane loads, for ragged octets
    // Two ragged tiles at 3 bits keep within 128 registers (4 waves per SIMD) only if what is cheap to compute again is not kept, and if the
    // second tile's exchange does not move up: with 129 registers 25000 x 288 batch 3 takes 8.5 us instead of 6.2, x 12320 52 instead of 42.
    constexpr bool kTight = B == 3 && R == 2 && RAG && !(WIDE && REFILL);
    float4_t acc[R][kXSets][2]; // one accumulator per quad of an octet (and 8 batch rows): independent chains of matrix instructions
#pragma unroll
    for (int tile = 0; tile < R; ++tile)
#pragma unroll
        for (int q = 0; q < kXSets; ++q) acc[tile][q][0] = acc[tile][q][1] = float4_t{0.f, 0.f, 0.f, 0.f};

    // Octet o of a row = chunks 8 o .. 8 o + 7 (span o / 8); the waves split the row's pairs of octets
    // evenly.  The loads of an octet are issued before the arithmetic of the octet before it (two
    // register sets; REFILL: the activations have one, see launch_tile_r).  Every pass of the loop issues the same loads and has no exit in the middle, so the
    // wait before the arithmetic leaves exactly the newer loads in flight: a row with an odd number of
    // octets gets one more (the last one again, activations out of range), and the loads issued in the
    // last pass for the pass after it repeat a valid octet and are dropped.  The products of that padding
    // octet do not count (its centroids are real ones, and infinity x 0 is not 0): masked centroids in the
    // RAG instances, the sums of before it in the others (0 to 1 % of the call; a branch around its
    // arithmetic cost 7 % on rows without such an octet: b = 3, 4 then schedule with 78 registers
    // instead of 107).
    struct XLoads { // the activations of an octet; run t at base + t * step
        uint32_t lane[kXSets], base, step;
    };
    auto load_run = [&](const XLoads &l, int t, u32x4 (&X)[kXSets][4]) {
#pragma unroll
        for (int q = 0; q < kXSets; ++q) X[q][t] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, l.lane[q], l.base + (uint32_t)t * l.step, 0);
    };
    auto issue = [&](int o, bool real, u32x4 (&X)[kXSets][4], uint32_t (&Q)[R][2][B], auto with_x) {
        const int span = o >> 3, oi = o & 7;
        const int rem = chunks - span * kSpanLanes;
        const int nl = rem < kSpanLanes ? rem : kSpanLanes;
        const int left = chunks - o * 8; // chunks of this octet and beyond
        if constexpr (kTight) asm volatile("" : "+v"(lanes));
        XLoads l;
#pragma unroll
        for (int q = 0; q < kXSets; ++q) l.lane[q] = real && (!RAG || (lanes & 7) < left) ? xoff_lane[q] : 0x80000000u;
        l.base = (uint32_t)span * (kSpanCols * 2u) + (uint32_t)oi * 128u;
        l.step = (uint32_t)(16 * nl);
        if constexpr (decltype(with_x)::value) {
#pragma unroll
            for (int t = 0; t < 4; ++t) load_run(l, t, X);
        }
        // no records, no memory access (the addresses are valid all the same)
        const uint32_t records = SKIP ? (uint32_t)__builtin_amdgcn_readfirstlane(real ? -1 : 0) : 0xffffffffu;
        const __amdgpu_buffer_rsrc_t srsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint8_t *>(slices + (size_t)g0 * chunks * 16), 0, records, kBufferRsrcWord3);
        const uint32_t soct = (uint32_t)o * 128u;
        const int clane = RAG ? lanes >> 8 : 0;
        const uint32_t back = RAG && clane >= left ? (uint32_t)(clane - (left - 1)) * 16u : 0u; // chunks that do not exist: the last one again
#pragma unroll
        for (int tile = 0; tile < R; ++tile)
#pragma unroll
            for (int s = 0; s < B; ++s)
#pragma unroll
                for (int half = 0; half < 2; ++half)
                    Q[tile][half][s] = __builtin_amdgcn_raw_buffer_load_b32(srsrc, soff_lane(tile, half) - back,
                                                                            soct + (uint32_t)s * (uint32_t)slice_bytes, kBufferNonTemporal);
        return l;
    };
    // `used(t)`: after the last tile has used the activations of run t
    auto compute = [&](const u32x4 (&X)[kXSets][4], const uint32_t (&Q)[R][2][B], int o, auto &&used) {
        if constexpr (kTight) asm volatile("" : "+v"(put0), "+v"(get0));
        const int put[2] = {put0, put0 ^ 16}, get[2] = {get0, (get0 ^ 16) + 64}; // [half of the row groups], [quad]
        const uint32_t keep[2] = {kg < chunks - o * 8 ? 0xffffffffu : 0u, kg + 4 < chunks - o * 8 ? 0xffffffffu : 0u}; // RAG
#pragma unroll
        for (int tile = 0; tile < R; ++tile) {
            const uint8_t *tt = tab + tile * TT::kTileBytes;
            if constexpr (kTight) __builtin_amdgcn_sched_barrier(0);
            uint32_t W[2][8]; // [quad of the octet]
            {
                uint32_t q[2][B];
#pragma unroll
                for (int s0 = 0; s0 < B; s0 += 2) {
#pragma unroll
                    for (int s = s0; s < B && s < s0 + 2; ++s)
#pragma unroll
                        for (int half = 0; half < 2; ++half) bounce[(s - s0) * 128 + put[half]] = Q[tile][half][s];
                    wave_lds_fence();
#pragma unroll
                    for (int s = s0; s < B && s < s0 + 2; ++s)
#pragma unroll
                        for (int h = 0; h < 2; ++h) q[h][s] = bounce[(s - s0) * 128 + get[h]];
                    wave_lds_fence();
                }
                if constexpr (TT::kPair4) {
                    merge_words_pair4(q[0], W[0]);
                    merge_words_pair4(q[1], W[1]);
                } else {
                    merge_words<B, TT::kExtra>(q[0], W[0]);
                    merge_words<B, TT::kExtra>(q[1], W[1]);
                }
                if constexpr (TT::kPerm) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int u = 0; u < 8; u += TT::kPair ? 2 : 1) W[h][u] &= TT::kClean;
                }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                uint32_t P[2][4]; // packed centroid pairs: P[h][j] = columns 2j, 2j + 1 of run t, quad h
                if constexpr (TT::kPair || TT::kPair4) {
                    uint32_t ad[2][4];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t v = W[h][2 * t];
                        ad[h][0] = TT::template addr<0>(v, rowbase);
                        ad[h][1] = TT::template addr<1>(v, rowbase);
                        ad[h][2] = TT::template addr<2>(v, rowbase);
                        ad[h][3] = TT::template addr<3>(v, rowbase);
                    }
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int j = 0; j < 4; ++j) P[h][j] = *reinterpret_cast<const uint32_t *>(tt + ad[h][j]);
                } else {
                    uint32_t ae[2][4], ao[2][4];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t ve = W[h][2 * t], vo = W[h][2 * t + 1];
                        ae[h][0] = TT::template addr<0>(ve, rowbase);
                        ae[h][1] = TT::template addr<1>(ve, rowbase);
                        ae[h][2] = TT::template addr<2>(ve, rowbase);
                        ae[h][3] = TT::template addr<3>(ve, rowbase);
                        ao[h][0] = TT::template addr<0>(vo, rowbase);
                        ao[h][1] = TT::template addr<1>(vo, rowbase);
                        ao[h][2] = TT::template addr<2>(vo, rowbase);
                        ao[h][3] = TT::template addr<3>(vo, rowbase);
                    }
                    uint32_t we[2][4], wo[2][4];
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            we[h][j] = *reinterpret_cast<const uint16_t *>(tt + ae[h][j]);
                            wo[h][j] = *reinterpret_cast<const uint16_t *>(tt + ao[h][j]);
                        }
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int j = 0; j < 4; ++j) P[h][j] = we[h][j] | (wo[h][j] << 16);
                }
                if constexpr (RAG) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int j = 0; j < 4; ++j) P[h][j] &= keep[h];
                }
                // both quads against the same B: the even columns of the first product and the odd ones of the second count
                const u32x4 a0 = {P[0][0], P[0][1], P[0][2], P[0][3]}, a1 = {P[1][0], P[1][1], P[1][2], P[1][3]};
#pragma unroll
                for (int q = 0; q < kXSets; ++q) {
                    acc[tile][q][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a0), __builtin_bit_cast(half8_t, X[q][t]),
                                                                             acc[tile][q][0], 0, 0, 0);
                    acc[tile][q][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a1), __builtin_bit_cast(half8_t, X[q][t]),
                                                                             acc[tile][q][1], 0, 0, 0);
                }
                if (tile == R - 1) used(t);
            }
        }
    };

    const int nocts = (chunks + 7) >> 3;
    const int npairs = (nocts + 1) >> 1;
    const int p1 = first_pair(npairs, wave + 1, reciprocal);
    u32x4 XA[kXSets][4], XB[kXSets][4];
    uint32_t QA[R][2][B], QB[R][2][B];
    int p = first_pair(npairs, wave, reciprocal); // < npairs, also for a wave without pairs
    // The wave's first octet.  Waves without pairs (short rows at b = 3, 4, 8: they help to build the tables) would load and drop one, in the way
    // of the others at the vector L1: at b = 3, 4 they leave it out, at b = 8, where a branch costs the longer rows 1 %, their activations
    // ask for no memory.  Loaded / left out, us: 18532 x 512 batch 14 b = 3 7.1 / 6.1, 8592 x 480 batch 16 b = 4 6.1 / 5.3.  Not where
    // several workgroups share a CU and rows are long (SKIP): no such waves in single calls, and list and fused launches, which have them, load.
    auto load_first = [&]() {
        constexpr bool kBranch = !SKIP && (B == 3 || B == 4);
        if (!kBranch || p < p1) issue(2 * p, SKIP || B != 8 || p < p1, XA, QA, std::true_type());
    };
    // ---- tables of the R tiles into LDS (rows past the matrix repeat the last row; never stored).
    // Thread (row = tid % 16, copy = (tid / 16) % 2, part = tid / 32) writes the entries of the pieces
    // part, part + nparts, ... of its row and copy: the 32 lanes of an LDS clock hit 32 different banks
    // (with one row per wave every lane of a store would land in the same bank).  A thread loads 16
    // bytes at a time and issues its loads before the first store that depends on them (one dword load
    // per loop pass cost a memory round trip per pass and one cache access per lane: 4 to 7 us per
    // workgroup).  The loads of the wave's first octet go out between the table loads and the table
    // stores, so that they are in flight during the stores and do not delay the tables (loads return in
    // order).
    {
        const int srow = tid & 15, scopy = (tid >> 4) & 1, part = tid >> 5, nparts = nth >> 5;
        if constexpr (TT::kPair4) {
            // the rows as stored (16 entries = 32 bytes each; 36 bytes apart in LDS, so that the rows fall on
            // different banks) first, then the 256 pair entries of every row and copy: thread (row, copy, part) writes
            // entries part + k * parts, 16 rows x 2 copies = 32 banks a clock.  With 256 or 512 threads the loop over k
            // is unrolled: the even and odd table positions are then the thread's own (from `part`) plus a
            // constant, i.e. an immediate offset of the LDS read, and an entry costs two reads, one pack and one
            // write.
            constexpr int kNatDwords = 9;
            for (int e = tid; e < R * kTileRows * 8; e += nth) {
                const int r = e >> 3;
                const int row = row0 + r < M ? row0 + r : M - 1;
                reinterpret_cast<uint32_t *>(nat)[r * kNatDwords + (e & 7)] = reinterpret_cast<const uint32_t *>(lut + (size_t)row * 16)[e & 7];
            }
            load_first();
            __syncthreads();
            auto build = [&](auto log2_parts) {
                constexpr int L = decltype(log2_parts)::value;
                const uint16_t *even = nat + srow * (2 * kNatDwords) + pair4_even(part);
                const uint16_t *odd = nat + srow * (2 * kNatDwords) + pair4_odd(part);
                uint8_t *base = tab + ((srow << 2) | (scopy << 6)) + (part << 7);
#pragma unroll
                for (int tile = 0; tile < R; ++tile)
#pragma unroll
                    for (int k = 0; k < (256 >> L); ++k)
                        *reinterpret_cast<uint32_t *>(base + tile * TT::kTileBytes + (k << (L + 7))) =
                            (uint32_t)even[tile * kTileRows * 2 * kNatDwords + pair4_even(k << L)] |
                            ((uint32_t)odd[tile * kTileRows * 2 * kNatDwords + pair4_odd(k << L)] << 16);
            };
            if (nth == 256) build(std::integral_constant<int, 3>{});
            else if (nth == 512) build(std::integral_constant<int, 4>{});
            else {
#pragma unroll
                for (int tile = 0; tile < R; ++tile) {
                    const uint16_t *src = nat + (tile * kTileRows + srow) * (2 * kNatDwords);
                    uint8_t *base = tab + tile * TT::kTileBytes + ((srow << 2) | (scopy << 6));
                    for (int d = part; d < 256; d += nparts)
                        *reinterpret_cast<uint32_t *>(base + (d << 7)) = (uint32_t)src[pair4_even(d)] | ((uint32_t)src[pair4_odd(d)] << 16);
                }
            }
        } else if constexpr (TT::kPair) {
            // natural rows (8 entries = 16 bytes each, 20 bytes apart in LDS: 16 rows on 16 banks) first, then the
            // pair entries from LDS; unrolled like the 4-bit build above (entries part + k * parts of a thread's
            // row and copy: the even and odd centroid of an entry sit at the thread's own offset + a constant)
            constexpr int kNatDwords = 5;
            for (int e = tid; e < R * kTileRows * 4; e += nth) {
                const int r = e >> 2;
                const int row = row0 + r < M ? row0 + r : M - 1;
                reinterpret_cast<uint32_t *>(nat)[r * kNatDwords + (e & 3)] = reinterpret_cast<const uint32_t *>(lut + (size_t)row * 8)[e & 3];
            }
            load_first();
            __syncthreads();
            auto build = [&](auto log2_parts) {
                constexpr int L = decltype(log2_parts)::value;
                const uint16_t *even = nat + srow * (2 * kNatDwords) + pair3_even(part);
                const uint16_t *odd = nat + srow * (2 * kNatDwords) + pair3_odd(part);
                uint8_t *base = tab + ((srow << 2) | (scopy << 6)) + (TT::byte_of(part) << TT::kShift);
#pragma unroll
                for (int tile = 0; tile < R; ++tile)
#pragma unroll
                    for (int k = 0; k < (64 >> L); ++k)
                        *reinterpret_cast<uint32_t *>(base + tile * TT::kTileBytes + (TT::byte_of(k << L) << TT::kShift)) =
                            (uint32_t)even[tile * kTileRows * 2 * kNatDwords + pair3_even(k << L)] |
                            ((uint32_t)odd[tile * kTileRows * 2 * kNatDwords + pair3_odd(k << L)] << 16);
            };
            if (nth == 256) build(std::integral_constant<int, 3>{});
            else if (nth == 512) build(std::integral_constant<int, 4>{});
            else {
#pragma unroll
                for (int tile = 0; tile < R; ++tile) {
                    uint8_t *base = tab + tile * TT::kTileBytes + ((srow << 2) | (scopy << 6));
                    for (int d = part; d < 64; d += nparts)
                        *reinterpret_cast<uint32_t *>(base + (TT::byte_of(d) << TT::kShift)) =
                            pair_entry(nat + (tile * kTileRows + srow) * (2 * kNatDwords), d);
                }
            }
        } else {
            constexpr int kPieces = (2 << B) / 16; // 16-byte pieces (8 entries) of a row's table
            // b >= 7: a thread loads a piece once and writes it to both copies, two neighbours reading 32 contiguous bytes of a row and
            // starting with different copies (32 lanes on 32 banks); the smaller tables give every copy threads of its own.
            // 4096 x 4096 batch 8 b = 7/8 7.4/8.05 -> 7.0/7.6 us, 28672 x 8192 48.3/54.6 -> 47.3/53.5, 4096 x 1024 batch 6 4.55/5.3 ->
            // 4.35/5.15.
            constexpr bool kBoth = B >= 7;
            constexpr int kBurst = kBoth ? 2 : 4; // pieces per thread in the first pass: all of them from 4 waves on
            const int prow = kBoth ? (tid >> 1) & 15 : srow, pcopy = kBoth ? tid & 1 : scopy;
            auto piece = [&](int j) { return kBoth ? 2 * (part + j * nparts) + (tid & 1) : part + j * nparts; };
            auto store_piece = [&](uint8_t *base, int pc, const u32x4 &v) {
#pragma unroll
                for (int c = 0; c < (kBoth ? 2 : 1); ++c)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        uint8_t *dst = base + ((pcopy ^ c) << 6);
                        *reinterpret_cast<uint16_t *>(dst + (TT::byte_of(8 * pc + 2 * e) << TT::kShift)) = (uint16_t)v[e];
                        *reinterpret_cast<uint16_t *>(dst + (TT::byte_of(8 * pc + 2 * e + 1) << TT::kShift)) = (uint16_t)(v[e] >> 16);
                    }
            };
            const u32x4 *src[R];
            uint8_t *base[R];
            u32x4 v[R][kBurst];
#pragma unroll
            for (int tile = 0; tile < R; ++tile) {
                const int row = row0 + tile * kTileRows + prow < M ? row0 + tile * kTileRows + prow : M - 1;
                src[tile] = reinterpret_cast<const u32x4 *>(lut + ((size_t)row << B));
                base[tile] = tab + tile * TT::kTileBytes + (prow << 2);
#pragma unroll
                for (int j = 0; j < kBurst; ++j) {
                    const int pc = piece(j);
                    v[tile][j] = src[tile][pc < kPieces ? pc : kPieces - 1];
                }
            }
            // The octet's loads wait for the tables (the statements use their registers): every CU's tables then arrive ahead of
            // every slice instead of between them, and the stores below run while the slices are on their way.  4096 x 4096 batch 8
            // b = 5/6/7 6.4/6.8/7.8 -> 6.2/6.6/7.35 us, 4099 x 2208 b = 7 batch 5 8.2 -> 7.7, 28672 x 8192 0.97 to 1.01.
#pragma unroll
            for (int tile = 0; tile < R; ++tile)
#pragma unroll
                for (int j = 0; j < kBurst; ++j) asm volatile("" : "+v"(v[tile][j]));
            load_first();
#pragma unroll
            for (int tile = 0; tile < R; ++tile) {
#pragma unroll
                for (int j = 0; j < kBurst; ++j) {
                    const int pc = piece(j);
                    if (pc < kPieces) store_piece(base[tile], pc, v[tile][j]);
                }
                // workgroups of fewer than 4 waves (rows of less than 2048 columns) at b >= 7: the rest
                for (int j = kBurst; piece(j) < kPieces; ++j) store_piece(base[tile], piece(j), src[tile][piece(j)]);
            }
        }
    }
    __syncthreads();

    float4_t before[R][kXSets][2]; // the sums ahead of the wave's last octet
#pragma unroll
    for (int tile = 0; tile < R; ++tile)
#pragma unroll
        for (int q = 0; q < kXSets; ++q) before[tile][q][0] = before[tile][q][1] = float4_t{0.f, 0.f, 0.f, 0.f};
    for (; p < p1; ++p) {
        const bool second = 2 * p + 1 < nocts;
        const int o1 = second ? 2 * p + 1 : 2 * p;
        // the loads of octet o: its activations into the other set ahead of the arithmetic, or (WIDE) run by run into the one that is in use
        auto ahead = [&](int o, bool real, u32x4 (&X)[kXSets][4], uint32_t (&Q)[R][2][B]) {
            const XLoads l = issue(o, real, X, Q, std::bool_constant<!REFILL>());
            __builtin_amdgcn_sched_barrier(0); // keep the loads ahead of the arithmetic they overlap with
            return [&XA, &load_run, l](int t) {
                if constexpr (REFILL) {
                    __builtin_amdgcn_sched_barrier(kNoMemory);
                    load_run(l, t, XA);
                    __builtin_amdgcn_sched_barrier(kNoMemory);
                }
            };
        };
        u32x4 (&X1)[kXSets][4] = REFILL ? XA : XB;
        compute(XA, QA, 2 * p, ahead(o1, second, XB, QB));
        auto next = ahead(p + 1 < p1 ? 2 * p + 2 : 2 * p, !SKIP || p + 1 < p1, XA, QA);
        if constexpr (RAG) {
            compute(X1, QB, 2 * p + 1, next); // the padding octet has no chunks: all centroids masked
        } else {
#pragma unroll
            for (int tile = 0; tile < R; ++tile)
#pragma unroll
                for (int q = 0; q < kXSets; ++q) { before[tile][q][0] = acc[tile][q][0]; before[tile][q][1] = acc[tile][q][1]; }
            compute(X1, QB, o1, next);
        }
    }
    if (!RAG && (nocts & 1) && p1 == npairs) { // the padding octet does not count
#pragma unroll
        for (int tile = 0; tile < R; ++tile)
#pragma unroll
            for (int q = 0; q < kXSets; ++q) { acc[tile][q][0] = before[tile][q][0]; acc[tile][q][1] = before[tile][q][1]; }
    }

    // ---- acc[tile][q][h][r] of lane (i, kg): output row 4 kg + r of the tile over the wave's columns of quad h; column i is batch row
    //      i / 2 (+ 8 q) where i % 2 == h.  The two halves of a batch row are neighbouring lanes; waves are added in fixed order
    //      (lane and thread number again from the hardware: kept through the loop they cost registers)
    const int olane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), oi = olane & 15, okg = olane >> 4;
    __syncthreads(); // every wave is done with the tables, whose memory now takes the partial sums
#pragma unroll
    for (int tile = 0; tile < R; ++tile)
#pragma unroll
        for (int q = 0; q < kXSets; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float half = (oi & 1) ? acc[tile][q][1][r] : acc[tile][q][0][r];
                const float sum = half + dpp_get<0xB1>(half); // quad_perm [1,0,3,2]
                if (!(oi & 1)) red[wave][tile][4 * okg + r][(oi >> 1) + 8 * q] = sum;
            }
    __syncthreads();
    for (int o = wave * 64 + olane; o < R * kTileRows * kCols; o += nth) {
        const int n = o % kCols, r = o / kCols; // r = row inside the workgroup's R tiles
        float s = 0.f;
        for (int w = 0; w < nwaves; ++w) s += red[w][r >> 4][r & 15][n];
        const int row = row0 + r;
        if (row < M && n < batch) {
            const __half hv = __float2half_rn(s);
            y[(size_t)n * M + row] = __builtin_bit_cast(uint16_t, hv);
        }
    }
}

// No bound on the waves per SIMD here and in the multi kernel: with at most 4 the b = 3, 4 instances of one tile take 107 registers
// instead of 74..80 and workgroups of 8 waves then lose residency, b = 5, 6 go from 5 waves to 4 for nothing.  Bounded / unbounded, us: 16384 x 12288
// b = 4 batch 3 28.4 / 25.9, 5120 x 2208 b = 4 batch 5 11.6 / 8.9.  Asked for the waves that they have anyway (as the list kernel is), they
// schedule worse: 4099 x 2208 b = 7 batch 5 7.0 -> 7.2, 9000 x 3104 b = 5 batch 6 11.5 -> 12.1.
template <int B, int R, int MAXT, bool RAG, bool WIDE, bool SKIP, bool REFILL>
__global__ __launch_bounds__(MAXT) __attribute__((amdgpu_waves_per_eu(B == 3 && R == 2 && RAG && !WIDE ? 4 : 1))) void gemv_tile_kernel(
    const uint8_t *__restrict__ slices, size_t slice_bytes, const uint16_t *__restrict__ lut, const uint16_t *__restrict__ x,
    uint16_t *__restrict__ y, int M, int K, int batch, uint32_t reciprocal)
{
    gemv_tile_body<B, R, MAXT, RAG, WIDE, SKIP, REFILL>(slices, slice_bytes, lut, x, y, M, K, batch, (int)blockIdx.x, reciprocal);
}

// Several matrices of equal row length at one bit-width and batch in one launch (the projections of a
// decoder layer that share their input): workgroup -> (matrix, tile) through the prefix sums of the
// tile counts, which the launcher puts into group_begin.
template <int B, int MAXT>
__global__ __launch_bounds__(MAXT) void gemv_tile_multi_kernel(MultiArgs a, uint32_t reciprocal)
{
    int m = 0;
#pragma unroll
    for (int i = 1; i < kMaxMulti; ++i)
        if (i < a.count && (int)blockIdx.x >= a.group_begin[i]) m = i;
    gemv_tile_body<B, 1, MAXT, false, false, true, false>(a.slices[m], a.slice_bytes[m], a.lut[m], a.x[m], a.y[m], a.M[m], a.K, a.batch,
                               (int)blockIdx.x - a.group_begin[m], reciprocal);
}

// List and fused launches leave the octet that a wave's last pass drops unrequested (SKIP; single calls: launch_tile_r), us with it / without:
// 7B decoder layer b = 3/5/8 batch 4 25.9/39.3/53.1 -> 24.9/38.2/49.0, batch 8 31.6/43.7/58.3 -> 29.3/41.0/53.6, 6 of 8192 x 2816 b = 8 batch 8
// 43.5 -> 37.4, 2 of 11008 x 4096 b = 4 batch 8 15.6 -> 14.9, 8 of 2048 x 2048 b = 3 batch 4 7.4 -> 7.5 (a few scalar instructions ahead of
// the loads).

// A work list of matrices of any shapes (rows of one class of length) at one bit-width and batch.  The bound asks for the registers
// that the single instances take by themselves: without it these settle at 107 / 108 / 130 at b = 3 / 4 / 5 (4 / 4 / 3 waves per SIMD
// instead of 6 / 6 / 5).  Without / with, us: b = 5 decoder layer batch 8 50.1 / 44.7, 3 of 8192 x 12288 batch 4 66.8 / 53.3.
template <int B, int MAXT>
__global__ __launch_bounds__(MAXT) __attribute__((amdgpu_waves_per_eu(B <= 4 ? 6 : B <= 6 ? 5 : 4))) void gemv_tile_list_kernel(ListArgs a, int batch, uint32_t reciprocal)
{
    int it = 0;
#pragma unroll
    for (int i = 1; i < kMaxListItems; ++i)
        if (i < a.count && (int)blockIdx.x >= a.group_begin[i]) it = i;
    const ListItem &I = a.item[it];
    gemv_tile_body<B, 1, MAXT, false, false, true, false>(I.slices, I.slice_bytes, I.lut, I.x, I.y, I.M, I.K, batch, (int)blockIdx.x - a.group_begin[it],
                                             reciprocal);
}

// Waves per workgroup of a single call that no option decides.  From 9270 calls (14 heights, 23 row lengths, every b, batch 3..8);
// time with 4 waves over the time with the number chosen, or the other way round where the rule says 4:
//   8 (a wave per pair of octets on shorter rows) on rows of 12288 columns or more, so that a wave still runs several passes, and where
//   every tile has a CU of its own: 4096x11008 b = 4 batch 4 1.21, 4096x8192 b = 8 1.09, 4096x2208 b = 5 batch 8 1.14.  From the 257th
//   tile on a CU gets two tiles while others idle, and 4 are ahead: 4112x5120 b = 8 batch 8 1.14, b = 3 1.10; except for rows of
//   5 pairs, which 4 waves take in two rounds (4112x2208 b = 7 1.07), and b = 5 on long rows (5120x8192 1.04).
//   With 5 to 7 waves the 4-bit pair tables are built by the general loop: 4096x3072 1.18 with 4.  10 to 12 pairs are two rounds of 8
//   waves or three of 4: 4096x6144 b = 8 1.07 with 4, at b = 3, 4 0.97.  Nine batch rows and more: 4 (4096x4096 7.3 against 7.9 us).
//   Rows of fewer than 4 pairs: waves without columns help to build the large tables (b = 3, 4, 8; 8192x512 b = 4 3.05, b = 3 1.42, b = 8
//   1.08, 20480x512 b = 8 1.30, but 16384x512 b = 8, four tiles per CU, 0.92; at batch 9 to 16
//   1.10 there), the others lose by them (28672x512 b = 6 1.65, 4096x1024 b = 5 1.08 without).
static int tile_waves(const GemvArgs &a, int tiles, int npairs, bool wide)
{
    const bool eight = a.K >= 12288 || (tiles <= 256 && !(a.b >= 5 && npairs >= 10 && npairs <= 12)) ||
                       (tiles <= 320 && (npairs == 5 || (a.b == 5 && a.K >= 8192)));
    int nw = !wide && eight ? 8 : 4;
    if (nw > npairs) nw = npairs;
    if (a.b == 4 && nw < 8) nw = 4;
    const bool helpers = a.b <= 4 || (a.b == 8 && (wide || tiles < 768 || tiles > 1024)) || (a.b == 7 && npairs == 1 && tiles <= 256);
    return nw < 4 && helpers ? 4 : nw;
}

template <int B, int R, bool WIDE> static hipError_t launch_tile_r(const GemvArgs &a, hipStream_t stream)
{
    constexpr int kMaxWaves = 8;
    const int npairs = ((a.K + 255) / 256 + 1) / 2;
    const int tiles = (a.M + 15) / 16;
    int nw;
    if (a.waves_per_group > 0) nw = a.waves_per_group < npairs ? a.waves_per_group : npairs;
    else if (a.variant == 0) nw = tile_waves(a, tiles, npairs, WIDE);
    else { // a handle that asks for this kernel: the rule of the fused launches, with which it promises equal bits
        nw = a.K >= 12288 ? kMaxWaves : 4; // (waves beyond the row's pairs add nothing to the sums)
    }
    const dim3 grid((tiles + R - 1) / R), block(64 * nw);
    auto launch = [&](auto ragged, auto skip, auto refill) {
        hipLaunchKernelGGL((gemv_tile_kernel<B, R, 64 * kMaxWaves, decltype(ragged)::value, WIDE, decltype(skip)::value, decltype(refill)::value>), grid, block,
                           nw * kExchangeBytes, stream, a.slices, a.slice_bytes, a.lut, a.x, a.y, a.M, a.K, a.batch, wave_reciprocal(nw));
    };
    // The octet that the last pass of a wave requests and drops (with 4096 columns on 4 waves one of five) is left out where several
    // workgroups share a CU, which then want the bandwidth; elsewhere the few scalar instructions ahead of the loads cost 0.05 us.
    // With it / without, us: 11008x4096 b = 4 batch 16 15.3 / 14.8, b = 8 batch 16 22.0 / 21.1, b = 3 batch 8 9.0 / 8.8, 28672x8192 b = 5
    // batch 16 56.9 / 55.1, b = 4 batch 8 40.6 / 40.1, 6144x4128 b = 5 batch 8 12.4 / 12.25; 4096x4096 b = 4 batch 8 5.53 / 5.63, 8192x512
    // 4.57 / 4.63, 8192x1024 b = 3 batch 6 4.21 / 4.27.
    const bool skip = grid.x > 256 && a.K > 2048;
    const std::true_type yes;
    const std::false_type no;
    if constexpr (!WIDE) {
        if (a.K % 256) skip ? launch(yes, yes, no) : launch(yes, no, no);
        else skip ? launch(no, yes, no) : launch(no, no, no);
    } else {
        // Batch 9 to 16: one set of activation registers, a run's loaded again, for the octet after, once its last tile has used them.  With
        // two sets as at batch 3 to 8 the registers of one tile cost a wave per SIMD at b = 5 to 8 (134 to 170 instead of 103 to 122),
        // of two tiles at b = 4 to 7 (172 to 255 instead of 130 to 166).  Two sets / one, us: 22589 x 2560 b = 5 batch 10 19.9 / 15.6,
        // 24352 x 1920 b = 6 batch 9 19.3 / 16.9, 10816 x 2240 b = 5 batch 13 12.8 / 10.0, 11008 x 4096 b = 4 batch 16 10.6 / 10.1, 28672 x
        // 8192 b = 5 47.8 / 44.6.  Where every workgroup has a CU to itself or rows are short, b = 3, 4 have as many waves as they need
        // either way and the loads of two sets are further ahead (two sets over one: up to 4096 rows 0.98, 2101 x 26624 0.83); on long
        // whole rows that outweighs the wave at b = 5 to 8 as well (16k columns and more 0.96 to 0.99, 2870 x 27648 b = 5 0.93).
        const std::bool_constant<(B >= 5)> many;
        if (skip) a.K % 256 ? launch(yes, yes, yes) : launch(no, yes, yes);
        else if (a.K % 256) launch(yes, no, many);
        else a.K < 12288 ? launch(no, no, many) : launch(no, no, no);
    }
    return hipGetLastError();
}

template <int B> static hipError_t launch_tile_b(const GemvArgs &a, hipStream_t stream)
{
    // two tiles per workgroup re-read and re-arrange the activations half as often, at more registers:
    // measured faster on rows of 16384 columns or more, and at 3 bits (where the loads outweigh the
    // arithmetic) on matrices tall enough to fill the device with half as many workgroups (28672 x 8192 at
    // batch 4 and 8: 29-34 -> 28 us; 8192 x 8192: 11.8 -> 12.5, so not there).  On long rows, one tile over two tiles: from
    // 512 tiles on 8192x20480 b = 3 batch 8 1.24, b = 5 1.05; with 257 to 511, where half as many workgroups leave CUs idle, 6144x20480
    // b = 3 1.14 to 1.23, b = 4 1.05 to 1.16, b = 5 to 8 0.94 at batch 3 and 1.01 to 1.04 at 8; up to 256 4096x28672 0.6.  Rows that are not
    // whole octets mask their centroids: 8192x16512 b = 5 0.82 to 0.90, b = 8 0.80 (ALU kernel over two tiles 0.90), 13824x16512
    // b = 5 0.94 to 1.02, b = 3 1.26.
    const int tiles = (a.M + 15) / 16;
    const bool long_rows = a.K >= 16384 && (a.K % 256 == 0 ? tiles >= 512 || (tiles > 256 && (B <= 4 || a.batch >= 7)) : tiles >= 512 && B <= 4);
    const bool two = a.variant == 10 || (a.variant != 9 && (long_rows || (B == 3 && tiles >= 1536)));
    if (a.batch <= 8) return two ? launch_tile_r<B, 2, false>(a, stream) : launch_tile_r<B, 1, false>(a, stream);
    // Batch 9 to 16.  Two tiles load the activations half as often, which pays where these weigh most (long rows, many batch rows, few bits;
    // by half more where rows begin inside a 128-byte line) and where as many tiles fall to the busiest CU either way (769 to 1024 and
    // 1281 to 1536 tiles); on short rows the CU wants more workgroups.  From 27 000 calls on either form (4112 to 28672 rows, all b, batch
    // 9, 12, 14, 16); time with two tiles over time with one at batch 9 / 16, whole rows:
    //                       b = 3                   b = 4                   b = 5, 6                b = 7, 8
    //   columns             2-4k 4-6k      8-12k    2-4k 4-6k      8-12k    2-4k 4-6k      8-12k    2-4k 4-6k      8-12k
    //   448..512 tiles      1.18 1.18/1.06 /0.94    1.21 1.22/1.09 /0.95    1.23 1.22/1.15 /1.05    1.24 1.21/1.12 /1.03
    //   769..1024           0.97 0.90/0.79 /0.73    1.02 0.93/0.84 /0.77    1.08 1.04/0.93 /0.84    1.07 1.01/0.91 /0.85
    //   1025..1280          1.01 0.94/0.85 /0.82    1.22 1.16/1.04 /0.92    1.12 1.09/1.00 /0.94    1.31 1.23/1.10 /1.01
    //   1281..1536          0.86 0.82/0.75 /0.71    1.14 1.05/0.92 /0.82    1.00 0.98/0.89 /0.82    1.20 1.09/0.96 /0.88
    //   1537..1792          1.04 0.99/0.85 /0.80    1.11 1.03/0.92 /0.86    1.12 1.09/0.97 /0.93    1.19 1.14/1.00 /0.94
    // (rows of 1537 to 2048 columns, one pair of octets for every wave, 0.80 to 1.01 at batch 16 and 1281 to 1536 tiles; the lines between
    // the classes come from single calls: 24895 x 1696 b = 8 batch 16 30.8 / 28.0 us, 12300 x 1024 b = 3 batch 16 6.3 / 5.6, 8000 x 9344 b = 4
    // batch 11 18.4 / 19.5.)  Over another 3780 calls the rule is 0.3 to 1.0 % behind the better form of each, by b, at worst 1.28 where it
    // keeps one tile on fewer than 448 (5261 x 24576 b = 3 batch 15).
    const bool many = a.batch >= 11;
    const int k = a.K % 64 ? a.K + a.K / 2 : a.K, never = 1 << 30;
    int from; // columns from which two tiles are ahead
    if (tiles < 448) from = never;
    else if (tiles <= 512) from = many ? (B == 3 ? 6144 : B == 4 || a.K % 256 ? 8192 : never) : a.K % 64 ? 24576 : never;
    else if (tiles <= 768) from = a.batch >= 13 && B <= 4 ? (B == 3 ? 6144 : 8192) : never;
    else if (tiles <= 1024) from = many && B == 3 ? 1025 : many || B <= 4 ? 1537 : 6144;
    else if (tiles <= 1280) from = B == 3 ? (many ? 1537 : 4096) : many && B <= 6 ? (B == 4 ? 6144 : 8192) : never;
    else if (tiles <= 1536) from = B == 3 ? 0 : B == 5 || B == 6 || (many && a.K <= 2048) ? 1537 : many ? 3584 : 8192;
    else if (B == 3) from = a.K % 256 ? 0 : 1537;
    else from = many ? (a.K <= 2048 && a.K % 256 ? 1537 : B <= 6 ? 4096 : 6144) : B == 4 ? 8192 : never;
    const bool wide_two = k >= from;
    return wide_two ? launch_tile_r<B, 2, true>(a, stream) : launch_tile_r<B, 1, true>(a, stream);
}

// Waves per workgroup of a list or fused launch whose shortest row has min_pairs pairs of octets: as single calls on this kernel by option, but
// at b = 5, 6, 7, where waves without columns were slower in single calls (tile_waves), no more than that row has pairs: one short row
// then leaves the longer ones of the launch with few waves.  At b = 3, 4, 8 waves without columns help to build the tables
// (a sum of zero waves more: the bits are the same).  One wave per pair / with helpers, us: 8 of
// 8192 x 512 batch 4 b = 3 14.7 / 12.1, b = 4 56.3 / 16.7, b = 8 28.4 / 22.4, 8 of 8192 x 1024 b = 4 41.6 / 18.4, 6 of 4096 x 1536 16.8 / 10.3, 4 of
// 2048 x 512 15.0 / 6.2; b = 8 with four tiles per CU, 8 of 2048 x 1024 7.4 / 8.2: not there, as in single calls (tile_waves).
static int launch_waves(int b, bool long_rows, int min_pairs, int tiles)
{
    const int nw = long_rows ? 8 : 4;
    const bool helpers = b <= 4 || (b == 8 && (tiles < 768 || tiles > 1024));
    return nw > min_pairs && !helpers ? min_pairs : nw;
}

template <int B> static hipError_t launch_tile_multi_b(MultiArgs &m, int total_tiles, hipStream_t stream)
{
    constexpr int kMaxWaves = 8;
    const int npairs = (m.K / (8 * kChunkSlots) + 1) / 2;
    const int nw = launch_waves(B, m.K >= 12288, npairs, total_tiles);
    hipLaunchKernelGGL((gemv_tile_multi_kernel<B, 64 * kMaxWaves>), dim3(total_tiles), dim3(64 * nw), nw * kExchangeBytes, stream, m, wave_reciprocal(nw));
    return hipGetLastError();
}

// batch 2..8, K % 256 == 0 (the caller checks); one tile per workgroup
hipError_t launch_matrix_tile_multi(const MultiArgs &a, int b, hipStream_t stream)
{
    MultiArgs m = a;
    int total = 0;
    for (int i = 0; i < m.count; ++i) {
        m.group_begin[i] = total;
        total += (m.M[i] + 15) / 16;
    }
    switch (b) {
    case 3: return launch_tile_multi_b<3>(m, total, stream);
    case 4: return launch_tile_multi_b<4>(m, total, stream);
    case 5: return launch_tile_multi_b<5>(m, total, stream);
    case 6: return launch_tile_multi_b<6>(m, total, stream);
    case 7: return launch_tile_multi_b<7>(m, total, stream);
    case 8: return launch_tile_multi_b<8>(m, total, stream);
    }
    return hipErrorInvalidValue;
}

template <int B> static hipError_t launch_tile_list_b(const ListArgs &a, int total_tiles, int nw, int batch, hipStream_t stream)
{
    hipLaunchKernelGGL((gemv_tile_list_kernel<B, 512>), dim3(total_tiles), dim3(64 * nw), nw * kExchangeBytes, stream, a, batch, wave_reciprocal(nw));
    return hipGetLastError();
}

hipError_t launch_matrix_tile_list(ListArgs &a, int b, int batch, hipStream_t stream)
{
    int total = 0, min_pairs = 1 << 30;
    bool long_rows = false;
    for (int i = 0; i < a.count; ++i) {
        a.group_begin[i] = total;
        total += (a.item[i].M + 15) / 16;
        const int npairs = (a.item[i].K / (8 * kChunkSlots) + 1) / 2;
        if (npairs < min_pairs) min_pairs = npairs;
        long_rows = a.item[i].K >= 12288;
    }
    for (int i = a.count; i < kMaxListItems; ++i) a.group_begin[i] = 0x7fffffff;
    const int nw = launch_waves(b, long_rows, min_pairs, total);
    switch (b) {
    case 3: return launch_tile_list_b<3>(a, total, nw, batch, stream);
    case 4: return launch_tile_list_b<4>(a, total, nw, batch, stream);
    case 5: return launch_tile_list_b<5>(a, total, nw, batch, stream);
    case 6: return launch_tile_list_b<6>(a, total, nw, batch, stream);
    case 7: return launch_tile_list_b<7>(a, total, nw, batch, stream);
    case 8: return launch_tile_list_b<8>(a, total, nw, batch, stream);
    }
    return hipErrorInvalidValue;
}

// batch 2..16
hipError_t launch_matrix_tile(const GemvArgs &a, hipStream_t stream)
{
    switch (a.b) {
    case 3: return launch_tile_b<3>(a, stream);
    case 4: return launch_tile_b<4>(a, stream);
    case 5: return launch_tile_b<5>(a, stream);
    case 6: return launch_tile_b<6>(a, stream);
    case 7: return launch_tile_b<7>(a, stream);
    case 8: return launch_tile_b<8>(a, stream);
    }
    return hipErrorInvalidValue;
}

} // namespace apgemv
