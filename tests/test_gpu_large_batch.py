"""GPU parity of the large-batch path: the dequantise kernel (bit-exact) and dequantise + dense GEMM."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2402_10517_amd import inputs
from gpu_util import check_against_oracle, check_planted, plant_infinities

pytestmark = pytest.mark.gpu
ALL_BITS = list(range(3, 9))


@pytest.fixture(scope="module")
def B():
    from paper_2402_10517_amd import binding
    return binding


@pytest.mark.parametrize("M,K", [(512, 512), (37, 96), (70, 2048 + 160), (10, 9 * 2048 + 32), (129, 4096)])
def test_dequantize_is_bit_exact(B, M, K):
    import torch
    idx, luts, _ = inputs.make_case(21, M, K)
    rng = np.random.default_rng(M + K)
    for b in ALL_BITS:                       # unsorted tables, signed zeros, subnormals, extremes
        t = luts[b][:, rng.permutation(1 << b)].copy()
        t[0, 0] = np.float16(-0.0)
        t[0, 1] = np.float16(6e-8)
        t[1 % M, 2] = np.float16(65504.0)
        luts[b] = t
    pm = B.ap_pack(idx, luts)
    guard = 64
    for b in ALL_BITS:
        buf = torch.full((guard + M * K + guard,), 7.0, dtype=torch.float16, device="cuda")
        w = buf[guard:guard + M * K].view(M, K)
        sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert B.lib.ap_dequantize(pm.handle, b, w.data_ptr(), sp) == 0
        torch.cuda.synchronize()
        out = buf.cpu().numpy()
        assert np.all(out[:guard] == 7.0) and np.all(out[-guard:] == 7.0)
        expect = luts[b].view(np.uint16)[np.arange(M)[:, None], idx >> (8 - b)]
        assert np.array_equal(out[guard:-guard].view(np.uint16).reshape(M, K), expect)
        # the oracle's own dense matrix is the same values
        assert np.array_equal(oracle.dequantize(idx, luts[b], b),
                              expect.view(np.float16).astype(np.float64))
    pm.close()


@pytest.mark.parametrize("batch", [1, 17, 40])
def test_gemm_path_against_oracle_small(B, batch):
    import torch
    M, K = 136, 2048 + 96
    idx, luts, x = inputs.make_case(22, M, K, batch=batch)
    pm = B.ap_pack(idx, luts)
    for b in (3, 5, 8):
        y = B.ap_gemm(pm, b, torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        check_against_oracle(y.cpu().numpy(), idx, luts[b], b, x)
    pm.close()


def test_gemm_path_llama_shape_sampled_rows(B):
    import torch
    M, K, batch = 11008, 4096, 64
    idx, luts, x = inputs.make_case(23, M, K, batch=batch, bit_widths=[4, 8])
    pm = B.ap_pack(idx, luts)
    rows = np.random.default_rng(1).integers(0, M, size=96)
    xd = torch.from_numpy(x).cuda()
    work = torch.empty(M * K * 2, dtype=torch.uint8, device="cuda")
    for b in (4, 8):
        y = B.ap_gemm(pm, b, xd, work=work)
        torch.cuda.synchronize()
        check_against_oracle(y.cpu().numpy(), idx, luts[b], b, x, rows=rows)
    # too small a workspace is rejected before any work is enqueued
    sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert B.lib.ap_gemm(pm.handle, 4, xd.data_ptr(), xd.data_ptr(), batch, work.data_ptr(), 1024, sp) == 5
    pm.close()


# sizes at the edges of the fused kernel: tiles of 64 rows (16 groups of 4), steps of 4 chunks (128 columns) with a ragged
# one, rows shorter than a step, several column parts (few row blocks, long rows), 1..4 tiles of 16 batch rows and several
# batch tiles; M not a multiple of 4
@pytest.mark.parametrize("M,K", [(1, 32), (63, 96), (65, 128), (130, 2048 + 160), (37, 9 * 2048 + 32), (260, 4096)])
@pytest.mark.parametrize("batch", [1, 16, 17, 48, 49, 64, 65, 130])
def test_fused_gemm_tile_edges(B, M, K, batch):
    import torch
    idx, luts, x = inputs.make_case(42, M, K, batch=batch)
    pm = B.ap_pack(idx, luts)
    guard = 64
    xd = torch.from_numpy(x).cuda()
    work = torch.empty(M * K * 2, dtype=torch.uint8, device="cuda")   # the smallest workspace the call accepts
    sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for b in ALL_BITS:
        for static in (False, True):
            buf = torch.full((guard + batch * M + guard,), -7.0, dtype=torch.float16, device="cuda")
            yp = buf.data_ptr() + 2 * guard
            if static:
                assert B.lib.ap_gemm_static(pm.handle, b, xd.data_ptr(), yp, batch, sp) == 0
            else:
                assert B.lib.ap_gemm(pm.handle, b, xd.data_ptr(), yp, batch, work.data_ptr(), work.numel(), sp) == 0
            torch.cuda.synchronize()
            out = buf.cpu().numpy()
            assert np.all(out[:guard] == -7.0) and np.all(out[-guard:] == -7.0)
            check_against_oracle(out[guard:-guard].reshape(batch, M), idx, luts[b], b, x)
    pm.close()


# more row blocks times batch tiles than CUs (4 waves per workgroup; 64 batch rows with 2 steps per wave, the most without a copy of
# x, and with a third, ragged one), and both sides of the largest batches that run on the fused kernel, in sampled rows
@pytest.mark.parametrize("M,K,batch,bits", [(16400, 160, 17, ALL_BITS), (16400, 160, 48, ALL_BITS), (16400, 160, 64, ALL_BITS),
                                            (5602, 1024, 190, ALL_BITS), (5602, 1056, 190, ALL_BITS),
                                            (700, 544, 256, [6, 8]), (700, 544, 257, [6, 8]), (700, 544, 384, [4, 5]),
                                            (700, 544, 385, [4, 5]), (700, 544, 512, [3]), (700, 544, 513, [3])])
def test_fused_gemm_many_workgroups_and_largest_batches(B, M, K, batch, bits):
    import torch
    idx, luts, x = inputs.make_case(47, M, K, batch=batch, bit_widths=bits)
    rows = np.unique(np.concatenate([np.arange(66), np.random.default_rng(batch).integers(0, M, size=64), np.arange(M - 70, M)]))
    pm = B.ap_pack(idx, luts)
    xd = torch.from_numpy(x).cuda()
    sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for b in bits:
        y = torch.full((batch, M), -7.0, dtype=torch.float16, device="cuda")
        assert B.lib.ap_gemm_static(pm.handle, b, xd.data_ptr(), y.data_ptr(), batch, sp) == 0
        for out in (B.ap_gemm(pm, b, xd), y):
            torch.cuda.synchronize()
            check_against_oracle(out.cpu().numpy(), idx, luts[b], b, x, rows=rows)
    pm.close()


# 64 batch rows per workgroup with a copy of x at every bit-width, on 8 waves: one column part, two and three (partial sums behind the
# copy; outputs whose number is and is not a multiple of 4); a ragged last step, M not a multiple of 64.  (M, K, batch, parts);
# test_fused_plan.py checks on the host that these are the plans
COPIED_X = [(2101, 2208, 250, 1), (1501, 4256, 250, 2), (1300, 6240, 250, 3)]


@pytest.mark.parametrize("M,K,batch,parts", COPIED_X)
def test_fused_gemm_with_a_copy_of_x(B, M, K, batch, parts):
    import torch
    idx, luts, x = inputs.make_case(53, M, K, batch=batch)
    rows = np.unique(np.concatenate([np.arange(66), np.random.default_rng(K).integers(0, M, size=30), np.arange(M - 70, M)]))
    pm = B.ap_pack(idx, luts)
    xd = torch.from_numpy(x).cuda()
    sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for b in ALL_BITS:
        y = torch.full((batch, M), -7.0, dtype=torch.float16, device="cuda")
        assert B.lib.ap_gemm_static(pm.handle, b, xd.data_ptr(), y.data_ptr(), batch, sp) == 0
        for out in (B.ap_gemm(pm, b, xd), y):
            torch.cuda.synchronize()
            check_against_oracle(out.cpu().numpy(), idx, luts[b], b, x, rows=rows)
    pm.close()


# ap_gemm_static in several passes: more rows than one pass takes, and rows so long that the copy of all of them exceeds the
# static array (passes of half the rows); and the sizes on either side of its dense kernel (DENSE_EDGES: the longest rows that it takes)
PASSES_OF_HALF_THE_ROWS = [(100, 38304, 500, [3, 8]), (20, 65536 + 96, 300, [8])]

DENSE_EDGES = [(96, 128, 700, [8]), (33, 128, 49, [8]), (209, 96, 300, [8]), (96, 64, 700, [3, 4, 5, 6, 7]), (209, 32, 300, [3, 4, 5, 6, 7]),
               (7, 256, 700, ALL_BITS)]


@pytest.mark.parametrize("M,K,batch,bits", PASSES_OF_HALF_THE_ROWS + DENSE_EDGES + [(M, K + 32, batch, bits) for M, K, batch, bits in DENSE_EDGES] +
                         [(2100, 2048, 2100, [5]), (20, 65536 + 96, 300, [3]), (96, 256, 700, ALL_BITS),
                          (96, 288, 700, [4, 7]), (33, 512, 49, [6, 8]), (33, 544, 49, [6, 8])])
def test_static_gemm_passes_and_dense_kernel(B, M, K, batch, bits):
    import torch
    idx, luts, x = inputs.make_case(48, M, K, batch=batch, bit_widths=bits)
    rows = np.unique(np.random.default_rng(batch).integers(0, M, size=24))
    pm = B.ap_pack(idx, luts)
    xd = torch.from_numpy(x).cuda()
    sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    guard = 64
    for b in bits:
        buf = torch.full((guard + batch * M + guard,), -7.0, dtype=torch.float16, device="cuda")
        assert B.lib.ap_gemm_static(pm.handle, b, xd.data_ptr(), buf.data_ptr() + 2 * guard, batch, sp) == 0
        torch.cuda.synchronize()
        out = buf.cpu().numpy()
        assert np.all(out[:guard] == -7.0) and np.all(out[-guard:] == -7.0)
        check_against_oracle(out[guard:-guard].reshape(batch, M), idx, luts[b], b, x, rows=rows)
    pm.close()


def test_fused_gemm_non_finite_values_stay_where_they_are(B):
    # one infinite weight in some rows (b = 3, 8; also in the ragged last step) and an infinity in one activation reach exactly
    # the outputs that use them; an x that is not 16-byte aligned gives the same values by the other route
    import torch
    M, K, batch = 70, 2048 + 160, 20
    for b in (3, 8):
        idx, luts, x = inputs.make_case(43, M, K, batch=batch, bit_widths=[b])
        cells = [(0, K - 1, 1), (5, K - 32, -1), (18, 2048 + 3, 1), (40, 2047, 1), (63, 0, -1), (69, 2048 + 50, 1)]
        plant_infinities(idx, luts[b], b, x, cells)
        x[3, 100] = np.float16(np.inf)
        w = luts[b][np.arange(M), idx[:, 100] >> (8 - b)].astype(np.float64)
        assert np.all(w != 0)
        with np.errstate(invalid="ignore"):
            row3 = np.inf * w
            for r, c, sign in cells:
                row3[r] += sign * np.inf * x[3, c].astype(np.float64)
        keep = np.arange(batch) != 3
        pm = B.ap_pack(idx, luts)
        xd = torch.from_numpy(x).cuda()
        shifted = torch.empty(batch * K + 1, dtype=torch.float16, device="cuda")[1:].view(batch, K)
        shifted.copy_(xd)
        ys = [B.ap_gemm(pm, b, xd), B.ap_gemm(pm, b, shifted)]
        torch.cuda.synchronize()
        for y in ys:
            got = y.cpu().numpy()
            check_planted(got[keep], idx, luts[b], b, x[keep], cells, rows=range(M))
            assert np.array_equal(got[3].astype(np.float64), row3, equal_nan=True)
        pm.close()
