"""GPU parity: the HIP path, called through the C-ABI, against the CPU oracle on the same inputs."""
import ctypes

import numpy as np
import pytest

from paper_2402_10517_amd import inputs
from gpu_util import check_against_oracle, check_planted, plant_infinities, run_gemv

pytestmark = pytest.mark.gpu
ALL_BITS = list(range(3, 9))


@pytest.fixture(scope="module")
def B():
    from paper_2402_10517_amd import binding
    return binding


@pytest.fixture(scope="module")
def tiny(B):
    idx, luts, x = inputs.make_case(1, 512, 512)
    pm = B.ap_pack(idx, luts)
    yield idx, luts, x, pm
    pm.close()


@pytest.mark.parametrize("b", ALL_BITS)
def test_config1_tiny_all_bit_widths(B, tiny, b):
    idx, luts, x, pm = tiny
    y = run_gemv(pm, b, x)
    check_against_oracle(y, idx, luts[b], b, x)


def test_device_round_trip_is_bit_exact(B, tiny):
    idx, _, _, pm = tiny
    assert np.array_equal(B.ap_unpack(pm), idx)
    for (M, K) in [(37, 2048 + 160), (5, 96)]:
        idx2, luts2, _ = inputs.make_case(11, M, K)
        pm2 = B.ap_pack(idx2, luts2)
        assert np.array_equal(B.ap_unpack(pm2), idx2)
        pm2.close()


# several spans per row, a ragged last span, rows not a multiple of 4, 1/2/4 waves per group
RAGGED = [(37, 96), (4, 32), (70, 2048 + 160), (129, 4096 + 32), (66, 3 * 2048), (10, 5 * 2048 + 736),
          (257, 9 * 2048 + 32)]


@pytest.mark.parametrize("M,K", RAGGED)
@pytest.mark.parametrize("b", ALL_BITS)
def test_ragged_shapes(B, M, K, b):
    idx, luts, x = inputs.make_case(12, M, K)
    pm = B.ap_pack(idx, {b: luts[b]})
    y = run_gemv(pm, b, x)
    check_against_oracle(y, idx, luts[b], b, x)
    pm.close()


@pytest.mark.parametrize("batch", range(1, 9))
@pytest.mark.parametrize("b", [3, 4, 6, 8])
def test_batches_one_to_eight(B, batch, b):
    M, K = 132, 2048 + 512
    idx, luts, x = inputs.make_case(13, M, K, batch=batch, sigma=0.01)
    pm = B.ap_pack(idx, {b: luts[b]})
    y = run_gemv(pm, b, x)
    assert y.shape == (batch, M)
    check_against_oracle(y, idx, luts[b], b, x)
    # a row of a batched call equals the batch-1 call on that row, bit for bit or within tolerance
    y0 = run_gemv(pm, b, x[batch - 1:batch])
    check_against_oracle(y0, idx, luts[b], b, x[batch - 1:batch])
    pm.close()


@pytest.mark.parametrize("batch", [9, 12, 16])
def test_batches_nine_to_sixteen_run_as_two_passes(B, batch):
    # rows 8.. of a larger batch equal a separate call on those rows, bit for bit; canaries around y;
    # shapes that reach the ALU kernels and (K % 256 == 0, forced) the tile kernel in both passes
    import ctypes
    import torch
    for (M, K, opts) in [(132, 2048 + 96, {}), (70, 2048 + 768, dict(variant=9))]:
        idx, luts, x = inputs.make_case(29, M, K, batch=batch, sigma=0.01)
        pm = B.ap_pack(idx, luts).set_options(**opts)
        guard = 64
        sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        xd = torch.from_numpy(x).cuda()
        for b in (3, 5, 8):
            ybuf = torch.full((guard + batch * M + guard,), -7.0, dtype=torch.float16, device="cuda")
            assert B.lib.ap_gemv(pm.handle, b, xd.data_ptr(), ybuf.data_ptr() + 2 * guard, batch, sp) == 0
            torch.cuda.synchronize()
            out = ybuf.cpu().numpy()
            assert np.all(out[:guard] == -7.0) and np.all(out[-guard:] == -7.0)
            y = out[guard:-guard].reshape(batch, M)
            check_against_oracle(y, idx, luts[b], b, x)
            y_tail = run_gemv(pm, b, x[8:])
            assert np.array_equal(y[8:].view(np.uint16), y_tail.view(np.uint16))
        pm.close()


@pytest.mark.parametrize("b", ALL_BITS)
def test_one_hot_activation_is_exact(B, b):
    M, K = 64, 2048 + 96
    idx, luts, _ = inputs.make_case(14, M, K)
    pm = B.ap_pack(idx, {b: luts[b]})
    for j in (0, 1, 7, 8, 511, 512, 1023, 2047, 2048, 2049, K - 33, K - 1):
        x = np.zeros((1, K), dtype=np.float16)
        x[0, j] = 1.0
        y = run_gemv(pm, b, x)
        expect = luts[b][np.arange(M), idx[:, j] >> (8 - b)]
        assert np.array_equal(y[0].view(np.uint16) & 0x7fff != 0, expect.view(np.uint16) & 0x7fff != 0)
        assert np.array_equal(y[0], expect), "column %d" % j
    pm.close()


@pytest.mark.parametrize("b", ALL_BITS)
def test_integer_table_pins_bit_order_end_to_end(B, b):
    M, K = 24, 2048 + 64
    idx, _, _ = inputs.make_case(15, M, K)
    lut = np.tile(np.arange(1 << b, dtype=np.float16), (M, 1))
    pm = B.ap_pack(idx, {b: lut})
    for j in (0, 5, 300, 2047, 2050, K - 1):
        x = np.zeros((1, K), dtype=np.float16)
        x[0, j] = 1.0
        y = run_gemv(pm, b, x)
        assert np.array_equal(y[0].astype(np.int64), idx[:, j].astype(np.int64) >> (8 - b))
    # a short all-ones prefix keeps the exact integer sum below 2048, so binary16 holds it exactly
    ncols = max(1, 2048 // (1 << b) // 2)
    x = np.zeros((1, K), dtype=np.float16)
    x[0, :ncols] = 1.0
    y = run_gemv(pm, b, x)
    assert np.array_equal(y[0].astype(np.int64), (idx[:, :ncols].astype(np.int64) >> (8 - b)).sum(axis=1))
    pm.close()


# kernel families for the adversarial inputs: the dispatcher's own choice, the one-row-per-lane
# matrix-core kernel for every b, the matrix-core kernel with in-wave exchange, the matrix-core kernel
# on tiles of 16 rows (one and two tiles per workgroup); the matrix-core kernels need K % 128 == 0
# (K % 256 == 0 on tiles) and batch >= 3 / >= 2, which the shapes below satisfy
FAMILIES = [dict(), dict(mfma_min_batch=-3), dict(variant=3), dict(variant=9), dict(variant=10)]


@pytest.mark.parametrize("family", range(len(FAMILIES)))
@pytest.mark.parametrize("batch", [1, 3, 5, 8])
@pytest.mark.parametrize("b", ALL_BITS)
def test_adversarial_tables(B, b, batch, family):
    M, K = 48, 2048 + 256
    assert K % 256 == 0                                   # so that the matrix-core kernels are reachable
    idx, luts, x = inputs.make_case(16, M, K, batch=batch)
    rng = np.random.default_rng(b)
    E = 1 << b
    lut = luts[b].copy()
    lut = lut[:, rng.permutation(E)]                      # unsorted
    lut[0, :] = np.float16(6.0e-8)                        # subnormals
    lut[1, ::2] = np.float16(-0.0)
    lut[2, :] = np.float16(0.25)                          # all entries equal
    lut[3, 0] = np.float16(65504.0)
    lut[3, E - 1] = np.float16(-65504.0)
    idx[5, :] = 0xA5                                      # a row whose indices are all equal
    xs = (x.astype(np.float32) * 1e-3).astype(np.float16) # keeps 65504 * x finite
    pm = B.ap_pack(idx, {b: lut}).set_options(**FAMILIES[family])
    for xv in (xs, np.zeros_like(x)):
        y = run_gemv(pm, b, xv)
        check_against_oracle(y, idx, lut, b, xv)
    pm.close()


@pytest.mark.parametrize("family", range(len(FAMILIES)))
@pytest.mark.parametrize("batch", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("b", ALL_BITS)
def test_subnormal_centroids_are_not_flushed(B, b, batch, family):
    # every centroid is a binary16 subnormal (k * 2^-24), activations are large: a path that
    # flushed subnormal inputs to zero (the matrix instructions included) would return 0 where the
    # result is of order 10
    M, K = 20, 2048 + 256
    assert K % 256 == 0
    rng = np.random.default_rng(100 + b)
    idx = rng.integers(0, 256, size=(M, K), dtype=np.uint8)
    lut = (rng.integers(1, 1024, size=(M, 1 << b)).astype(np.uint16)).view(np.float16)
    x = np.full((batch, K), 512.0, dtype=np.float16)
    x[:, ::3] = -256.0
    pm = B.ap_pack(idx, {b: lut}).set_options(**FAMILIES[family])
    y = run_gemv(pm, b, x)
    assert np.all(np.abs(y.astype(np.float64)) > 0.05)
    check_against_oracle(y, idx, lut, b, x)
    pm.close()


@pytest.mark.parametrize("rg", [2, 3, 4])
@pytest.mark.parametrize("batch", [1, 2, 5, 8])
def test_several_row_groups_per_workgroup(B, rg, batch):
    # the variant that keeps activations in registers across row groups, forced on small ragged
    # shapes: rows not a multiple of 4*rg, a ragged last span, 1..4 waves per group
    for (M, K) in [(4 * rg * 3 + 5, 2048 + 160), (7, 96), (4 * rg + 1, 3 * 2048 + 32 * 17)]:
        idx, luts, x = inputs.make_case(18, M, K, batch=batch, sigma=0.01)
        pm = B.ap_pack(idx, luts).set_options(row_groups=rg)
        for b in ALL_BITS:
            y = run_gemv(pm, b, x)
            check_against_oracle(y, idx, luts[b], b, x)
        pm.close()


@pytest.mark.parametrize("batch", [3, 4, 5, 8])
def test_matrix_core_variant_for_every_bit_width(B, batch):
    # forced for every b (the dispatcher uses it for b >= 6 only): several spans, a ragged last span
    # of 4-chunk blocks, rows not a multiple of 4 or 16, one and four row groups per workgroup
    for rg in (1, 4):
        for (M, K) in [(37, 128), (70, 2048 + 640), (21, 3 * 2048 + 128)]:
            idx, luts, x = inputs.make_case(19, M, K, batch=batch, sigma=0.01)
            pm = B.ap_pack(idx, luts).set_options(mfma_min_batch=-3, row_groups=rg)
            for b in ALL_BITS:
                y = run_gemv(pm, b, x)
                check_against_oracle(y, idx, luts[b], b, x)
            pm.close()


@pytest.mark.parametrize("batch", [2, 3, 4, 5, 7, 8])
def test_matrix_core_variant_with_in_block_exchange(B, batch):
    # forced for every b and batch >= 2: one span, several spans with a ragged last span of 4-chunk
    # blocks, more spans than waves (a wave takes two spans), rows not a multiple of 4
    # one, two and four row groups per workgroup (the last two reuse the activations of a span)
    for rg in (1, 2, 4):
        for (M, K) in [(37, 128), (70, 2048 + 640), (21, 3 * 2048 + 128), (9, 9 * 2048 + 256)]:
            idx, luts, x = inputs.make_case(21, M, K, batch=batch, sigma=0.01)
            pm = B.ap_pack(idx, luts).set_options(variant=B.VARIANT_EXCHANGE, row_groups=rg)
            for b in ALL_BITS:
                y = run_gemv(pm, b, x)
                check_against_oracle(y, idx, luts[b], b, x)
            pm.close()


@pytest.mark.parametrize("batch", [2, 3, 4, 5, 6, 7, 8])
def test_matrix_core_variant_on_tiles_of_16_rows(B, batch):
    # forced for every b and batch >= 2: one octet of chunks, several spans with a ragged last span, an
    # odd number of octets, more octet pairs than waves, rows not a multiple of 4 or 16 (tiles and row
    # groups partly or wholly past the matrix), one and two tiles per workgroup; workgroups of 1, 2, 3, 4 and 8
    # waves (the pair tables of the 3- and 4-bit paths are built by a different loop at 4 and 8 waves)
    for variant in (B.VARIANT_TILE, B.VARIANT_TILE2):
        for (M, K) in [(37, 256), (70, 2048 + 768), (21, 3 * 2048 + 256), (9, 9 * 2048 + 512), (130, 4096), (16, 512),
                       (20, 768), (40, 1280)]:
            idx, luts, x = inputs.make_case(27, M, K, batch=batch, sigma=0.01)
            pm = B.ap_pack(idx, luts).set_options(variant=variant)
            for b in ALL_BITS:
                y = run_gemv(pm, b, x)
                check_against_oracle(y, idx, luts[b], b, x)
            pm.close()


@pytest.mark.parametrize("b", [7, 8])
def test_bank_per_lane_variant(B, b):
    # forced (the dispatcher does not choose it): one lane per LDS bank column, 8 copies of a table,
    # a lane owns one row of 4 chunks: ragged spans whose last quad is partly filled, rows not a
    # multiple of 4, 1..8 waves per group (1, 2, 4, 8 or 16 table pieces per thread), unsorted tables
    rng = np.random.default_rng(40 + b)
    for (M, K) in RAGGED + [(512, 512), (33, 8 * 2048), (6, 14 * 2048)]:
        idx, luts, x = inputs.make_case(24, M, K, bit_widths=[b])
        lut = luts[b][:, rng.permutation(1 << b)].copy()
        pm = B.ap_pack(idx, {b: lut}).set_options(variant=B.VARIANT_BANK_PER_LANE)
        y = run_gemv(pm, b, x)
        check_against_oracle(y, idx, lut, b, x)
        pm.close()


@pytest.mark.parametrize("b", ALL_BITS)
def test_two_row_groups_per_workgroup_variant(B, b):
    # forced (the dispatcher uses it on large matrices only): 2..8 spans, a ragged last span, an odd
    # number of row groups (the last workgroup holds one group), rows not a multiple of 4; the outputs
    # are bit-identical to the kernel with one group per workgroup, except where that kernel runs a ragged
    # last span of at most 32 chunks on both halves of the wave (b = 4, 5, 6), which this variant does not
    for (M, K) in [(70, 2048 + 160), (129, 4096 + 32), (66, 3 * 2048), (10, 5 * 2048 + 736), (4, 8 * 2048), (37, 2048 + 32)]:
        idx, luts, x = inputs.make_case(26, M, K, bit_widths=[b])
        pm = B.ap_pack(idx, luts).set_options(variant=B.VARIANT_PAIR)
        y = run_gemv(pm, b, x)
        check_against_oracle(y, idx, luts[b], b, x)
        pm.set_options(variant=B.VARIANT_NO_PAIR)
        y1 = run_gemv(pm, b, x)
        check_against_oracle(y1, idx, luts[b], b, x)
        ragged = (K // 32) % 64
        if not (b in (4, 5, 6) and 0 < ragged <= 32):
            assert np.array_equal(y.view(np.uint16), y1.view(np.uint16))
        pm.close()


@pytest.mark.parametrize("batch", [1, 2, 8])
def test_fused_launch_equals_separate_calls(B, batch):
    import torch
    K = 2048 + 256
    mats = []
    for k, M in enumerate([64, 37, 130, 8]):
        idx, luts, x = inputs.make_case(20, M, K, batch=batch, salt=k)
        mats.append((idx, luts, x, B.ap_pack(idx, luts)))
    shared_x = torch.from_numpy(mats[0][2]).cuda()
    for b in ALL_BITS:
        for count in (1, 3, 4):
            triples, ys = [], []
            for (idx, luts, x, pm) in mats[:count]:
                y = torch.full((batch, pm.M), -3.0, dtype=torch.float16, device="cuda")
                triples.append((pm, shared_x, y))
            B.ap_gemv_multi(triples, b)
            torch.cuda.synchronize()
            for (idx, luts, x, pm), (_, _, y) in zip(mats[:count], triples):
                sep = B.ap_gemv(pm, b, shared_x)
                torch.cuda.synchronize()
                if batch <= 2:   # same kernel as the single call: bit-identical
                    assert np.array_equal(y.cpu().numpy().view(np.uint16), sep.cpu().numpy().view(np.uint16))
                check_against_oracle(y.cpu().numpy(), idx, luts[b], b, mats[0][2])
    # row lengths must agree at batch >= 2; at batch 1 any shapes share the launch
    idx, luts, x = inputs.make_case(20, 16, 512, batch=batch)
    other = B.ap_pack(idx, luts)
    y0 = torch.empty((batch, 64), dtype=torch.float16, device="cuda")
    y1 = torch.full((batch, 16), -3.0, dtype=torch.float16, device="cuda")
    x1 = torch.from_numpy(x).cuda()
    if batch == 1:
        B.ap_gemv_multi([(mats[0][3], shared_x, y0), (other, x1, y1)], 4)
        torch.cuda.synchronize()
        check_against_oracle(y1.cpu().numpy(), idx, luts[4], 4, x)
        check_against_oracle(y0.cpu().numpy(), mats[0][0], mats[0][1][4], 4, mats[0][2])
    else:
        with pytest.raises(B.ApError) as e:
            B.ap_gemv_multi([(mats[0][3], shared_x, y0), (other, x1, y1)], 4)
        assert e.value.status == 2
    for m in mats:
        m[3].close()
    other.close()


@pytest.mark.parametrize("batch", [2, 3, 5, 8])
def test_fused_launch_on_the_tile_kernel(B, batch):
    # forced through the first handle (the library chooses it from 1024 row groups per launch on): rows not
    # a multiple of 16, a matrix smaller than a tile, a ragged last span, canaries around every output
    import torch
    K = 2048 + 768
    mats = []
    for k, M in enumerate([70, 37, 130, 8, 16]):
        idx, luts, x = inputs.make_case(31, M, K, batch=batch, salt=k)
        mats.append((idx, luts, x, B.ap_pack(idx, luts)))
    mats[0][3].set_options(variant=B.VARIANT_TILE)
    shared_x = torch.from_numpy(mats[0][2]).cuda()
    guard = 32
    for b in ALL_BITS:
        for count in (1, 3, 5):
            triples, bufs = [], []
            for (idx, luts, x, pm) in mats[:count]:
                buf = torch.full((guard + batch * pm.M + guard,), -3.0, dtype=torch.float16, device="cuda")
                bufs.append(buf)
                triples.append((pm, shared_x, buf[guard:guard + batch * pm.M].view(batch, pm.M)))
            B.ap_gemv_multi(triples, b)
            torch.cuda.synchronize()
            for (idx, luts, x, pm), buf in zip(mats[:count], bufs):
                out = buf.cpu().numpy()
                assert np.all(out[:guard] == -3.0) and np.all(out[-guard:] == -3.0)
                check_against_oracle(out[guard:-guard].reshape(batch, pm.M), idx, luts[b], b, mats[0][2])
                # the same arithmetic as a single call on the tile kernel: bit-identical
                pm.set_options(variant=B.VARIANT_TILE)
                sep = B.ap_gemv(pm, b, shared_x)
                torch.cuda.synchronize()
                assert np.array_equal(out[guard:-guard].reshape(batch, pm.M).view(np.uint16), sep.cpu().numpy().view(np.uint16))
    for m in mats:
        m[3].close()


@pytest.mark.parametrize("batch", [2, 5, 8])
def test_batched_work_list(B, batch):
    # items of several shapes and bit-widths: groups large enough for the tile kernel (same b, rows of one
    # class of length, >= 1024 row groups together) share a launch, the others run as single calls;
    # canaries around every output; a tile-kernel item is bit-identical to the single call on that kernel
    import ctypes
    import torch
    shapes = [(2100, 2048), (2050, 2304), (37, 256), (70, 2048 + 96), (2060, 12288), (2100, 12288 + 256), (16, 12544)]
    mats = []
    for k, (M, K) in enumerate(shapes):
        idx, luts, x = inputs.make_case(33, M, K, batch=batch, salt=k, bit_widths=[3, 4, 8], sigma=0.01)
        mats.append((idx, luts, x, B.ap_pack(idx, luts), torch.from_numpy(x).cuda()))
    guard = 32
    quads, bufs, meta = [], [], []
    for rep, bsel in enumerate([(3, 3, 4, 3, 4, 4, 4), (8, 8, 4, 8, 4, 4, 3)]):
        for (idx, luts, x, pm, xd), b in zip(mats, bsel):
            buf = torch.full((guard + batch * pm.M + guard,), -5.0, dtype=torch.float16, device="cuda")
            bufs.append(buf)
            quads.append((pm, b, xd, buf[guard:guard + batch * pm.M].view(batch, pm.M)))
            meta.append((idx, luts, x, pm, xd, b))
    B.ap_gemv_list_batch(quads, batch)
    torch.cuda.synchronize()
    for (idx, luts, x, pm, xd, b), buf in zip(meta, bufs):
        out = buf.cpu().numpy()
        assert np.all(out[:guard] == -5.0) and np.all(out[-guard:] == -5.0)
        y = out[guard:-guard].reshape(batch, pm.M)
        check_against_oracle(y, idx, luts[b], b, x)
    if batch == 2:
        # batch 2: every item ran in a list launch of the kernel that single calls use, bit for bit
        for k, (idx, luts, x, pm, xd, b) in enumerate(meta):
            sep = B.ap_gemv(pm, b, xd)
            torch.cuda.synchronize()
            assert np.array_equal(bufs[k].cpu().numpy()[guard:-guard].reshape(batch, pm.M).view(np.uint16),
                                  sep.cpu().numpy().view(np.uint16))
    else:
        # the first two items of the first half (b = 3, 2048 and 2304 columns: 1038 row groups together) ran on
        # the tile kernel with 4 waves per tile, like a single call on it
        for k in (0, 1):
            idx, luts, x, pm, xd, b = meta[k]
            pm.set_options(variant=B.VARIANT_TILE)
            sep = B.ap_gemv(pm, b, xd)
            torch.cuda.synchronize()
            assert np.array_equal(bufs[k].cpu().numpy()[guard:-guard].reshape(batch, pm.M).view(np.uint16),
                                  sep.cpu().numpy().view(np.uint16))
            pm.set_options(variant=B.VARIANT_AUTO)
    # argument checks: status of the first bad item, nothing enqueued; batch range
    bad = list(quads)
    bad[3] = (quads[3][0], 5, quads[3][2], quads[3][3])       # no table for b = 5
    with pytest.raises(B.ApError) as e:
        B.ap_gemv_list_batch(bad, batch)
    assert e.value.status == 3
    with pytest.raises(B.ApError) as e:
        B.ap_gemv_list_batch(quads, 9)
    assert e.value.status == 6
    for m in mats:
        m[3].close()


def test_work_list_mixed_shapes_and_bit_widths(B):
    # one launch per 32 items: 40 items of 7 different shapes (1..9 spans, ragged spans, rows not a
    # multiple of 4), each with its own bit-width; every output bit-identical to a separate ap_gemv
    # call and within tolerance of the oracle; canaries between the outputs stay untouched
    import torch
    shapes = [(37, 96), (64, 2048 + 160), (130, 4096 + 32), (8, 512), (21, 3 * 2048), (5, 9 * 2048 + 32), (257, 1024)]
    mats = []
    for k, (M, K) in enumerate(shapes):
        idx, luts, x = inputs.make_case(25, M, K, salt=k)
        mats.append((idx, luts, x, B.ap_pack(idx, luts), torch.from_numpy(x).cuda()))
    rng = np.random.default_rng(25)
    picks = [(int(rng.integers(0, len(shapes))), int(rng.integers(3, 9))) for _ in range(40)]
    guard = 16
    total = sum(mats[m][3].M + guard for m, _ in picks) + guard
    ybuf = torch.full((total,), -7.0, dtype=torch.float16, device="cuda")
    quads, offs, off = [], [], guard
    for m, b in picks:
        M = mats[m][3].M
        quads.append((mats[m][3], b, mats[m][4], ybuf[off:off + M]))
        offs.append(off)
        off += M + guard
    B.ap_gemv_list(quads)
    torch.cuda.synchronize()
    out = ybuf.cpu().numpy()
    mask = np.ones(total, dtype=bool)
    for (m, b), o in zip(picks, offs):
        idx, luts, x, pm, xd = mats[m]
        y = out[o:o + pm.M].reshape(1, -1)
        mask[o:o + pm.M] = False
        sep = B.ap_gemv(pm, b, xd)
        torch.cuda.synchronize()
        assert np.array_equal(y.view(np.uint16), sep.cpu().numpy().view(np.uint16)), (m, b)
        check_against_oracle(y, idx, luts[b], b, x)
    assert np.all(out[mask] == -7.0)
    # a bad item anywhere in the list: its status, and nothing is enqueued
    ybuf.fill_(-7.0)
    bad = list(quads)
    pm3 = B.ap_pack(mats[0][0], {3: mats[0][1][3]})
    bad[35] = (pm3, 5, mats[0][4], ybuf[offs[35]:offs[35] + pm3.M])          # no table for b = 5
    with pytest.raises(B.ApError) as e:
        B.ap_gemv_list(bad)
    assert e.value.status == 3
    torch.cuda.synchronize()
    assert np.all(ybuf.cpu().numpy() == -7.0)
    assert B.lib.ap_gemv_list(None, 1, None) == 1
    assert B.lib.ap_gemv_list(B.make_list(quads), 0, None) == 1
    pm3.close()
    for m in mats:
        m[3].close()


def test_graph_capture_and_replay_match_eager(B, tiny):
    # ap_gemv and ap_gemv_multi allocate nothing and synchronise nothing, so a stream capture can
    # record them; every replay (with eager work and synchronisations in between) must reproduce
    # the eager result bit for bit
    import torch
    idx, luts, x, pm = tiny
    xd = torch.from_numpy(x).cuda()
    eager = {b: B.ap_gemv(pm, b, xd).clone() for b in ALL_BITS}
    torch.cuda.synchronize()
    ys = {b: torch.zeros((1, pm.M), dtype=torch.float16, device="cuda") for b in ALL_BITS}
    ym = torch.zeros((1, pm.M), dtype=torch.float16, device="cuda")
    cap = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(cap):
        for b in ALL_BITS:                       # warm-up on the capture stream
            B.ap_gemv(pm, b, xd, y=ys[b], stream=cap)
        cap.synchronize()
        with torch.cuda.graph(g, stream=cap):
            for b in ALL_BITS:
                B.ap_gemv(pm, b, xd, y=ys[b], stream=cap)
            B.ap_gemv_multi([(pm, xd, ym)], 5, stream=cap)
    torch.cuda.synchronize()
    for rep in range(4):
        for b in ALL_BITS:
            ys[b].zero_()
        ym.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for b in ALL_BITS:
            assert torch.equal(ys[b], eager[b]), (rep, b)
        assert torch.equal(ym, eager[5])
        # eager work between replays
        assert torch.equal(B.ap_gemv(pm, 4 + rep % 3, xd), eager[4 + rep % 3])
        torch.cuda.synchronize()


def test_dispatch_sequence_without_repacking_and_determinism(B, tiny):
    import torch
    idx, luts, x, pm = tiny
    before = pm.buf.clone()
    fresh = {b: run_gemv(pm, b, x) for b in ALL_BITS}
    rng = np.random.default_rng(4)
    for b in rng.integers(3, 9, size=24).tolist():
        y = run_gemv(pm, b, x)
        assert np.array_equal(y.view(np.uint16), fresh[b].view(np.uint16))   # bit-identical repeats
    assert torch.equal(before, pm.buf)                                         # blob untouched


def test_output_canaries_and_sparse_support(B):
    import torch
    M, K = 100, 2048 + 64
    idx, luts, x = inputs.make_case(17, M, K, batch=3)
    pm = B.ap_pack(idx, {3: luts[3], 4: luts[4], 8: luts[8]})
    guard = 64
    ybuf = torch.full((guard + 3 * M + guard,), -7.0, dtype=torch.float16, device="cuda")
    xd = torch.from_numpy(x).cuda()
    sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for b in (3, 4, 8):
        st = B.lib.ap_gemv(pm.handle, b, xd.data_ptr(), ybuf.data_ptr() + 2 * guard, 3, sp)
        assert st == 0
        torch.cuda.synchronize()
        out = ybuf.cpu().numpy()
        assert np.all(out[:guard] == -7.0) and np.all(out[-guard:] == -7.0)
        check_against_oracle(out[guard:-guard].reshape(3, M), idx, luts[b], b, x)
    for b in (5, 6, 7, 2, 9):
        assert B.lib.ap_gemv(pm.handle, b, xd.data_ptr(), ybuf.data_ptr(), 3, sp) == 3
    assert B.lib.ap_gemv(pm.handle, 3, xd.data_ptr(), ybuf.data_ptr(), 0, sp) == 6
    assert B.lib.ap_gemv(pm.handle, 3, xd.data_ptr(), ybuf.data_ptr(), 17, sp) == 6
    assert B.lib.ap_gemv(pm.handle, 3, xd.data_ptr() + 2, ybuf.data_ptr(), 1, sp) == 1
    pm.close()


def test_option_values_are_checked(B, tiny):
    _, _, _, pm = tiny
    L = B.lib
    for opt, bad in ((0, 9), (0, -1), (1, 0), (1, 5), (2, 10), (3, 2), (3, 6), (3, 11), (9, 0)):
        assert L.ap_set_option(pm.handle, opt, bad) == 1, (opt, bad)
    for opt, good, default in ((0, 2, 0), (1, 1, -1), (2, 9, 0), (3, 1, 0)):
        assert L.ap_set_option(pm.handle, opt, good) == 0
        assert L.ap_set_option(pm.handle, opt, default) == 0


def test_smaller_parent_bit_width(B):
    n, M, K = 6, 40, 2048 + 32
    rng = np.random.default_rng(6)
    idx = rng.integers(0, 1 << n, size=(M, K), dtype=np.uint8)
    luts = {b: rng.normal(0, 0.02, size=(M, 1 << b)).astype(np.float16) for b in range(3, n + 1)}
    x = rng.normal(0, 1, size=(2, K)).astype(np.float16)
    pm = B.ap_pack(idx, luts, n=n)
    for b in range(3, n + 1):
        y = run_gemv(pm, b, x)
        check_against_oracle(y, idx, luts[b], b, x, n=n)
    pm.close()


def test_attach_to_a_device_copy(B, tiny):
    idx, luts, x, pm = tiny
    pm2 = pm.clone()
    assert pm2.buf.data_ptr() != pm.buf.data_ptr()
    for b in (3, 8):
        assert np.array_equal(run_gemv(pm2, b, x).view(np.uint16), run_gemv(pm, b, x).view(np.uint16))
    pm2.close()


@pytest.mark.parametrize("batch", [1, 4])
def test_quantised_model_end_to_end(B, batch):
    # weights -> incremental upscaling (host) -> pack -> GEMV at every bit-width; the oracle takes
    # the same indices and tables, and the b-bit result must approach the dense product as b grows
    rng = np.random.default_rng([20240210, 31, batch])
    M, K = 96, 2048 + 320
    W = rng.standard_t(5, (M, K)).astype(np.float32) * 0.02
    S = (rng.gamma(0.5, 1.0, (M, K)) + 1e-6).astype(np.float32)
    idx, luts = B.ap_quantize(W, S, 3, 8, 15)
    x = rng.normal(0, 1, (batch, K)).astype(np.float16)
    pm = B.ap_pack(idx, luts)
    dense = x.astype(np.float64) @ W.astype(np.float64).T
    errs = []
    for b in ALL_BITS:
        y = run_gemv(pm, b, x)
        check_against_oracle(y, idx, luts[b], b, x)
        errs.append(float(np.sqrt(np.mean((y.astype(np.float64) - dense) ** 2))))
    assert errs[-1] < errs[0] / 8 and errs[3] < errs[0]
    pm.close()


@pytest.mark.parametrize("seed", range(6))
def test_random_shapes_bit_widths_and_batches(B, seed):
    # a seeded sweep over shapes the fixed cases do not name: any M, any K % 32 == 0 up to ~5 spans,
    # random supported sets of bit-widths, every batch size; default dispatch
    rng = np.random.default_rng([20240210, 99, seed])
    for _ in range(8):
        M = int(rng.integers(1, 300))
        K = 32 * int(rng.integers(1, 330))
        batch = int(rng.integers(1, 9))
        bits = sorted(set(int(v) for v in rng.integers(3, 9, size=3)))
        idx, luts, x = inputs.make_case(30 + seed, M, K, batch=batch, sigma=0.02, bit_widths=bits)
        pm = B.ap_pack(idx, luts)
        for b in bits:
            y = run_gemv(pm, b, x)
            check_against_oracle(y, idx, luts[b], b, x)
        assert np.array_equal(B.ap_unpack(pm), idx)
        pm.close()


def test_issue_probe_runs_every_kind(B):
    """The measurement aid launches and completes for every kind (it has no output to compare)."""
    import torch
    for kind in range(7):
        assert B.lib.ap_probe_issue(kind, 3, None) == 0
    torch.cuda.synchronize()



@pytest.mark.parametrize("batch", [3, 5, 8, 9, 13, 16])
def test_tile_kernel_on_ragged_rows_and_at_batch_nine_to_sixteen(B, batch):
    # matrices tall enough for the dispatcher to choose the kernel by itself: rows of fewer chunks than an octet, an octet
    # of 1, 4 or 7 chunks at the end, an odd number of octets, whole octets (batch 9 and more), a last tile of fewer than
    # 16 rows and one or two tiles per workgroup; canaries around y.  An infinity in the table of one row and in the last
    # column of x reaches exactly the outputs that use it.
    import ctypes
    import torch
    shapes = [(8195, 32), (3073, 8192 + 32), (4099, 8192 + 128 + 96), (8196, 256 + 224), (4100, 512), (15363, 768)]
    for (M, K) in shapes:
        rows = np.unique(np.concatenate([np.arange(20), np.random.default_rng(M).integers(0, M, size=60), np.arange(M - 20, M)]))
        idx, luts, x = inputs.make_case(44, M, K, batch=batch, sigma=0.01)
        guard = 64
        sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        for b in ALL_BITS:
            pm = B.ap_pack(idx, {b: luts[b]})
            xd = torch.from_numpy(x).cuda()
            ybuf = torch.full((guard + batch * M + guard,), -7.0, dtype=torch.float16, device="cuda")
            assert B.lib.ap_gemv(pm.handle, b, xd.data_ptr(), ybuf.data_ptr() + 2 * guard, batch, sp) == 0
            torch.cuda.synchronize()
            out = ybuf.cpu().numpy()
            assert np.all(out[:guard] == -7.0) and np.all(out[-guard:] == -7.0)
            check_against_oracle(out[guard:-guard].reshape(batch, M), idx, luts[b], b, x, rows=rows)
            pm.close()
    # one infinite weight in the row's single ragged chunk, an infinity in the last column of x
    M, K, b = 3073, 8192 + 32, 5
    idx, luts, x = inputs.make_case(45, M, K, batch=batch, bit_widths=[b])
    cells = [(7, K - 5, 1)]
    plant_infinities(idx, luts[b], b, x, cells)
    pm = B.ap_pack(idx, luts)
    check_planted(run_gemv(pm, b, x), idx, luts[b], b, x, cells, rows=range(64))
    w = luts[b][np.arange(64), idx[:64, K - 1] >> (8 - b)].astype(np.float64)
    assert np.all(w != 0)
    x[1, K - 1] = np.float16(-np.inf)
    got = run_gemv(pm, b, x)
    keep = np.arange(batch) != 1
    check_planted(got[keep], idx, luts[b], b, x[keep], cells, rows=range(64))
    with np.errstate(invalid="ignore"):
        expect = -np.inf * w
        expect[7] += np.inf * x[1, K - 5].astype(np.float64)
    assert np.array_equal(got[1, :64].astype(np.float64), expect, equal_nan=True)
    pm.close()


# tables of 128 and 256 entries staged by workgroups of 1, 2 and 3 waves, in one tile per workgroup and in two (batch 16)
@pytest.mark.parametrize("K", [512, 1024, 1504])
@pytest.mark.parametrize("M,batch", [(4099, 5), (14355, 8), (14355, 16)])
def test_tile_kernel_large_tables_from_few_waves(B, M, batch, K):
    rows = np.unique(np.concatenate([np.arange(34), np.random.default_rng(K).integers(0, M, size=60), np.arange(M - 34, M)]))
    idx, luts, x = inputs.make_case(50, M, K, batch=batch, sigma=0.01, bit_widths=[7, 8])
    pm = B.ap_pack(idx, luts)
    for b in (7, 8):
        check_against_oracle(run_gemv(pm, b, x), idx, luts[b], b, x, rows=rows)
    pm.close()


# more workgroups than CUs on rows of more than 2048 columns, whose dropped loads are left out: an odd and an even number of octets, a
# ragged row, and both sides of 256 workgroups, in sampled rows
@pytest.mark.parametrize("K", [2304, 4096, 2080])
@pytest.mark.parametrize("M,batch", [(4096, 8), (4099, 8), (4099, 16)])
def test_tile_kernel_leaves_out_dropped_loads(B, M, batch, K):
    rows = np.unique(np.concatenate([np.arange(18), np.random.default_rng(K).integers(0, M, size=40), np.arange(M - 18, M)]))
    idx, luts, x = inputs.make_case(51, M, K, batch=batch, sigma=0.01)
    pm = B.ap_pack(idx, luts)
    for b in ALL_BITS:
        check_against_oracle(run_gemv(pm, b, x), idx, luts[b], b, x, rows=rows)
    pm.close()


# two tiles per workgroup on ragged rows: at 3 bits on tall matrices, on long rows, and at batch 9 to 16
@pytest.mark.parametrize("M,K,batch,bits", [(24580, 416, 8, [3]), (8180, 16384 + 32, 5, [4]), (15363, 800, 16, ALL_BITS),
                                            (8190, 288, 9, ALL_BITS)])
def test_two_tiles_per_workgroup_on_ragged_rows(B, M, K, batch, bits):
    rows = np.unique(np.concatenate([np.arange(34), np.random.default_rng(M).integers(0, M, size=60), np.arange(M - 34, M)]))
    idx, luts, x = inputs.make_case(49, M, K, batch=batch, sigma=0.01, bit_widths=bits)
    pm = B.ap_pack(idx, luts)
    for b in bits:
        check_against_oracle(run_gemv(pm, b, x), idx, luts[b], b, x, rows=rows)
    pm.close()


def _octet_cells(M, K):
    """One cell per row: columns of the last octet of 256 columns (its first and last chunk, the first and the last of
    its four runs) and of the first one; rows of different tiles."""
    span0 = (K - 1) // 2048 * 2048
    nl = (K - span0) // 32                        # chunks of the last span; chunk c holds columns span0 + 8 nl t + 8 c .. + 7
    first, last = 8 * ((nl - 1) // 8), nl - 1
    cols = [span0 + 8 * nl * t + 8 * c + 3 * t % 8 for c in (first, last) for t in (0, 3)] + [0]
    rows = [0, 5, 18, M // 2, M - 1, 40]
    return [(r, c, sign) for r, c, sign in zip(rows, cols + [K - 1], (1, -1, 1, 1, -1, 1))]


# Odd and even numbers of octets, whole and ragged, at sizes that the dispatcher gives to the tile kernel with one and with two
# tiles per workgroup: an octet that only pads a row to a pair of them must not reach the result, and infinity x 0 would.
@pytest.mark.parametrize("M,K,bits", [(8190, 32, [3, 4, 5, 8]), (8190, 256, [3, 4, 5, 8]), (8190, 544, [3, 4, 5, 8]),
                                      (8190, 768, [3, 4, 5, 8]), (8190, 800, [3, 4, 5, 8]), (8190, 1024, [3, 4, 5, 8]),
                                      (3073, 8192 + 32, [3, 6]), (3073, 8192 + 256, [4, 7]), (24577, 768, [3, 8])])
@pytest.mark.parametrize("batch", [3, 8, 16])
def test_infinite_centroid_in_the_last_octet(B, M, K, bits, batch):
    import ctypes
    import torch
    sp = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    cells = _octet_cells(M, K)
    rows = np.unique(np.concatenate([np.arange(48), np.random.default_rng(M).integers(0, M, size=40), np.arange(M - 20, M)]))
    idx0, luts, x = inputs.make_case(46, M, K, batch=batch, sigma=0.01, bit_widths=bits)
    for b in bits:
        idx = idx0.copy()
        plant_infinities(idx, luts[b], b, x, cells)
        pm = B.ap_pack(idx, luts)
        pm2 = pm.clone()
        xd = torch.from_numpy(x).cuda()
        outs = [B.ap_gemv(pm, b, xd), B.ap_gemm(pm, b, xd)]
        if M * K * 2 <= 32 << 20:
            y = torch.empty((batch, M), dtype=torch.float16, device="cuda")
            assert B.lib.ap_gemm_static(pm.handle, b, xd.data_ptr(), y.data_ptr(), batch, sp) == 0
            outs.append(y)
        if batch <= 8:
            ys = [torch.empty((batch, M), dtype=torch.float16, device="cuda") for _ in range(4)]
            B.ap_gemv_list_batch([(pm, b, xd, ys[0]), (pm2, b, xd, ys[1])], batch)
            B.ap_gemv_multi([(pm, xd, ys[2]), (pm2, xd, ys[3])], b)
            outs += ys
        torch.cuda.synchronize()
        for y in outs:
            check_planted(y.cpu().numpy(), idx, luts[b], b, x, cells, rows)
        pm.close()
        pm2.close()


def test_binding_outputs_streams_and_errors(B, tiny):
    # a given y is filled and returned, a vector x gives one row, another stream is used when named and when current, and a
    # refused call (missing bit-width, closed matrix, small workspace) raises the library's status
    import torch
    idx, luts, x = inputs.make_case(1, 512, 512, batch=3)
    pm = B.ap_pack(idx, {4: luts[4]})
    xd = torch.from_numpy(x).cuda()
    expect = B.ap_gemv(pm, 4, xd)
    assert expect.shape == (3, 512) and expect.dtype == torch.float16 and expect.device == xd.device
    assert torch.equal(B.ap_gemv(pm, 4, xd[0]), B.ap_gemv(pm, 4, xd[:1]))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for call in (B.ap_gemv, B.ap_gemm):
        y = torch.full((3, 512), -7.0, dtype=torch.float16, device="cuda")
        assert call(pm, 4, xd, y=y) is y and torch.equal(y, expect)
        y.fill_(-7.0)
        side.wait_stream(torch.cuda.current_stream())
        call(pm, 4, xd, y=y, stream=side)
        side.synchronize()
        assert torch.equal(y, expect)
        with torch.cuda.stream(side):
            y2 = call(pm, 4, xd)
        side.synchronize()
        assert torch.equal(y2, expect)
        with pytest.raises(B.ApError) as e:
            call(pm, 5, xd)
        assert e.value.status == 3
        with pytest.raises(AssertionError):
            call(pm, 4, xd.t())
    with pytest.raises(B.ApError) as e:
        B.ap_gemm(pm, 4, xd, work=torch.empty(1024, dtype=torch.uint8, device="cuda"))
    assert e.value.status == 5
    pm.close()
    for call in (B.ap_gemv, B.ap_gemm):
        with pytest.raises(B.ApError) as e:
            call(pm, 4, xd)
        assert e.value.status == 1


def _pool_stream(address):
    """The stream whose blocks of the caching allocator hold this address."""
    import torch
    for s in torch.cuda.memory_snapshot():
        if s["address"] <= address < s["address"] + s["total_size"]:
            return s["stream"]
    raise AssertionError("not the allocator's memory")


def test_memory_of_a_call_on_a_named_stream_is_that_streams(B):
    # what the binding allocates for a call on a stream that is not current comes from that stream's blocks (so work queued on the
    # current stream neither uses nor gets them meanwhile), and a returned tensor's block also waits for the current stream
    import torch
    M, K, batch = 2048 + 16, 2048, 40
    idx, luts, x = inputs.make_case(52, M, K, batch=batch)
    pm = B.ap_pack(idx, {4: luts[4]})
    xd = torch.from_numpy(x).cuda()
    x3 = xd[:3].contiguous()
    side = torch.cuda.Stream()
    here = torch.cuda.current_stream().cuda_stream
    expect = [B.ap_gemm(pm, 4, xd), B.ap_gemv(pm, 4, x3), B.ap_dequantize(pm, 4)]
    assert all(_pool_stream(t.data_ptr()) == here for t in expect)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    for call, want in zip((lambda: B.ap_gemm(pm, 4, xd, stream=side), lambda: B.ap_gemv(pm, 4, x3, stream=side),
                           lambda: B.ap_dequantize(pm, 4, stream=side)), expect):
        out = call()
        assert _pool_stream(out.data_ptr()) == side.cuda_stream and torch.cuda.current_stream().cuda_stream == here
        # blocks of the sizes of work and out, overwritten on the current stream while the call may still run
        for n in (M * K * 2, out.numel() * 2):
            torch.empty(n, dtype=torch.uint8, device="cuda").fill_(0xff)
        side.synchronize()
        assert torch.equal(out, want)
        # the current stream still has work ahead of its use of out when out is released
        address, shape = out.data_ptr(), out.shape
        torch.cuda._sleep(20_000_000)
        kept = out.clone()
        del out
        with torch.cuda.stream(side):
            again = torch.empty(shape, dtype=torch.float16, device="cuda")
            assert again.data_ptr() != address
            again.fill_(-7.0)
        torch.cuda.synchronize()
        assert torch.equal(kept, want)
    # the workspace, released when ap_gemm returned, is among the named stream's blocks
    assert any(s["stream"] == side.cuda_stream and s["total_size"] >= M * K * 2 for s in torch.cuda.memory_snapshot())
    pm2 = B.ap_pack(idx, {4: luts[4]}, stream=side)
    assert _pool_stream(pm2.buf.data_ptr()) == side.cuda_stream
    assert torch.equal(B.ap_gemv(pm2, 4, x3), expect[1])
    # named and current the same stream, and a named default stream beside another current one
    with torch.cuda.stream(side):
        out = B.ap_gemv(pm, 4, x3, stream=side)
        assert _pool_stream(out.data_ptr()) == side.cuda_stream
        out2 = B.ap_gemv(pm, 4, x3, stream=torch.cuda.default_stream())
        assert _pool_stream(out2.data_ptr()) == here
    torch.cuda.synchronize()
    assert torch.equal(out, expect[1]) and torch.equal(out2, expect[1])
    pm.close()
    pm2.close()


def test_products_refuse_tensors_that_are_too_small(B, tiny):
    # the binding refuses, before any launch, what a kernel would read or write past its end; what holds enough is taken as before:
    # a longer vector x, a y of another type or shape or in pinned host memory, a y in the middle of a larger tensor
    import torch
    M, K, batch = 512, 512, 3
    idx, luts, x = inputs.make_case(1, M, K, batch=batch)
    pm = B.ap_pack(idx, {4: luts[4]})
    xd = torch.from_numpy(x).cuda()
    expect = B.ap_gemv(pm, 4, xd)
    for call in (B.ap_gemv, B.ap_gemm):
        for bad in (xd[:, :K - 32].contiguous(), torch.empty((batch, 0), dtype=torch.float16, device="cuda")):
            with pytest.raises(AssertionError):
                call(pm, 4, bad)
        base = torch.zeros((batch + 1) * M, dtype=torch.float16, device="cuda")
        for bad in (base[:batch * M - 1].clone(), base[M + 1:], torch.zeros((batch, M), dtype=torch.float16),
                    torch.zeros(batch * M, dtype=torch.uint8, device="cuda"), torch.zeros((batch, 0), dtype=torch.float16, device="cuda")):
            with pytest.raises(AssertionError):
                call(pm, 4, xd, y=bad)
        torch.cuda.synchronize()
        assert not base.any()
        call(pm, 4, xd, y=base[M:])
        assert torch.equal(base[M:].view(batch, M), expect) and not base[:M].any()
        ints = torch.zeros((M, batch), dtype=torch.int16, device="cuda")
        call(pm, 4, xd, y=ints)
        assert torch.equal(ints.view(torch.float16).view(batch, M), expect)
        pinned = torch.zeros((batch, M), dtype=torch.float16, pin_memory=True)
        call(pm, 4, xd, y=pinned)
        torch.cuda.synchronize()
        assert torch.equal(pinned, expect.cpu())
    with pytest.raises(AssertionError):
        B.ap_gemv(pm, 4, xd[0, :K - 1].clone())
    assert torch.equal(B.ap_gemv(pm, 4, xd.view(-1)), expect[:1])
    # a workspace that says it is larger than its memory
    work = torch.zeros(1, dtype=torch.uint8, device="cuda").expand(M * K * 2)
    for w in (work, torch.zeros(M * K * 2, dtype=torch.uint8)):
        with pytest.raises(B.ApError) as e:
            B.ap_gemm(pm, 4, xd, work=w)
        assert e.value.status == 5
    pm.close()


@pytest.mark.parametrize("batch", [3, 5, 8, 9, 13, 16])
def test_small_and_ragged_matrices_at_batches(B, batch):
    # calls that go to the tile kernel by size alone (few tiles, short rows, rows that end inside 128 or 256 columns) and their
    # neighbours that do not: both sides of the lines that the choice draws at 256, 1280, 2560 rows and 512, 2048, 4096 columns
    shapes = [(256, 32), (253, 512), (257, 2048), (260, 2080), (1277, 512), (1280, 1632), (1281, 4096), (1285, 4128), (2557, 2592),
              (2561, 2176)]
    for k, (M, K) in enumerate(shapes):
        idx, luts, x = inputs.make_case(41, M, K, batch=batch, salt=k)
        pm = B.ap_pack(idx, luts)
        rows = np.unique(np.r_[0:17, M // 2:M // 2 + 16, M - 17:M])
        for b in ALL_BITS:
            check_against_oracle(run_gemv(pm, b, x), idx, luts[b], b, x, rows=rows)
        pm.close()


def test_batch_2_on_the_tile_kernel_same_bits_in_lists_and_fused_launches(B):
    # b = 4 at batch 2 goes to the tile kernel from 2^27 weights on (the last three shapes: 4 and 8 waves, one and two tiles per workgroup);
    # list and fused launches of such matrices, among others that stay on the batch-1/2 kernel, give the bits of single calls
    import torch
    shapes = [(8192, 8192), (8192, 7936), (4096, 16384), (6150, 11008), (16384, 4096), (8205, 16640), (2050, 4096), (70, 2048 + 96),
              (16384, 8192), (12283, 11008), (8179, 16640)]
    mats = []
    for k, (M, K) in enumerate(shapes):
        idx, luts, x = inputs.make_case(42, M, K, batch=2, salt=k, bit_widths=[4, 5], sigma=0.01)
        mats.append((idx, luts, x, B.ap_pack(idx, luts), torch.from_numpy(x).cuda()))
    single = {}
    for k, (idx, luts, x, pm, xd) in enumerate(mats):
        rows = np.unique(np.r_[0:20, pm.M // 2:pm.M // 2 + 16, pm.M - 20:pm.M])
        for b in (4, 5):
            single[k, b] = y = B.ap_gemv(pm, b, xd)
            check_against_oracle(y.cpu().numpy(), idx, luts[b], b, x, rows=rows)
    picks = [(k, b) for b in (4, 5, 4) for k in range(len(mats))] + [(0, 4)] * 34   # more than one launch's worth
    out = [torch.full((2, mats[k][3].M), -5.0, dtype=torch.float16, device="cuda") for k, b in picks]
    B.ap_gemv_list_batch([(mats[k][3], b, mats[k][4], y) for (k, b), y in zip(picks, out)], 2)
    for (k, b), y in zip(picks, out):
        assert torch.equal(y.view(torch.int16), single[k, b].view(torch.int16)), (shapes[k], b)
    out = [torch.full((2, shapes[k][0]), -5.0, dtype=torch.float16, device="cuda") for k in range(len(mats))]
    for b in (4, 5):
        for group in ([4, 6], [0], [6], [8, 0], [8], [5, 10]):        # equal row length
            B.ap_gemv_multi([(mats[k][3], mats[k][4], out[k]) for k in group], b)
            for k in group:
                assert torch.equal(out[k].view(torch.int16), single[k, b].view(torch.int16)), (shapes[k], b)
    for m in mats:
        m[3].close()


@pytest.mark.parametrize("b", ALL_BITS)
def test_short_rows_in_list_and_fused_launches(B, b):
    # rows of 1, 2 and 3 pairs of octets, where a launch has waves without columns at b = 3, 4, 8; of 513 row groups and 129 tiles each: one (fewer
    # groups than a list or fused launch on tiles takes), and launches below, inside and above the 768..1024 tiles at b = 8
    import torch
    for K in (256, 768, 1280):
        idx, luts, x = inputs.make_case(43, 2050, K, batch=5, bit_widths=[b], sigma=0.01)
        pm, xd = B.ap_pack(idx, luts), torch.from_numpy(x).cuda()
        for count in (1, 4, 7, 8):
            out = [torch.full((5, pm.M), -5.0, dtype=torch.float16, device="cuda") for _ in range(2 * count)]
            B.ap_gemv_list_batch([(pm, b, xd, y) for y in out[:count]], 5)
            B.ap_gemv_multi([(pm, xd, y) for y in out[count:]], b)
            for y in (out[0], out[-1]):
                check_against_oracle(y.cpu().numpy(), idx, luts[b], b, x)
            for k in range(2 * count):
                first = out[0] if k < count else out[count]
                assert torch.equal(out[k].view(torch.int16), first.view(torch.int16))
                if count > 1:                                        # the same kernel and number of waves in both
                    assert torch.equal(out[k].view(torch.int16), out[0].view(torch.int16))
        pm.close()


@pytest.mark.parametrize("b", [5, 6, 7])
def test_short_and_long_rows_in_one_work_list(B, b):
    # the shortest row sets the waves of a list launch at these bit-widths (one of 256 columns: a single wave takes all columns of the others)
    import torch
    shapes = [(2050, 256), (4099, 4096), (515, 11008), (2050, 1280)]
    mats = []
    for k, (M, K) in enumerate(shapes):
        idx, luts, x = inputs.make_case(47, M, K, batch=4, salt=k, bit_widths=[b], sigma=0.01)
        mats.append((idx, luts, x, B.ap_pack(idx, luts), torch.from_numpy(x).cuda()))
    out = [torch.full((4, M), -5.0, dtype=torch.float16, device="cuda") for M, K in shapes]
    B.ap_gemv_list_batch([(m[3], b, m[4], y) for m, y in zip(mats, out)], 4)
    for (idx, luts, x, pm, xd), y in zip(mats, out):
        rows = np.unique(np.r_[0:20, pm.M - 20:pm.M])
        check_against_oracle(y.cpu().numpy(), idx, luts[b], b, x, rows=rows)
        pm.close()


@pytest.mark.parametrize("batch", [9, 16])
@pytest.mark.parametrize("M,K", [(250, 12288 + 256), (1029, 8192 + 64), (7190, 4352), (12305, 6144 + 96), (20481, 1792)])
def test_nine_to_sixteen_batch_rows_over_several_passes(B, M, K, batch):
    # waves that load activations again for a second, third and later octet: even and odd numbers of octets, ragged last ones, one tile per
    # workgroup and (from 449 tiles on) two
    idx, luts, x = inputs.make_case(46, M, K, batch=batch, sigma=0.01)
    pm = B.ap_pack(idx, luts)
    rows = np.unique(np.r_[0:20, M // 2:M // 2 + 16, M - 20:M])
    for b in ALL_BITS:
        check_against_oracle(run_gemv(pm, b, x), idx, luts[b], b, x, rows=rows)
    pm.close()
