"""How a product is divided on the fused large-batch kernel, and which products run there (csrc/kernels.h), on the CPU."""
import collections
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
STATIC_BYTES = 32 << 20                       # scratch of ap_gemm_static
Plan = collections.namedtuple("Plan", "taken ntiles nj blocks waves steps parts copy_bytes gemm_pays static_dense")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """[(M, K, b, batch, work_bytes), ...] -> [Plan, ...]"""
    exe = str(tmp_path_factory.mktemp("plan") / "fused_plan")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"),
                           os.path.join(ROOT, "tests", "host", "fused_plan.cpp"), "-o", exe])

    def ask(products):
        text = "".join("%d %d %d %d %d\n" % p for p in products)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")[:-1]
        assert len(out) == len(products)
        return [Plan(*map(int, line.split())) for line in out]
    return ask


def test_copy_of_x_is_decided_for_the_parts_that_fit(plans):
    # the steps of a wave without a copy of x stay within what the copy was measured against, also where the scratch holds fewer
    # parts than wanted; copy and partial sums lie within the scratch
    rng = random.Random(3)
    products = [(64, 1952, 3, 492, 64 * 1952 * 2)]
    while len(products) < 20000:
        M, K = round(16 * 1800 ** rng.random()), round(900 ** rng.random()) * 32
        work = rng.choice([M * K * 2, M * K * 2 + rng.randrange(1 << 22), STATIC_BYTES])
        products.append((M, K, rng.randint(3, 8), rng.randint(1, 1024), work))
    for (M, K, b, batch, work), p in zip(products, plans(products)):
        what = (M, K, b, batch, work, p)
        assert p.parts >= 1 and p.ntiles * p.nj * 16 >= batch and p.blocks * 64 >= M, what
        if not p.taken:
            assert p.copy_bytes > work, what
            continue
        assert p.copy_bytes + (batch * M * 4 * p.parts if p.parts > 1 else 0) <= work, what
        if p.nj == 4 and p.copy_bytes == 0:
            assert p.steps <= (1 if b == 8 else 2) * p.waves * p.parts, what


@pytest.mark.parametrize("M,K,b,batch,fused", [
    # small products are ahead on the fused kernel, which needs no copy of x for them
    (512, 256, 8, 256, True), (256, 416, 7, 64, True), (1024, 32, 4, 192, True), (2048, 32, 8, 160, True), (512, 1056, 8, 128, True),
    (512, 1056, 7, 128, True), (300, 3072, 8, 192, True), (512, 4096, 8, 128, True), (64, 8192, 8, 64, True),
    # but not with a copy of x and unevenly divided steps, nor without room for the partial sums
    (300, 2304, 8, 64, False), (300, 2816, 8, 192, False), (256, 3584, 8, 192, False), (300, 2816, 7, 192, True),
    (64, 5632, 8, 64, False), (256, 13824, 8, 256, False), (400, 16384, 5, 384, False), (400, 16384, 5, 320, True)])
def test_route_of_gemm_with_the_smallest_workspace(plans, M, K, b, batch, fused):
    p, = plans([(M, K, b, batch, M * K * 2)])
    assert (p.taken and p.gemm_pays) == fused, p


@pytest.mark.parametrize("M,K,b,batch,dense", [
    (300, 256, 8, 128, False), (300, 256, 3, 128, False), (300, 512, 8, 512, False), (1024, 256, 5, 512, False), (64, 96, 5, 200, False),
    (64, 96, 8, 200, True), (64, 160, 8, 200, False), (64, 32, 3, 200, True), (300, 32, 7, 500, True), (1024, 32, 8, 200, True),
    (1024, 32, 8, 1500, False), (1024, 32, 5, 200, False), (8, 128, 8, 200, True), (64, 32, 8, 48, False)])
def test_route_of_static_gemm(plans, M, K, b, batch, dense):
    p, = plans([(M, K, b, batch, STATIC_BYTES)])
    assert p.static_dense == dense, p


def test_plans_that_the_gpu_tests_name(plans):
    # the shapes of the GPU tests reach the paths that they are there for
    from test_gpu_large_batch import ALL_BITS, COPIED_X, DENSE_EDGES, PASSES_OF_HALF_THE_ROWS
    from test_zz_no_alloc import SEQUENCE
    for M, K, batch, parts in COPIED_X:
        for work in (M * K * 2, STATIC_BYTES):
            for p in plans([(M, K, b, batch, work) for b in ALL_BITS]):
                assert p.taken and p.nj == 4 and p.waves == 8 and p.copy_bytes > 0 and p.parts == parts, (M, K, batch, work, p)
    for M, K, batch, bits in DENSE_EDGES:
        for p, past in zip(plans([(M, K, b, batch, STATIC_BYTES) for b in bits]), plans([(M, K + 32, b, batch, STATIC_BYTES) for b in bits])):
            assert p.static_dense and not past.static_dense, (M, K, batch, p, past)
    for M, K, batch, bits in PASSES_OF_HALF_THE_ROWS:
        for p, half in zip(plans([(M, K, b, batch, STATIC_BYTES) for b in bits]), plans([(M, K, b, batch // 2, STATIC_BYTES) for b in bits])):
            assert not p.taken and p.copy_bytes > STATIC_BYTES and half.taken, (M, K, batch, p, half)
    for (M, K, batch), bits, keeps in SEQUENCE:
        for p in plans([(M, K, b, batch, STATIC_BYTES) for b in bits]):
            assert p.taken and p.static_dense == (keeps == "dense")
            if keeps and keeps != "dense":
                assert (p.copy_bytes > 0, p.parts > 1) == ("copy" in keeps, "parts" in keeps), (M, K, batch, keeps, p)
