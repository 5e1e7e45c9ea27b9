"""How a product is divided on the fused large-batch kernel (csrc/kernels.h: fused_plan), on the CPU."""
import collections
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
STATIC_BYTES = 32 << 20                       # scratch of ap_gemm_static
Plan = collections.namedtuple("Plan", "taken ntiles nj blocks waves steps parts copy_bytes")
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


def test_plans_that_the_gpu_tests_name(plans):
    # the shapes of the GPU tests reach the paths that they are there for
    from test_gpu_large_batch import ALL_BITS, COPIED_X, PASSES_OF_HALF_THE_ROWS
    from test_zz_no_alloc import SEQUENCE
    for M, K, batch, parts in COPIED_X:
        for work in (M * K * 2, STATIC_BYTES):
            for p in plans([(M, K, b, batch, work) for b in ALL_BITS]):
                assert p.taken and p.nj == 4 and p.waves == 8 and p.copy_bytes > 0 and p.parts == parts, (M, K, batch, work, p)
    for M, K, batch, bits in PASSES_OF_HALF_THE_ROWS:
        for p, half in zip(plans([(M, K, b, batch, STATIC_BYTES) for b in bits]), plans([(M, K, b, batch // 2, STATIC_BYTES) for b in bits])):
            assert not p.taken and p.copy_bytes > STATIC_BYTES and half.taken, (M, K, batch, p, half)
    for (M, K, batch), bits, keeps in SEQUENCE:
        for p in plans([(M, K, b, batch, STATIC_BYTES) for b in bits]):
            assert p.taken
            if keeps:
                assert (p.copy_bytes > 0, p.parts > 1) == ("copy" in keeps, "parts" in keeps), (M, K, batch, keeps, p)
