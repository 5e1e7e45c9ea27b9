"""What fused launches and work lists send to the device (csrc/api.cpp), on the CPU: the kernel launchers only note what they are given."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2402_10517_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")),
                                reason="needs g++ and the HIP headers")
LAYER_13B = [(5120, 5120)] * 4 + [(13824, 5120)] * 2 + [(5120, 13824)]


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """(kind, batch, [(M, K, b), ...]) -> (["kernel:items", ...], whether unused items of lists were zero)"""
    exe = str(tmp_path_factory.mktemp("launches") / "launches")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"),
                           os.path.join(ROOT, "tests", "host", "launches.cpp"), os.path.join(CSRC, "api.cpp"), os.path.join(CSRC, "pack.cpp"),
                           "-L" + os.path.join(ROCM, "lib"), "-lamdhip64", "-Wl,-rpath," + os.path.join(ROCM, "lib"), "-lpthread", "-o", exe])

    def ask(kind, batch, items):
        text = "%s %d %d\n%s" % (kind, batch, len(items), "".join("%d %d %d\n" % it for it in items))
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()
        return out[:-1], out[-1] == "clean"
    return ask


def at(b, shapes):
    return [(M, K, b) for M, K in shapes]


@pytest.mark.parametrize("shapes", [[(8192, 8192), (1024, 8192), (1024, 8192)], [(8192, 8192), (4096, 8192)], [(4096, 16384), (1024, 16384)],
                                    [(13824, 5120), (13824, 5120)], [(5120, 5120)] * 3, [(8704, 16384), (1024, 16384)]])
def test_projections_that_share_their_input_are_one_launch(launches, shapes):
    # at batch 2 and 4 bits a further launch for the large matrices alone made these 3 to 19 % slower
    for b in (4, 5):
        for batch in (2, 3, 8):
            assert len(launches("fused", batch, at(b, shapes))[0]) == 1, (shapes, b, batch)


def test_batch_2_in_a_launch_of_its_own_only_where_that_pays(launches):
    # of 2^27 weights and more, evenly spread over the CUs
    assert launches("fused", 2, at(4, [(28672, 8192)] * 2))[0] == ["tile_list:2"]
    assert sorted(launches("fused", 2, at(4, [(28672, 8192), (1024, 8192)]))[0]) == ["alu_list:1", "tile_list:1"]
    assert launches("fused", 2, at(5, [(28672, 8192)] * 2))[0] == ["alu_fused:2"]


def test_work_lists_at_batch_2(launches):
    for bits in ([4] * 7, [3, 4, 5, 4, 4, 6, 4], [5, 5, 5, 3, 4, 6, 5]):
        items = [(M, K, b) for (M, K), b in zip(LAYER_13B, bits)]
        assert launches("list", 2, items)[0] == ["alu_list:7"], bits
    assert launches("list", 2, at(4, LAYER_13B) * 6)[0] == ["alu_list:32", "alu_list:10"]
    layer = [(8192, 8192)] * 2 + [(1024, 8192)] * 2 + [(28672, 8192)] * 2 + [(8192, 28672)]
    assert sorted(launches("list", 2, at(4, layer))[0]) == ["alu_list:4", "tile_list:1", "tile_list:2"]


@pytest.mark.parametrize("batch", [1, 2, 3])
def test_unused_items_of_a_work_list_are_zero(launches, batch):
    # a list goes to the device whole, as the argument of the kernel
    items = at(4, [(4096, 4096), (1024, 4096), (28672, 8192), (8192, 28672)])
    for kind in ("list", "fused") if batch == 2 else ("list",):
        out, clean = launches(kind, batch, items[:3] if kind == "list" else items[2:3])
        assert clean, (kind, out)
