"""Which kernel a chunk whose segments the host knows goes to, on both sides of the lines of the rule (tests/host_short.cpp): "short" (the
kernel for chunks with little work), "four" or "eight" (the shared-tile kernel on the host's division, 4 or 8 slots to a
workgroup), "self" (the launch that divides itself)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(HIP_INCLUDE, "hip")),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("short") / "host_short")
    csrc = os.path.join(ROOT, "paper_2401_11181_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-static-libasan", "-static-libubsan", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-I", HIP_INCLUDE,
                    "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(ROOT, "tests", "host_short.cpp"),
                    os.path.join(csrc, "tetri_host.cpp"), os.path.join(csrc, "tetri_plan.cpp"), "-o", exe], check=True)
    return exe


# heads, kv heads, FP8, segments (rows, cached tokens), kernel; 256 compute units
CHOICES = [
    # fewer row blocks than compute units, one workgroup to each: 16 steps on a wavefront, over codes 12
    (40, 40, 0, [(128, 3900)], "short"), (40, 40, 0, [(128, 4000)], "four"), (40, 40, 1, [(100, 2900)], "short"), (40, 40, 1, [(100, 3000)], "four"),
    # two: 20, 15
    (32, 8, 0, [(128, 10000)], "short"), (32, 8, 0, [(128, 10300)], "four"), (8, 2, 1, [(512, 7100)], "short"), (8, 2, 1, [(512, 7300)], "four"),
    # more: 128
    (32, 8, 0, [(64, 32000)], "short"), (8, 2, 1, [(128, 32500)], "short"),
    # more row blocks than compute units, not two each
    (40, 40, 0, [(256, 1700)], "short"), (40, 40, 0, [(256, 2100)], "four"), (40, 40, 1, [(256, 700)], "short"), (40, 40, 1, [(256, 1100)], "four"),
    # even work over several segments; uneven work
    (32, 8, 1, [(300, 1000), (212, 200)], "short"), (32, 8, 1, [(36, 1191), (476, 0)], "four"), (40, 40, 1, [(200, 2000), (312, 600)], "short"),
    (32, 8, 1, [(200, 2000), (312, 600)], "four"),
    # the longest wavefront as laid out: 16 steps, 24, 29
    (40, 40, 0, [(1024, 0)], "short"), (16, 16, 0, [(1235, 0), (139, 0), (1196, 0), (258, 657), (17, 90)], "four"),
    (32, 8, 0, [(538, 0), (591, 32), (45, 158), (505, 729)], "four"),
    # row tiles and helpers that fill the chip; not even, not filling, too long
    (40, 40, 1, [(512, 1000)], "self"), (40, 40, 0, [(100, 3000), (412, 0)], "four"), (40, 40, 0, [(384, 3000)], "four"), (40, 40, 0, [(512, 2560)], "eight"),
    # ... over 16-bit rows, or with more than four tiles to a head
    (40, 40, 0, [(512, 1000)], "four"), (24, 8, 1, [(896, 1000)], "four"), (20, 20, 0, [(1024, 1000)], "four"), (12, 12, 1, [(1792, 600)], "four"),
    # 4 or 8 slots
    (40, 40, 0, [(512, 6144)], "eight"), (24, 8, 0, [(512, 4000)], "four"), (16, 16, 0, [(1024, 2560)], "short"), (16, 16, 0, [(1024, 4200)], "eight"),
    (32, 8, 0, [(2048, 300)], "eight"),
    # more short tiles than compute units: nothing to balance; one long context; one that is long beside few
    (32, 8, 0, [(102, 0)] * 40, "self"), (32, 8, 1, [(102, 512)] + [(102, 0)] * 39, "self"), (32, 8, 0, [(102, 641)] + [(102, 0)] * 39, "self"),
    (32, 8, 0, [(102, 1000)] + [(102, 0)] * 39, "four"), (32, 8, 0, [(102, 641)] + [(102, 0)] * 30, "four"), (16, 16, 0, [(103, 0)] * 40, "self"),
    # 35 tiles of 8 slots, all long, for 32 workgroups
    (40, 40, 1, [(609, 11542), (752, 63), (210, 251), (75, 4326), (779, 11722), (134, 241), (477, 143)], "four"),
]


# Over codes: one segment with more than two row blocks to a compute unit (30000 steps in all, 22 on a wavefront); between one and two (17 steps
# times the part of the two)
CODES = [
    (40, 40, 1, [(512, 896)], "short"), (40, 40, 1, [(512, 897)], "self"), (32, 8, 1, [(1024, 384)], "short"), (32, 8, 1, [(1024, 385)], "eight"),
    (40, 40, 1, [(1024, 192)], "short"), (40, 40, 1, [(1024, 193)], "four"), (40, 40, 1, [(412, 0), (100, 1500)], "four"),
    (40, 40, 1, [(256, 1024)], "short"), (40, 40, 1, [(384, 1200)], "short"), (40, 40, 1, [(384, 1700)], "four"), (32, 8, 1, [(480, 1300)], "short"),
]


def test_choice_over_codes(driver):
    check(driver, CODES)


def test_choice(driver):
    check(driver, CHOICES)


def check(driver, CHOICES):
    for heads in sorted({c[:2] for c in CHOICES}):
        cases = [c for c in CHOICES if c[:2] == heads]
        text = "".join("%d %d %s\n" % (c[2], len(c[3]), " ".join("%d %d" % s for s in c[3])) for c in cases)
        res = subprocess.run([driver, str(heads[0]), str(heads[1])], input=text, capture_output=True, text=True, timeout=60)
        assert res.returncode == 0, res.stderr
        assert list(zip([c[2:4] for c in cases], res.stdout.split())) == [(c[2:4], c[4]) for c in cases]
