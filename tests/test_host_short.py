"""The launch that the host makes of a chunk for the kernel of chunks with little work: every step of every row block once, by
teams of every size, with the keys split or not (tests/host_short.cpp)."""
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


def test_packed_words(driver):
    """The words that a launch's shape travels in, at the smallest and largest of every field (those of a drawn launch: test_teams)."""
    res = subprocess.run([driver], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and int(res.stdout.split()[0]) > 10000, res.stdout + res.stderr


# teams: log2 of the team sizes that the drawn launches have to show
@pytest.mark.parametrize("heads, dim, chunk, teams", [((40, 40), 128, 512, (0, 1, 2, 3)), ((40, 40), 64, 2048, (0, 1, 2)), ((32, 8), 128, 512, (0, 1, 2, 3)),
                                                      ((24, 8), 128, 500, (0, 1, 2)), ((6, 3), 64, 500, (0, 1, 3)), ((4, 4), 128, 4096, (0, 1, 2)),
                                                      ((2, 1), 128, 64, (3,)), ((32, 8), 128, 1, (3,))])
def test_teams(driver, heads, dim, chunk, teams):
    res = subprocess.run([driver, "19", "300", str(heads[0]), str(heads[1]), str(dim), str(chunk)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
    nums = [int(x.rstrip(",")) for x in res.stdout.split() if x.rstrip(",").isdigit()]
    assert nums[0] >= 200 and all(nums[1 + t] > 0 for t in teams), res.stdout
    assert nums[5] > 0 or heads[0] * -(-chunk // 32) > 128, res.stdout
    assert chunk < 4096 or nums[6] > 120, res.stdout                   # (row blocks: up to 128 of them)
    assert heads != (2, 1) or nums[7] == 16, res.stdout                # (parts of a row block's keys: up to 16)
