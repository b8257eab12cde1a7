"""Wait states around inline assembly in the device helpers: the compiler does not look into inline assembly, so what it would keep apart
itself is kept apart there by hand.  Small kernels are compiled for gfx950 and their instructions read; no GPU is used."""
import os
import re
import subprocess

import pytest

from paper_2401_11181_amd import build

PRELUDE = '#include <hip/hip_runtime.h>\n#include "attn_common.h"\nusing namespace tetri_dev;\n'


def instructions(tmp_path, source, kernel):
    """The kernel's instructions in order, as (name, operands)."""
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PRELUDE + source)
    subprocess.run([build.hipcc(), "-x", "hip", "-S", "--cuda-device-only", "-w", str(src), "-o", str(out), "-I", os.path.join(build.ROOT, "include"),
                    "-I", build.CSRC] + build.HIP_FLAGS, check=True, capture_output=True)
    body = re.search(r"^%s:(.*?)s_endpgm" % kernel, out.read_text(), re.S | re.M).group(1)
    lines = (l.split(";")[0].split("//")[0].strip() for l in body.split("\n"))
    return [(l.split()[0], l[len(l.split()[0]):].strip()) for l in lines if l and not l.startswith(".") and not l.endswith(":")]


def registers(operand):
    m = re.match(r"v\[(\d+):(\d+)\]|v(\d+)", operand.strip())
    if not m:
        return set()
    return {int(m.group(3))} if m.group(3) else set(range(int(m.group(1)), int(m.group(2)) + 1))


# A value is stored and its registers are written to right away, as a loop over rows may do.
STORE = """
extern "C" __global__ void probe(%(type)s *to, const %(type)s *from, uint32_t x)
{
    %(pointer)s p = (%(pointer)s)(uintptr_t)(to + threadIdx.x);
    %(type)s v = from[threadIdx.x];
    v ^= 1u;
    %(store)s;
    v += x;
    ((global_u32x4_w *)(uintptr_t)(to + 1024))[threadIdx.x] = __builtin_bit_cast(u32x4, v);
}
"""
STORES = {
    "coherent": ("u32x4", "global_u32x4_w *", "store_coherent(p, v)"),
    "coherent-floats": ("u32x4", "f32x4 *", "store_coherent(p, __builtin_bit_cast(f32x4, v))"),
    "past-caches": ("u32x4", "global_u32x4_w *", "store_past_caches(p, v)"),
}


def wait_behind_store(code):
    """Wait states between the first store and the first instruction that writes to its data."""
    at = next(i for i, (op, _) in enumerate(code) if op.startswith("global_store"))
    operands = code[at][1].split(",")
    data, waits = registers(operands[1]), 0
    for op, text in code[at + 1:]:
        if op == "s_nop":
            waits += int(text) + 1
        elif op.startswith("v_") and registers(text.split(",")[0]) & data:
            return waits
        else:
            waits += 1
    raise AssertionError("nothing writes to the stored registers")


@pytest.mark.parametrize("name", sorted(STORES))
def test_stored_registers_are_left_alone_as_long_as_behind_an_ordinary_store(tmp_path, name):
    kind, pointer, store = STORES[name]
    own = wait_behind_store(instructions(tmp_path, STORE % {"type": kind, "pointer": "global_u32x4_w *", "store": "*p = v"}, "probe"))
    assert own > 0                                       # (the hazard is there)
    assert wait_behind_store(instructions(tmp_path, STORE % {"type": kind, "pointer": pointer, "store": store}, "probe")) >= own


def test_no_store_is_written_out_elsewhere():
    for name in sorted(os.listdir(build.CSRC)):
        if name.endswith((".hip", ".h")) and name != "attn_common.h":
            with open(os.path.join(build.CSRC, name)) as f:
                assert not re.search(r'"[^"]*\b(global|flat|buffer)_store', f.read()), name
