"""Wait states around inline assembly in the device helpers: the compiler does not look into inline assembly, so what it would keep apart
itself is kept apart there by hand.  Small kernels are compiled for gfx950 and their instructions read; no GPU is used."""
import os
import re
import shutil
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


def registers(operand, kind="v"):
    m = re.match(r"%s\[(\d+):(\d+)\]|%s(\d+)\b" % (kind, kind), operand.strip())
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


# O between two matrix products, multiplied by a transcendental result: with nothing else in the way that keeps them apart.
SCALE = """
extern "C" __global__ void probe(float *out, const bf16x8 *a, const bf16x8 *b, float x)
{
    f32x16 o[%(blocks)d];
    bf16x8 va[%(blocks)d];
    const bf16x8 vb = b[threadIdx.x];
    const float y = __builtin_amdgcn_exp2f(x + threadIdx.x);
    for (int i = 0; i < %(blocks)d; ++i) {
        for (int v = 0; v < 16; ++v) o[i][v] = 0.f;
        va[i] = a[i * 64 + threadIdx.x];
        o[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[i], vb, o[i], 0, 0, 0);
    }
    %(scale)s;
    for (int i = 0; i < %(blocks)d; ++i) o[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vb, va[i], o[i], 0, 0, 0);
    for (int i = 0; i < %(blocks)d; ++i)
        for (int v = 0; v < 16; ++v) out[(i * 16 + v) * 64 + threadIdx.x] = o[i][v];
}
"""


def waits_around_scaling(code):
    """The fewest wait states from a product to a multiplication of its result, from a multiplication to a product that adds to its
    result, and from the exponential to a multiplication by it."""
    states, product, scaled, exponential = 0, {}, {}, {}
    least = {}

    def note(what, since, reg):
        if reg in since:
            least[what] = min(least.get(what, 1 << 30), states - since[reg] - 1)

    for op, text in code:
        operands = text.split(",")
        states += int(text) + 1 if op == "s_nop" else 1
        if op.startswith("v_mfma"):
            for reg in registers(operands[3]):
                note("multiplied, product", scaled, reg)
            for reg in registers(operands[0]):
                product[reg] = states
                scaled.pop(reg, None)
        elif op.startswith("v_mul_f32"):
            to, = registers(operands[0])
            for source in operands[1:]:
                for reg in registers(source):
                    note("product, multiplied", product, reg)
                    note("exponential, multiplied", exponential, reg)
            scaled[to] = states
            product.pop(to, None)
        elif op.startswith("v_exp_f32"):
            exponential[next(iter(registers(operands[0])))] = states
    return least


@pytest.mark.parametrize("blocks", [2, 4])
def test_scaling_in_place_waits_as_long_as_the_compiler_does(tmp_path, blocks):
    own = "for (int i = 0; i < %d; ++i) for (int v = 0; v < 16; ++v) o[i][v] *= y" % blocks
    want, got = (waits_around_scaling(instructions(tmp_path, SCALE % {"blocks": blocks, "scale": scale}, "probe"))
                 for scale in (own, "scale_in_place(o, y)"))
    assert set(want) == set(got) == {"product, multiplied", "multiplied, product", "exponential, multiplied"}
    assert want["product, multiplied"] > 0               # (the hazard is there)
    assert got["product, multiplied"] >= want["product, multiplied"] and got["multiplied, product"] >= want["multiplied, product"], (want, got)
    assert got["exponential, multiplied"] >= 1           # (one wait state; the compiler's own code has the products in between)


# A load to LDS from a base that the instruction before has written to scalar registers: its address comes from there.
LOAD = """
extern "C" __global__ void probe(uint32_t *out, const uint64_t *bases)
{
    __shared__ __attribute__((aligned(1024))) char lds[4096];
    const uint64_t v = bases[threadIdx.x];
    const uint32_t t = threadIdx.x * 16, off[4] = {t, t + 16, t + 32, t + 48}, off2[2] = {t, t + 16}, off1[1] = {t};
    %(load)s;
    wait_vm<0>();
    out[threadIdx.x] = reinterpret_cast<uint32_t *>(lds)[threadIdx.x] + off[3] + off2[1] + off1[0];
}
"""
OWN_LOAD = """const char *base = (const char *)uniform_ptr((const void *)v);
    out[threadIdx.x + 64] = *(__attribute__((address_space(1))) const uint32_t *)((uintptr_t)base + t)"""
LOADS = {
    "four": "dma16_group4((const void *)v, off[0], off[1], off[2], off[3], lds_address(lds))",
    "two": "dma16_group2((const void *)v, off[0], off[1], lds_address(lds))",
    "stream-four": "dma16_stream((const void *)v, off, lds_address(lds))",
    "stream-two": "dma16_stream((const void *)v, off2, lds_address(lds))",
    "stream-one": "dma16_stream((const void *)v, off1, lds_address(lds))",
}


def waits_behind_scalar_writes(code):
    """The fewest wait states from a vector instruction that writes a scalar register to a memory instruction that reads it."""
    states, written, least = 0, {}, 1 << 30
    for op, text in code:
        operands = text.split(",")
        states += int(text, 0) + 1 if op == "s_nop" else 1
        if op.startswith(("global_", "buffer_", "flat_", "scratch_")):
            for reg in set().union(*(registers(x, "s") for x in operands)) & set(written):
                least = min(least, states - written[reg] - 1)
        elif op.startswith("v_"):
            to = operands[:1] if op.startswith(("v_readfirstlane", "v_readlane", "v_cmp")) else operands[1:2] if re.match(r"v_\w+_co_|v_mad_[ui]64|v_div_scale", op) else []
            for reg in set().union(*(registers(x, "s") for x in to)):
                written[reg] = states
        elif op.startswith("s_") and operands[0]:
            for reg in registers(operands[0], "s"):
                written.pop(reg, None)
    return least


@pytest.mark.parametrize("name", sorted(LOADS))
def test_scalar_bases_are_waited_for_as_long_as_in_front_of_an_ordinary_load(tmp_path, name):
    want, got = (waits_behind_scalar_writes(instructions(tmp_path, LOAD % {"load": load}, "probe")) for load in (OWN_LOAD, LOADS[name]))
    assert 0 < want <= got < 1 << 30                     # (the hazard is there)


def test_built_kernels_keep_them_apart(tmp_path):
    """The same in the library as built, all kernels (the shared-tile kernels multiply O in place in a block of its own, by instructions of
    their own): 11 wait states from a product to a multiplication of its result, one from there to a product that adds to it, two from
    a store of more than 8 bytes to a write to its data, five from a vector instruction that writes a scalar register (spilled ones come
    back by such) to a load that takes its address from there; the compiler's own are the same."""
    if not os.path.exists(build.LIB):
        build.build()
    lib = tmp_path / "lib.so"
    shutil.copyfile(build.LIB, lib)
    objdump = os.path.join(os.path.dirname(os.path.realpath(build.hipcc())), "..", "lib", "llvm", "bin", "llvm-objdump")
    subprocess.run([objdump, "--offloading", str(lib)], check=True, capture_output=True)
    kernels = multiplied = 0
    for part in sorted(tmp_path.glob("lib.so.*gfx950")):
        text = subprocess.run([objdump, "-d", "--mcpu=gfx950", str(part)], check=True, capture_output=True, text=True).stdout
        for body in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
            name, lines = body.split(">:", 1)
            code = [l.split("//")[0].split(None, 1) for l in lines.split("\n") if l.startswith("\t")]
            code = [(x[0], x[1].strip() if len(x) > 1 else "") for x in code]
            least = waits_around_scaling(code)
            assert waits_behind_scalar_writes(code) >= 5, name
            kernels += 1
            multiplied += "product, multiplied" in least
            assert least.get("product, multiplied", 11) >= 11 and least.get("multiplied, product", 1) >= 1, (name, least)
            for i, (op, operands) in enumerate(code):
                if re.match(r"(global|flat|buffer)_store_dwordx[34]", op):
                    data, waits = registers(operands.split(",")[1 if op[0] != "b" else 0]), 0
                    for other, text_ in code[i + 1:i + 3]:
                        if waits < 2 and other.startswith("v_"):
                            assert not registers(text_.split(",")[0]) & data, (name, op, operands, other, text_)
                        waits += int(text_, 0) + 1 if other == "s_nop" else 1
    assert kernels > 20 and multiplied > 10
