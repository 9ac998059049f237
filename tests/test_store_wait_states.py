"""What the compiler makes of write_out, a 16-byte store through the L2, where the stored registers are overwritten right behind it.

On gfx950 a vector instruction that overwrites the data of a store of more than 8 bytes has to stay two wait states behind the store; the
compiler sees to that where it knows the store.  Compiled here from the kernels' own header; nothing runs."""
import os
import re
import subprocess

from paper_1901_01965_amd import build

SOURCE = """
#include "kernel_common.h"
using namespace wg;
__global__ void overwritten(v4i* at) {
    v4i v = at[threadIdx.x];
    write_out(at + threadIdx.x + 64, v);
    v += 7;
    write_out(at + threadIdx.x + 128, v);
    v ^= 7;
    write_out(at + threadIdx.x + 192, v);
}
"""


def _registers(operand):
    wide = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    if wide:
        return set(range(int(wide.group(1)), int(wide.group(2)) + 1))
    one = re.fullmatch(r"v(\d+)", operand)
    return {int(one.group(1))} if one else set()


def _overwritten_early(body):
    """(store, instruction) where the data of a 16-byte store is overwritten less than two wait states behind it."""
    found = []
    for i, op in enumerate(body):
        if not re.match(r"(global|flat)_store_dwordx4 ", op):
            continue
        data, states = _registers(re.split(r"[,\s]+", op)[2].rstrip(",")), 0
        for behind in body[i + 1:]:
            if states >= 2:
                break
            name, _, rest = behind.partition(" ")
            if name == "s_nop":
                states += int(rest, 0) + 1
                continue
            if name.startswith("v_") and _registers(rest.split(",")[0].strip()) & data:
                found.append((op, behind))
                break
            states += 1
    return found


def _bodies(assembly):
    bodies, body = [], None
    for line in assembly.splitlines():
        text = line.split(";")[0].strip()
        if re.match(r"_Z\w+:", line):
            body = []
            bodies.append(body)
        elif body is not None and re.match(r"[a-z]+_", text):
            body.append(text)
    return bodies


def test_a_short_wait_is_found():
    store, add = "global_store_dwordx4 v[6:7], v[2:5], off sc1", "v_add_u32_e32 v4, 1, v4"
    assert _overwritten_early([store, "s_nop 0", add]) == [(store, add)]
    assert _overwritten_early([store, "v_mov_b32_e32 v9, 0", add]) == [(store, add)]
    assert _overwritten_early([store, "s_nop 1", add]) == _overwritten_early([store, "s_nop 0", "v_add_u32_e32 v1, 1, v1", add]) == []


def test_data_of_a_store_through_the_l2_stays_two_wait_states(tmp_path):
    source = tmp_path / "overwrite.hip"
    source.write_text(SOURCE)
    out = tmp_path / "overwrite.s"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.HIPCC_FLAGS +
                   ["-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "-S", "--cuda-device-only", str(source), "-o", str(out)],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    bodies = [b for b in _bodies(out.read_text()) if any("store_dwordx4" in op for op in b)]
    assert len(bodies) == 1
    stores = [op for op in bodies[0] if "store_dwordx4" in op]
    assert len(stores) == 3 and all(op.endswith("sc1") for op in stores)
    assert len({op.split(", ")[1] for op in stores}) == 1   # the same registers, or nothing is overwritten
    assert _overwritten_early(bodies[0]) == []
