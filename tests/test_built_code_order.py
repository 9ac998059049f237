"""The order of memory requests in the built limb-pair kernels, read from the library's own listing.

A wave asks for the next channel block's patch (16-byte transfers into LDS) and then for filter fragments, and later waits until
only as many requests are in flight as there are fragments younger than the patch.  A fragment requested before the transfers
would make that wait end early, and the transform read a patch that has not arrived: no result says so reliably."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1901_01965_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _kernels(listing):
    """name -> instructions, of a disassembly."""
    kernels, body = {}, None
    for line in listing.splitlines():
        head = re.match(r"[0-9a-f]+ <(.+)>:$", line)
        if head:
            body = kernels.setdefault(head.group(1), [])
        elif body is not None and line.strip():
            body.append(line.split("//")[0].strip())
    return kernels


def _transfers(body):
    return [i for i, op in enumerate(body) if op.startswith("buffer_load") and op.endswith(" lds")]


def _fragments_ahead_of_a_patch(body):
    """Requests between a barrier and the transfers into LDS that follow it."""
    early = []
    for i in _transfers(body):
        for op in reversed(body[:i]):
            if op.startswith("s_barrier") or (op.startswith("buffer_load") and op.endswith(" lds")):
                break
            if op.startswith(("buffer_load", "global_load", "flat_load")):
                early.append(op)
    return early


def test_a_listing_with_a_fragment_ahead_is_found():
    loop = ["s_barrier", "s_cbranch_scc1 4", "buffer_load_dwordx4 v2, s[24:27], s4 offen lds", "buffer_load_dwordx4 v[4:7], v3, s[20:23], s79 offen",
            "s_waitcnt vmcnt(6)", "s_barrier"]
    assert _fragments_ahead_of_a_patch(loop) == []
    loop[1], loop[2], loop[3] = loop[3], loop[1], loop[2]
    assert _fragments_ahead_of_a_patch(loop) == ["buffer_load_dwordx4 v[4:7], v3, s[20:23], s79 offen"]


def test_patches_are_requested_ahead_of_the_fragments_that_the_wait_counts(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    if not os.path.exists(build.LIB_PATH):
        build.build()
    library = shutil.copy(build.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", library], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    checked = 0
    for image in sorted(tmp_path.glob("*gfx950")):
        if b"lossless_pair_sums_kernel" not in image.read_bytes():
            continue
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--demangle", str(image)], check=True, stdout=subprocess.PIPE, text=True).stdout
        for name, body in _kernels(listing).items():
            if "lossless_pair" in name and _transfers(body):
                checked += 1
                assert _fragments_ahead_of_a_patch(body) == [], name
    # split channels in halves and quarters; not split, both again, int32 and int8 outputs
    assert checked == 6
