"""What the compiler made of the attention kernels, read from the code objects of the built library.

The decode worker counts the loads it has in flight and the prefill loop has no room to wait for reloads, so
spilled registers cost more than the values they hold: no kernel may have any scratch memory, except the two of the
prefill-heavy configuration, which are held to fewer registers than they ask for on purpose.
"""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2410_18038_amd import pod

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob: bytes):
    """The gfx950 code objects of every offload bundle in the library (one bundle per translation unit)."""
    at = blob.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, len_id = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + len_id]
            p += 24 + len_id
            if b"gfx950" in triple and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(MAGIC, p)


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_attention_kernels_have_no_scratch_memory(tmp_path):
    with open(pod.LIB_PATH, "rb") as f:
        blob = f.read()
    scratch = {}
    for i, obj in enumerate(code_objects(blob)):
        path = tmp_path / f"{i}.elf"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for name, size in re.findall(r"\.name:\s+(\S+).*?\.private_segment_fixed_size:\s+(\d+)", notes, re.S):
            scratch[name] = int(size)
    attention = {k: v for k, v in scratch.items() if re.search(r"(prefill|decode|fused|fused_cta|combine)_kernel", k)}
    # 2 types x 3 head_dims x (4 kernels x 4 layouts + combine)
    assert len(attention) == 2 * 3 * (4 * 4 + 1)
    assert {k: v for k, v in attention.items() if v} == {}


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_kernels_whose_units_merge_have_no_scratch_memory_either(tmp_path):
    with open(pod.LIB_PATH, "rb") as f:
        blob = f.read()
    scratch = {}
    for i, obj in enumerate(code_objects(blob)):
        path = tmp_path / f"{i}.elf"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for name, size in re.findall(r"\.name:\s+(\S+).*?\.private_segment_fixed_size:\s+(\d+)", notes, re.S):
            if re.search(r"(decode|fused|fused_cta)_merging", name):
                scratch[name] = int(size)
    # 2 types x 2 head_dims x 3 kernels x 4 layouts
    assert len(scratch) == 2 * 2 * 3 * 4
    assert {k: v for k, v in scratch.items() if v} == {}


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_counter_updates_without_a_result_are_waited_for(tmp_path):
    """The last workgroup of an attention kernel clears the counters after all have counted themselves in.  An atomic
    that returns its old value has arrived once that is used; one that returns nothing (the mark of an XCD whose
    queues are used up) has to be waited for on the spot, or it may land after the clearing and stay into the next call."""
    with open(pod.LIB_PATH, "rb") as f:
        blob = f.read()
    n_marks = 0
    for i, obj in enumerate(code_objects(blob)):
        path = tmp_path / f"{i}.elf"
        path.write_bytes(obj)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
        lines = [line.split("//")[0].split() for line in text.splitlines() if line.startswith("\t")]
        for at, words in enumerate(lines):
            if words[0].startswith("global_atomic") and "sc0" not in words:      # sc0: returns the old value
                n_marks += 1
                assert lines[at + 1][:2] == ["s_waitcnt", "vmcnt(0)"], " ".join(words + ["|"] + lines[at + 1])
    # 2 types x 3 head_dims x 3 kernels (decode, fused, fused_cta) x 4 layouts, as often as the compiler copies the walk
    # (the kernels whose units merge claim nothing)
    assert n_marks >= 2 * 3 * 3 * 4
