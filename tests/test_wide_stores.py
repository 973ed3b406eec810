"""The registers of a 12- or 16-byte store's data are not written right behind it.  They are read over several cycles; where the
store has a scalar offset the compiler keeps no distance, and the upper halves of some lanes' data were then the next
store's (large-M kernel, K slices: a few outputs in a million, now and then).  So no such store has a scalar offset, and
behind each of them stand the two wait states that the compiler keeps without one."""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2507_04610_amd import binding
from test_kernel_metadata import device_code_objects

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
STORE = re.compile(r"((?:buffer|global|flat)_store_dwordx[34]) (.*?)(?://|$)")
VECTOR = re.compile(r"(v_\w+) (v\[\d+:\d+\]|v\d+)")
NOP = re.compile(r"s_nop (\d+)")
WAIT_STATES = 2


def registers(operand):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"v(\d+)", operand)
    return {int(m.group(1))} if m else set()


def findings(text):
    """(wide stores, those with a register for a scalar offset, instructions that write a store's data too early)"""
    stores, offsets, early = 0, [], []
    live = []                                                # (wait states since the store, its data)
    for line in text.splitlines():
        m = VECTOR.search(line)
        if m and any(d & registers(m.group(2)) for _, d in live):
            early.append(line.strip())
        nop = NOP.search(line)
        passed = int(nop.group(1)) + 1 if nop else 1
        live = [(n + passed, d) for n, d in live if n + passed < WAIT_STATES]
        m = STORE.search(line)
        if m:
            stores += 1
            operands = [o.strip() for o in m.group(2).split(",")]
            buffer = m.group(1).startswith("buffer")
            live.append((0, registers(operands[0] if buffer else operands[1])))
            if buffer and not operands[3].split()[0].isdigit():                    # (data, lane offset, descriptor, scalar offset)
                offsets.append(line.strip())
    return stores, offsets, early


def test_findings():
    bad = """
        buffer_store_dwordx4 v[4:7], v1, s[8:11], s3 offen sc1
        buffer_store_dwordx4 v[8:11], v1, s[8:11], 0 offen sc1
        v_add_u32_e32 v20, v8, v9
        v_add_u32_e32 v9, 1, v2
        global_store_dwordx3 v[2:3], v[12:14], off
        s_nop 0
        v_mov_b32_e32 v13, v2
        global_store_dwordx4 v3, v[16:19], s[2:3]
        s_nop 1
        v_accvgpr_read_b32 v16, a3
    """
    stores, offsets, early = findings(bad)
    assert stores == 4
    assert [o.split()[1] for o in offsets] == ["v[4:7],"]
    assert [e.split()[1] for e in early] == ["v9,", "v13,"]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump of the ROCm toolchain is needed")
def test_data_of_wide_stores_is_left_alone():
    if not os.path.exists(binding.LIB_PATH):
        pytest.skip("libany4.so has not been built")
    stores, offsets, early = 0, [], []
    with tempfile.TemporaryDirectory() as tmp:
        for i, image in enumerate(device_code_objects(binding.LIB_PATH)):
            path = os.path.join(tmp, f"co{i}.elf")
            with open(path, "wb") as f:
                f.write(image)
            text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", path], capture_output=True, text=True, check=True).stdout
            n, o, e = findings(text)
            stores += n
            offsets += [(i, line) for line in o]
            early += [(i, line) for line in e]
    assert stores > 100
    assert not offsets, (len(offsets), offsets[:5])
    assert not early, (len(early), early[:5])
