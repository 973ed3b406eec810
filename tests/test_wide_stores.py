"""The registers of a 12- or 16-byte store's data are not written by the instruction right behind it.  They are read over
several cycles; with a scalar offset in the store the compiler puts such an instruction there, and the upper halves of some
lanes' data were then the next store's (large-M kernel, K slices: a few outputs in a million, now and then)."""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2507_04610_amd import binding
from test_kernel_metadata import device_code_objects

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
STORE = re.compile(r"(?:buffer|global|flat)_store_dwordx[34] (.*?)(?://|$)")
VECTOR = re.compile(r"(v_\w+) (v\[\d+:\d+\]|v\d+)")


def registers(operand):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"v(\d+)", operand)
    return {int(m.group(1))} if m else set()


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump of the ROCm toolchain is needed")
def test_data_of_wide_stores_stays_for_an_instruction():
    if not os.path.exists(binding.LIB_PATH):
        pytest.skip("libany4.so has not been built")
    stores, bad = 0, []
    with tempfile.TemporaryDirectory() as tmp:
        for i, image in enumerate(device_code_objects(binding.LIB_PATH)):
            path = os.path.join(tmp, f"co{i}.elf")
            with open(path, "wb") as f:
                f.write(image)
            text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", path], capture_output=True, text=True, check=True).stdout
            data = set()
            for line in text.splitlines():
                m = VECTOR.search(line)
                if m and data & registers(m.group(2)):
                    bad.append((i, line.strip()))
                data = set()
                m = STORE.search(line)
                if m:
                    stores += 1
                    operands = [o.strip() for o in m.group(1).split(",")]
                    data = registers(operands[0] if "buffer" in line else operands[1])
    assert stores > 100
    assert not bad, (len(bad), bad[:5])
