"""The large-M kernel's variants for rows beyond kNarrowK form every address of a copy in 64 bits: none of their copies to LDS
takes a 32-bit lane offset.  (Rows of weights lie K / 64 scales apart with groups of 64: 63 rows of them pass 2^32 bytes above
K = 2^31, which a 32-bit offset would wrap to another row's scales.)"""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2507_04610_amd import binding
from test_kernel_metadata import device_code_objects

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
KERNEL = re.compile(r"<_ZN4any414prefill_kernelILi\dELb[01]ELb[01]ELb[01]ELb([01])EE")     # <BITS, FINE, F16, NOLUT, WIDE>
COPY = re.compile(r"global_load_lds_\w+ (.*?)(?://|$)")


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump of the ROCm toolchain is needed")
def test_wide_copies_take_64_bit_addresses():
    if not os.path.exists(binding.LIB_PATH):
        pytest.skip("libany4.so has not been built")
    kernels = {"0": 0, "1": 0}
    copies, narrow = 0, []
    with tempfile.TemporaryDirectory() as tmp:
        for i, image in enumerate(device_code_objects(binding.LIB_PATH)):
            path = os.path.join(tmp, f"co{i}.elf")
            with open(path, "wb") as f:
                f.write(image)
            text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", path], capture_output=True, text=True, check=True).stdout
            wide = False
            for line in text.splitlines():
                if line.endswith(">:"):
                    m = KERNEL.search(line)
                    wide = bool(m) and m.group(1) == "1"
                    if m:
                        kernels[m.group(1)] += 1
                m = COPY.search(line) if wide else None
                if m:
                    copies += 1
                    if m.group(1).split(",")[-1].strip().split()[0] != "off":
                        narrow.append(line.strip())
    assert kernels["1"] == kernels["0"] >= 10 and copies > 10 * kernels["1"]
    assert not narrow, (len(narrow), narrow[:5])
