"""What the compiler made of the kernels: the notes of the code objects inside the built library, no GPU."""
import re
import struct
import subprocess

import pytest

from paper_2602_11235_amd import hta

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def kernel_notes(tmp_path):
    """(kernel name, bytes of scratch per lane, vector registers kept there) of every kernel of the library."""
    hta.load_library()
    data = open(hta.LIB_PATH, "rb").read()
    elf, notes = tmp_path / "code.elf", []
    at = data.find(BUNDLE)
    while at >= 0:  # [magic][number of entries][offset, size, length of the target's name, that name] ...
        count, = struct.unpack_from("<Q", data, at + len(BUNDLE))
        entry = at + len(BUNDLE) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            target = data[entry + 24:entry + 24 + length].decode()
            entry += 24 + length
            if "gfx950" in target and size:
                elf.write_bytes(data[at + offset:at + offset + size])
                text = subprocess.run([READELF, "--notes", str(elf)], capture_output=True, text=True, check=True).stdout
                for kernel in re.split(r"\n\s+- \.agpr_count", text)[1:]:
                    value = lambda key: re.search(r"\." + key + r":\s+(\S+)", kernel).group(1)
                    notes.append((value("name"), int(value("private_segment_fixed_size")), int(value("vgpr_spill_count"))))
        at = data.find(BUNDLE, at + 1)
    return notes


@pytest.mark.parametrize("kernel,variants", [("serve_kernel", 24), ("fwd_bf16_kernel", 16), ("brief_kernel", 24)])
def test_no_scratch(tmp_path, kernel, variants):
    """The kernels that live for microseconds, and the forward pass, keep all their registers."""
    notes = [n for n in kernel_notes(tmp_path) if kernel in n[0]]
    assert len(notes) >= variants
    assert not [n for n in notes if n[1] or n[2]]
