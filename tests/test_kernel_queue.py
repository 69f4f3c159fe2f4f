"""The work queue's request in the kernels that take one item after the other: nothing waits for it where it is made.  The AMD assembly of the code
objects inside the built library, no GPU."""
import re
import struct
import subprocess

import pytest

from paper_2602_11235_amd import hta
from tests.test_kernel_resources import BUNDLE

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """kernel name -> its instructions in order"""
    hta.load_library()
    data, elf, found = open(hta.LIB_PATH, "rb").read(), tmp_path_factory.mktemp("queue") / "code.elf", {}
    at = data.find(BUNDLE)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(BUNDLE))
        entry = at + len(BUNDLE) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            target = data[entry + 24:entry + 24 + length].decode()
            entry += 24 + length
            code = data[at + offset:at + offset + size]
            if "gfx950" in target and b"bwd_dkdv_" in code:
                elf.write_bytes(code)
                text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(elf)], capture_output=True, text=True, check=True).stdout
                for part in re.split(r"\n<(?=_Z)", text)[1:]:
                    name, body = part.split(">:", 1)
                    found[name] = [line.split("//")[0].strip() for line in body.splitlines() if line.strip()]
        at = data.find(BUNDLE, at + 1)
    return found


def at_once(code, i):
    for line in code[i + 1:i + 13]:
        if "vmcnt" in line:
            return True
        if "branch" in line:
            return False
    return False


def loads_in_flight(code, i):
    """16-byte loads in front of instruction i with no wait in between"""
    n = 0
    for line in reversed(code[:i]):
        if "vmcnt" in line:
            break
        n += line.startswith("global_load_dwordx4")
    return n


def atomics(code):
    return [i for i, line in enumerate(code) if line.startswith("global_atomic_add") and "sc0" in line]


def test_nothing_waits_for_the_next_item_where_it_is_asked_for(kernels):
    """The streaming dK/dV kernels: two loops over the rows, and nothing waits in them.  (Waited for at once: what queue_resolve takes from other lists, and
    asking behind an item without work.)"""
    chosen = {name: code for name, code in kernels.items() if "bwd_dkdv_kernel" in name}
    assert len(chosen) >= 10
    for name, code in chosen.items():
        assert sum(not at_once(code, i) for i in atomics(code)) >= 2, (name, [code[i:i + 9] for i in atomics(code)])


def test_waits_together_with_the_loads_of_the_last_keys(kernels):
    """A user's rows resident: no register to leave the answer in, so it waits where the wave waits for eight loads of 16 bytes."""
    chosen = [code for name, code in kernels.items() if "bwd_dkdv_resident_kernel" in name]
    assert chosen and all(max(loads_in_flight(code, i) for i in atomics(code)) >= 8 for code in chosen)
