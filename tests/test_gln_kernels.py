"""The group layer normalization's kernels in the built library, no GPU: each asks for its dynamic LDS, and which keep registers in scratch."""
import subprocess

from paper_2602_11235_amd import hta
from tests.test_kernel_resources import READELF, kernel_notes


def kernels(tmp_path):
    return [n for n in kernel_notes(tmp_path) if n[0].startswith(("_ZN3gln10fwd_kernelI", "_ZN3gln10bwd_kernelI"))]


def test_every_kernel_asks_for_its_lds(tmp_path):
    """One guarded static of allow_lds for each kernel, not one for all of a type."""
    symbols = subprocess.run([READELF, "--symbols", "--wide", hta.LIB_PATH], capture_output=True, text=True, check=True).stdout
    guards = {word for word in symbols.split() if word.startswith("_ZGVZN3gln") and "allow_lds" in word}
    assert len(guards) == len(kernels(tmp_path)) > 30


def test_scratch(tmp_path):
    """None, but for rows of four chunks in float32 with a gate, in the backward pass."""
    spilled = [n for n in kernels(tmp_path) if n[1] or n[2]]
    assert [n[0] for n in spilled] == ["_ZN3gln10bwd_kernelIfLi4ELi64ELb1ELi512EEEvNS_4ArgsE"] and spilled[0][1] <= 64
