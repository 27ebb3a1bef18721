"""Registers of the built step kernels, from the metadata of the library's own
code objects.  On these states the next register costs a wavefront a SIMD (or
goes to scratch), and with it 10 to 25% of the step."""
import re
import shutil
import struct
import subprocess

import pytest

from paper_2607_05668_amd import lbm

LLVM = "/opt/rocm/llvm/bin/"
READELF = LLVM + "llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
pytestmark = pytest.mark.skipif(shutil.which(READELF) is None, reason="no llvm-readelf")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Demangled kernel name -> (registers a lane, bytes of scratch a lane)."""
    data = open(lbm.LIB_PATH, "rb").read()
    folder = tmp_path_factory.mktemp("objects")
    out, at = {}, data.find(MAGIC)
    while at >= 0:
        pos = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            offset, size, n = struct.unpack_from("<QQQ", data, pos)
            target, pos = data[pos + 24:pos + 24 + n], pos + 24 + n
            if b"gfx950" not in target or not size:
                continue
            path = folder / f"{len(out)}.co"
            path.write_bytes(data[at + offset:at + offset + size])
            notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            for k in re.split(r"\n  - \.agpr_count:", notes)[1:]:
                get = lambda key: re.search(rf"\.{key}: +(\S+)", k).group(1)      # noqa: E731
                out[get("name")] = (int(get("vgpr_count")), int(get("private_segment_fixed_size")))
        at = data.find(MAGIC, at + 1)
    names = subprocess.run([LLVM + "llvm-cxxfilt"], input="\n".join(out), capture_output=True, text=True, check=True).stdout.split("\n")
    return dict(zip(names, out.values()))


def _matching(kernels, pattern):
    found = {k: v for k, v in kernels.items() if re.search(pattern, k)}
    assert found, pattern
    return found


# two wavefronts a SIMD hold 256 registers each
@pytest.mark.parametrize("state", ["SysCNSF2D, D2Q5, double", "SysNeoHooke, D2Q9, double"])
def test_single_steps_in_double_leave_two_wavefronts_a_simd(kernels, state):
    for name, (registers, _) in _matching(kernels, rf"k_step<{state}, false, \w+, true, 0>").items():
        assert registers <= 256, (name, registers)


# states that fill one wavefront's 512 registers
@pytest.mark.parametrize("state,scratch", [("SysCNSF2D, D2Q9, double", 0), ("SysMHD, D2Q9, double", 900),
                                           ("SysNSF17, D3Q7, double", 64)])
def test_single_steps_of_the_largest_states_spill_no_more(kernels, state, scratch):
    for name, (_, spilled) in _matching(kernels, rf"k_step<{state}, false, \w+, true, 0>").items():
        assert spilled <= scratch, (name, spilled)


# four wavefronts a SIMD hold 128 registers each
def test_single_step_of_the_deviations_leaves_four_wavefronts_a_simd(kernels):
    for name, (registers, scratch) in _matching(kernels, r"k_step_ne<SysNeoHooke, D2Q9, ").items():
        assert registers <= 128 and scratch <= 32, (name, registers, scratch)
