"""Registers of the built step kernels, from the metadata of the library's own
code objects.  On these states the next register costs a wavefront a SIMD (or
goes to scratch), and with it 10 to 25% of the step."""
import re
import shutil
import struct
import subprocess

import pytest

from paper_2607_05668_amd import lbm

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
pytestmark = pytest.mark.skipif(shutil.which(READELF) is None, reason="no llvm-readelf")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Kernel symbol -> (registers a lane, bytes of scratch a lane)."""
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
    return out


def _matching(kernels, kernel, system, lattice, rest):
    """Instantiations kernel<system, lattice, rest...> (mangled, a regular expression)."""
    start = f"{len(kernel)}{kernel}I{len(system)}{system}{len(lattice)}{lattice}{rest}"
    found = {k: v for k, v in kernels.items() if re.match("_Z" + start, k)}
    assert found, start
    return found


def _single_steps_in_double(kernels, system, lattice):      # no history, 32-bit offsets, BGK
    return _matching(kernels, "k_step", system, lattice, "dLb0ELb[01]ELb1ELi0EE").items()


# two wavefronts a SIMD hold 256 registers each
@pytest.mark.parametrize("state", [("SysCNSF2D", "D2Q5"), ("SysNeoHooke", "D2Q9")])
def test_single_steps_in_double_leave_two_wavefronts_a_simd(kernels, state):
    for name, (registers, _) in _single_steps_in_double(kernels, *state):
        assert registers <= 256, (name, registers)


# states that fill one wavefront's 512 registers
@pytest.mark.parametrize("state,scratch", [(("SysCNSF2D", "D2Q9"), 0), (("SysMHD", "D2Q9"), 900),
                                           (("SysNSF17", "D3Q7"), 64)])
def test_single_steps_of_the_largest_states_spill_no_more(kernels, state, scratch):
    for name, (_, spilled) in _single_steps_in_double(kernels, *state):
        assert spilled <= scratch, (name, spilled)


# four wavefronts a SIMD hold 128 registers each
def test_single_step_of_the_deviations_leaves_four_wavefronts_a_simd(kernels):
    for name, (registers, scratch) in _matching(kernels, "k_step_ne", "SysNeoHooke", "D2Q9", "").items():
        assert registers <= 128 and scratch <= 32, (name, registers, scratch)


# five wavefronts a SIMD, as many as their LDS leaves, hold 96 registers each,
# three hold 168
def test_moments_and_scales_of_the_deviations_leave_their_wavefronts(kernels):
    for name, (registers, _) in _matching(kernels, "k_moments_ne", "SysNeoHooke", "D2Q9", "[df]Lb1E").items():
        assert registers <= 96, (name, registers)
    for name, (registers, _) in _matching(kernels, "k_init_ne", "SysNeoHooke", "D2Q9", "Lb1ELb1E").items():
        assert registers <= 168, (name, registers)
