"""Register use of kernels in the built library (this repository's own build, read from its code objects' metadata):
those whose time hangs on the waves that fit a SIMD, and those that once spilled."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2104_04347_amd import build
from test_rounding_isa import BUNDLER, MAGIC, ROCM

READELF = os.path.join(ROCM, "llvm", "bin", "llvm-readelf")


def _kernels(lib: str, tmp) -> dict:
    """Demangled kernel name -> (vector registers, accumulation ones included; spilled vector registers)."""
    fat, copy = tmp / "fatbin", tmp / "lib.so"
    shutil.copyfile(lib, copy)                       # objcopy rewrites its input
    subprocess.run(["objcopy", "--dump-section", f".hip_fatbin={fat}", str(copy), str(tmp / "discard.so")],
                   check=True, capture_output=True)
    data = fat.read_bytes()
    starts = [m.start() for m in re.finditer(re.escape(MAGIC), data)]
    found = {}
    for a, b in zip(starts, starts[1:] + [len(data)]):
        src, co = tmp / "b.bin", tmp / "b.co"
        src.write_bytes(data[a:b])
        subprocess.run([BUNDLER, "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                        f"--input={src}", f"--output={co}"], check=True, capture_output=True)
        if co.stat().st_size == 0:
            continue
        notes = subprocess.run([READELF, "--notes", str(co)], check=True, capture_output=True, text=True).stdout
        for kernel in re.split(r"\n  - (?=\.agpr_count)", notes)[1:]:
            value = lambda key: int(re.search(rf"\.{key}:\s+(\d+)", kernel).group(1))      # noqa: E731
            found[re.search(r"\.symbol:\s+'?(\S+?)\.kd", kernel).group(1)] = (value("vgpr_count"),
                                                                               value("vgpr_spill_count"))
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True, check=True).stdout
    return {re.sub(r"^void |\(.*", "", n): v for n, v in zip(names.splitlines(), found.values())}


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not (shutil.which("objcopy") and shutil.which("c++filt") and os.path.exists(BUNDLER) and os.path.exists(READELF)):
        pytest.skip("needs binutils and the ROCm LLVM tools")
    assert os.path.exists(build.LIB), "build the library first (__graft_entry__.build())"
    return _kernels(build.LIB, tmp_path_factory.mktemp("co"))


def waves_per_simd(registers: int) -> int:
    """512 registers a SIMD lane, handed out in eights, eight waves at most."""
    return min(8, 512 // (-(-registers // 8) * 8))


# limited Euler in binary64: a wave fewer per SIMD cost up to a quarter of the time at N = 2^20
@pytest.mark.parametrize("P,waves", [(1, 4), (2, 3), (3, 2), (4, 2)])
def test_wide_tiles_keep_their_waves(kernels, P, waves):
    registers, spilled = kernels[f"wcc::k_half_step_wide<2, {P}, true, double>"]
    assert waves_per_simd(registers) >= waves and spilled == 0, registers


def test_batch_kernels_do_not_spill(kernels):
    """A bound on the staged degree-1 kernel once made it spill 43 vector registers in binary64 (a fifth of the time)."""
    batch = {n: v for n, v in kernels.items() if "k_batch_step<" in n}
    assert len(batch) > 20
    assert not {n: v for n, v in batch.items() if v[1]}


def test_2d_limiter_holds_one_general_division_a_field(tmp_path):
    """The general divisions of the 2D limiter, which data in range never reaches, are one instruction sequence for
    each characteristic field, run six times.  Six sequences a field took the 2D kernels 380 s to compile, one 108."""
    from test_rounding_isa import OBJDUMP, _disassemble
    if not (shutil.which("objcopy") and os.path.exists(BUNDLER) and os.path.exists(OBJDUMP)):
        pytest.skip("needs objcopy and the ROCm LLVM tools")
    count, name = {}, None
    for lines in _disassemble(build.LIB, tmp_path):
        for line in lines:
            m = re.match(r"^[0-9a-f]+ <(\S+)>:", line)
            if m:
                name = m.group(1)
            elif "v_div_fixup_f64" in line:
                count[name] = count.get(name, 0) + 1
    rows = {n: c for n, c in count.items() if "k2d_half_step_rowsILi2ELi3ELb1E" in n}
    assert rows
    # 4 fields; the gas state 6, the gradient's direction 4; 1 / rho of the old cell; dt and the two ratios dt / dx
    assert max(rows.values()) <= 4 + 6 + 4 + 1 + 3, rows
