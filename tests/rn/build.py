"""Build tests/rn/rn_check and tests/rn/rn_forms, test helpers that run the
device rounding helpers (paper_2104_04347_amd/csrc/wcc_rn.hpp) on operands from
files.  Compiled with the library's device flags; run by
__graft_entry__.build()."""
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
EXES = [os.path.join(HERE, name) for name in ("rn_check", "rn_forms")]
CSRC = os.path.join(ROOT, "paper_2104_04347_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def build() -> list:
    hipcc = shutil.which("hipcc") or os.path.join(ROCM, "bin", "hipcc")
    for exe in EXES:
        tmp = exe + ".tmp"
        cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off", "-fno-fast-math",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", f"-I{CSRC}",
               f"-I{os.path.join(ROOT, 'include')}", exe + ".hip", "-o", tmp]
        subprocess.run(cmd, check=True)
        os.replace(tmp, exe)
    return EXES


if __name__ == "__main__":
    print(*build())
    sys.exit(0)
