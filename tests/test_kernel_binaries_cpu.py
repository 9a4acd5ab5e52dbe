"""What the compiler made of the scan kernels in the last build (CPU only): spilled registers of the kernels that may spill, and
instructions that must not appear."""
import glob
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2604_04250_amd")

# Most vector registers a kernel of a family spills: what each family's worst kernel does.  The backward kernels with the valve or
# retentions fill the 128 registers of four waves a SIMD; behind the harmonic convolution with both kinds of logits the front-end holds the
# raw gradients, 48 neighbours' and 8 more sums beside.
CEILINGS = {"cawn_bwd_plain": 0, "cawn_bwd_valve": 0, "cawn_bwd_ret": 10, "cawn_bwd_hconv": 2, "cawn_bwd_hconv_valve": 9,
            "cawn_bwd_hconv_ret": 35, "cawn_fwd_hconv_valve_ret": 1}


def _reports():
    found = glob.glob(os.path.join(PKG, "csrc", "*.res.txt"))
    if not found:
        pytest.skip("no resource report: library was not built by paper_2604_04250_amd.build")
    return found


def test_spilled_registers_stay_below_each_familys_ceiling():
    seen = 0
    for path in _reports():
        most = CEILINGS.get(os.path.basename(path)[:-len(".res.txt")], 0)
        name = ""
        for line in open(path):
            key, _, val = line.partition(":")
            if key == "Function Name":
                name = val.strip()
            elif key.startswith("VGPRs Spill") and ("fwd_kernel" in name or "bwd_kernel" in name):
                assert int(val) <= most, (os.path.basename(path), name, int(val))
                seen += 1
    assert seen >= 35


def test_no_64_bit_shift_by_a_vector_register(tmp_path):
    """Gate masks came out wrong now and then while kernels shifted a 64-bit ballot by a vector register; no such shift
    is left in the library's device code, nor may the compiler form one unseen."""
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    lib = os.path.join(PKG, "libcawn.so")
    if not os.path.exists(objdump) or not os.path.exists(lib):
        pytest.skip("no disassembler, or no library")
    shutil.copy(lib, tmp_path / "lib.so")
    subprocess.run([objdump, "--offloading", str(tmp_path / "lib.so")], check=True, stdout=subprocess.DEVNULL, cwd=tmp_path)
    objects = [str(p) for p in tmp_path.iterdir() if "gfx950" in p.name]
    assert objects
    amount = re.compile(r"v_(?:lshlrev|lshrrev|ashrrev)_[bi]64(?:_e64)? v\[[0-9:]+\], [va]\d|"
                        r"v_lshl_add_u64 v\[[0-9:]+\], [^,]+, [va]\d")

    def scan(obj):
        kernels = shifts = 0
        with subprocess.Popen([objdump, "-d", "--no-show-raw-insn", obj], stdout=subprocess.PIPE, text=True) as p:
            for line in p.stdout:
                kernels += "_kernel" in line and line.rstrip().endswith(">:")
                shifts += "64" in line and amount.search(line) is not None
        assert p.returncode == 0
        return kernels, shifts
    with ThreadPoolExecutor(8) as ex:
        found = list(ex.map(scan, objects))
    assert sum(k for k, _ in found) >= 35
    assert sum(s for _, s in found) == 0
