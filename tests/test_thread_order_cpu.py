"""Kernels whose threads hand values over in LDS, run on the CPU a thread at a
time in several orders: a result that depends on the order lacks a barrier."""
import glob
import os
import re
import shutil
import subprocess

import pytest

TESTS = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(TESTS, "..", "paper_1901_02492_amd", "csrc")
INCLUDE = os.path.join(TESTS, "..", "include")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
CLANG = os.path.join(ROCM, "llvm", "bin", "clang++")


def _without_assembly(text):
    """The kernels' instructions in inline assembly: one is run here and has a
    function in its place, the others pin registers or are not reached."""
    text = text.replace('asm("v_cvt_i32_f64 %0, %1" : "=v"(d) : "v"(f));',
                        "d = saturating_int32(f);")
    out, at = [], 0
    for m in re.finditer(r"(?<![\w])asm( volatile)?\(", text):
        end, depth = m.end(), 1
        while depth:
            depth += {"(": 1, ")": -1}.get(text[end], 0)
            end += 1
        out.append(text[at:m.start()] + "(void)0")
        at = end
    text = "".join(out) + text[at:]
    return re.sub(r'\s+__asm\("llvm[^"]*"\)', "", text)


@pytest.mark.skipif(shutil.which(CLANG) is None, reason="needs ROCm's clang++")
@pytest.mark.parametrize("check", ["rescore", "lightcurve"])
def test_thread_order(check, tmp_path):
    for f in glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip")):
        (tmp_path / os.path.basename(f)).write_text(_without_assembly(open(f).read()))
    exe = str(tmp_path / "check")
    r = subprocess.run([CLANG, "-std=c++17", "-O1", "-w", "-ffp-contract=off",
                        "-fno-strict-aliasing",
                        "-D__HIP_PLATFORM_AMD__", "-I", str(tmp_path), "-I", TESTS, "-I", INCLUDE,
                        "-I", os.path.join(ROCM, "include"), "-x", "c++",
                        os.path.join(TESTS, f"{check}_order_check.cpp"), "-o", exe,
                        "-Wl,--unresolved-symbols=ignore-all"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
