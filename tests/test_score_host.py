"""CPU: the device half of csrc/rv.hip compiled for the host and run one workgroup at
a time with its waves in many orders (tests/emulator).  What two waves do without a
barrier between them shows as a wrong or an order-dependent result, or as waves at
different barriers.  Tolerance: none."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2012_12618_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


def device_half():
    """rv.hip up to its host side; its two pieces of AMD assembly as emulator calls."""
    src = open(os.path.join(CSRC, "rv.hip")).read()
    src, n = re.subn(r"\n// -+\n// Host side\n.*", "\n}  // namespace\n", src, flags=re.S)
    src, m = re.subn(r"__device__ int amdgcn_writelane\([^;]*;", "", src)
    src, k = re.subn(r"float e0, e1, e2, e3;\s*uint64_t m0.*?asm\(\"v_dot2_f32_f16.*?return [^;]*;",
                     "const uint32_t cc[4] = {c0, c1, c2, c3};\nconst float ww[4] = {w0, w1, w2, w3};\n"
                     "return emu::dot_count4(cc, ww, nd, t);", src, flags=re.S)
    assert (n, m, k) == (1, 1, 1)
    return src


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    if not os.path.exists(CLANG) and shutil.which("clang++") is None:
        pytest.skip("clang++ not found")
    d = tmp_path_factory.mktemp("score_host")
    (d / "device.inc").write_text(device_half())
    exe = str(d / "score_host_check")
    subprocess.run([CLANG if os.path.exists(CLANG) else "clang++", "-std=c++17", "-O1",
                    "-ffp-contract=off", "-w", "-I" + os.path.join(ROOT, "tests", "emulator"),
                    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                    f'-DRV_DEVICE_SOURCE="{d / "device.inc"}"', "-o", exe,
                    os.path.join(ROOT, "tests", "score_host_check.cpp")], check=True)

    def run(what):
        r = subprocess.run([exe, what], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout[-2000:] + r.stderr[-2000:]

    return run


@pytest.mark.parametrize("what", ["no-reference", "other-workgroups", "refit-order", "deferred"])
def test_any_order_of_the_waves(check, what):
    check(what)
