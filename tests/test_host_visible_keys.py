"""The forward and dQ kernels mask a half of 32 keys by a word of bits (csrc/swaa_common.h, visible_keys).  A host
program built from the same header checks it against the mask's definition, at the edges of halves, windows and sinks.  No GPU."""
import os
import shutil
import subprocess

import pytest

from paper_2512_10411_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not available")
def test_bits_say_which_keys_a_row_sees(tmp_path):
    exe = tmp_path / "visible_keys_check"
    cmd = [build.hipcc_path(), "--offload-arch=gfx950", "-O2", "-std=c++17", "-I", build.CSRC,
           "-I", os.path.join(os.path.dirname(HERE), "include"), "-o", str(exe),
           os.path.join(HERE, "host_checks", "visible_keys_check.hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    print(res.stdout)
    assert res.returncode == 0, res.stdout
    assert " 0 wrong" in res.stdout
