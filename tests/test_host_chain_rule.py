"""Calls whose longest row is the time run on 32 rows of a head per workgroup, the others on rows that walk their keys
together; what decides is that row's keys against those of all rows.  A host program built from the same source checks
both counts against the mask's definition, sinks included.  No GPU."""
import os
import shutil
import subprocess

import pytest

from paper_2512_10411_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not available")
def test_rows_are_counted_with_their_sinks(tmp_path):
    exe = tmp_path / "chain_rule_check"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [build.hipcc_path(), *flags, "-o", str(exe), os.path.join(HERE, "host_checks", "chain_rule_check.hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    print(res.stdout)
    assert res.returncode == 0, res.stdout
    assert " 0 wrong" in res.stdout
