"""The backward cuts the rows that see sink keys into segments and, where key tiles are few, all steps into pieces
(plan_bwd, csrc/swaa_bwd.hip).  A host program built from the same source checks that every row which sees a key tile
is in exactly one tile of that key tile's workgroups, whatever the batch and the sinks.  No GPU."""
import os
import shutil
import subprocess

import pytest

from paper_2512_10411_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not available")
def test_every_row_that_sees_a_key_tile_is_in_one_workgroups_list(tmp_path):
    exe = tmp_path / "bwd_plan_check"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [build.hipcc_path(), *flags, "-o", str(exe), os.path.join(HERE, "host_checks", "bwd_plan_check.hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    print(res.stdout)
    assert res.returncode == 0, res.stdout
    assert " 0 wrong" in res.stdout
