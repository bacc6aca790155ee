"""The split plan's candidates (csrc/swaa_fwd_split.h) are worked out on the device with an approximate
reciprocal.  A host program built from the same header checks that the first of them, the only one
sure to fit every workspace, splits nothing however that reciprocal comes out, that the units of a
batch spread over the eight dies evenly, and that two row tiles share a compute unit only where there is
nothing else; another, that one packed sequence is split alike whether its rows are stated or not.  No GPU."""
import os
import shutil
import subprocess

import pytest

from paper_2512_10411_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not available")
def test_first_candidate_shares_of_the_dies_and_order(tmp_path):
    exe = tmp_path / "split_plan_check"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [build.hipcc_path(), *flags, "-o", str(exe), os.path.join(HERE, "host_checks", "split_plan_check.hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    print(res.stdout)
    assert res.returncode == 0, res.stdout
    assert " 0 wrong" in res.stdout


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not available")
def test_one_packed_sequence_is_split_alike_whether_its_rows_are_stated_or_not(tmp_path):
    exe = tmp_path / "split_bounds_check"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [build.hipcc_path(), *flags, "-o", str(exe), os.path.join(HERE, "host_checks", "split_bounds_check.hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    print(res.stdout)
    assert res.returncode == 0, res.stdout
    assert " 0 wrong" in res.stdout
