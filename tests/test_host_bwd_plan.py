"""The backward cuts the rows that see sink keys into segments and, where key tiles are few, all steps into pieces
(plan_bwd, csrc/swaa_bwd.hip).  A host program built from the same source checks that every row which sees a key tile
is in exactly one tile of that key tile's workgroups, whatever the batch and the sinks.  No GPU."""
import os
import shutil
import subprocess

import pytest

from paper_2512_10411_amd import build

from test_gpu_bwd import LINE, NAN_LINE, UNITS

HERE = os.path.dirname(os.path.abspath(__file__))


needs_hipcc = pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                                 reason="hipcc not available")


def host_program(name, folder):
    exe = folder / name
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [build.hipcc_path(), *flags, "-o", str(exe), os.path.join(HERE, "host_checks", name + ".hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return str(exe)


@needs_hipcc
def test_every_row_that_sees_a_key_tile_is_in_one_workgroups_list(tmp_path):
    res = subprocess.run([host_program("bwd_plan_check", tmp_path)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    print(res.stdout)
    assert res.returncode == 0, res.stdout
    assert " 0 wrong" in res.stdout


@needs_hipcc
def test_the_gpu_tests_run_on_the_kernels_that_they_name(tmp_path):
    """The lists of tests/test_gpu_bwd.py name the dK/dV kernel of every call, in pieces and on whole key tiles."""
    calls = [(c, pieces) for c in UNITS + LINE + NAN_LINE for pieces in (1, 0)]
    text = "".join(" ".join(str(x) for x in (*c[:6], c[3] if c[6] is None else c[6], pieces)) + "\n" for c, pieces in calls)
    res = subprocess.run([host_program("bwd_kernel_of", tmp_path)], input=text, stdout=subprocess.PIPE, text=True, timeout=60, check=True)
    lines = [ln.split() for ln in res.stdout.splitlines()]
    assert len(lines) == len(calls)
    for (c, pieces), (n_split, _, eight) in zip(calls, lines):
        assert (int(n_split) > 1) == (pieces == 1 and len(c[7]) == 2), (c, pieces, n_split)
        assert ("8" if eight == "1" else "1") == c[7][0 if pieces else -1], (c, pieces)
    assert sum(c[7][-1] == "1" for c in UNITS) >= 7
