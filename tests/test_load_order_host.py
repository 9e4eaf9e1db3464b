"""Order of the tile loads in the code the compiler makes (no GPU): the kernels that wait until only the 8 youngest loads,
a tile of V, are in flight read the tile of K next, so no load of K may be issued behind one of V."""
import os
import re
import subprocess

import pytest

from paper_2502_01068_amd import build

WAIT = "s_waitcnt vmcnt(8)"


def _listing(source, tmp_path):
    out = str(tmp_path / "kernel.s")
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.run([build.HIPCC, *flags, "-S", "--cuda-device-only", os.path.join(build.CSRC, source), "-o", out],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return open(out).read()


def _runs(listing, kernel, is_k, is_v):
    """The K and V loads of every instance of a kernel, as strings of K and V that no wait or branch interrupts."""
    runs = []
    for body in re.findall(r"^(?:_Z\w*%s\w*):(.*?)^\.Lfunc_end" % kernel, listing, re.S | re.M):
        run = ""
        for line in (l.strip() for l in body.splitlines()):
            if line.startswith((".LBB", "s_cbranch", "s_branch", WAIT)):
                runs.append(run)
                run = ""
            elif is_k(line):
                run += "K"
            elif is_v(line):
                run += "V"
        runs.append(run)
    return [r for r in runs if r]


@pytest.mark.parametrize("source,kernel,is_k,is_v", [
    ("fkv_decode.hip", "k_decode", lambda s: s.startswith("global_load_lds_dwordx4"),
     lambda s: s.startswith("global_load_dwordx4") and s.endswith(" nt")),
    # only the instance that caches K: its loads of K and V differ in the text
    ("fkv_wout.hip", "k_wout_partialILb1E", lambda s: s.startswith("global_load_lds_dwordx4") and not s.endswith(" nt"),
     lambda s: s.startswith("global_load_lds_dwordx4") and s.endswith(" nt")),
], ids=["decode", "window_output"])
def test_v_is_requested_behind_k(source, kernel, is_k, is_v, tmp_path):
    listing = _listing(source, tmp_path)
    assert WAIT in listing
    runs = _runs(listing, kernel, is_k, is_v)
    assert "KKKKKKKKVVVVVVVV" in runs, runs  # a wave's first tile
    assert set(runs) <= {"KKKKKKKKVVVVVVVV", "KKKKKKKK", "VVVVVVVV"}, runs
