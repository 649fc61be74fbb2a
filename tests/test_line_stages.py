"""CPU: the transform stages of the line kernels, as the kernels run them.

Every split that is instantiated, in its two or three stages, with the
prime-factor maps, the LDS positions, the power twiddles and the table orders of
the device code, against a brute-force DFT in long double (g++ with
AddressSanitizer and UndefinedBehaviorSanitizer).  The splits are read from the
kernel sources; the combined launch has to hold the same ones."""
import concurrent.futures as cf
import os
import re
import shutil
import subprocess

import pytest

from test_fft_codelets import CSRC, HERE, _splits


def test_combined_launch_has_the_same_splits():
    src = open(os.path.join(CSRC, "line4_mixed.h")).read()
    mixed = {(int(n), int(a), int(b)) for n, a, b in re.findall(r"X\((\d+), (\d+), (\d+)\)", src)}
    assert mixed == {s for s in _splits() if s[0] <= 256}


def test_stages_against_brute_force_dft(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    splits, parts = _splits(), 6   # programs built side by side

    def run(part):
        d = tmp_path / str(part)
        d.mkdir()
        mine = splits[part::parts]
        (d / "line_splits.inc").write_text("\n".join("SPLIT(%d, %d)" % (a, b) for _, a, b in mine) + "\n")
        cmd = [gxx, "-std=c++17", "-O1", "-Wno-unknown-pragmas", "-fsanitize=address,undefined",
               "-fno-sanitize-recover=all", "-I", str(d), "-I", CSRC,
               os.path.join(HERE, "line_stages_check.cpp"), "-o", str(d / "check")]
        subprocess.run(cmd, check=True, capture_output=True, text=True)
        r = subprocess.run([str(d / "check")], capture_output=True, text=True, timeout=600)
        m = re.search(r"cases (\d+) failures 0 worst (\S+)", r.stdout)
        return r.returncode == 0 and m is not None and int(m.group(1)) == len(mine) > 0, r.stdout[-2000:] + r.stderr[-2000:]

    with cf.ThreadPoolExecutor(parts) as ex:
        for ok, text in ex.map(run, range(parts)):
            assert ok, text
