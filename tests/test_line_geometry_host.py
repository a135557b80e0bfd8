"""Bounds check of the whole-line kernels' layout on the CPU: tests/line_geometry_check.hip is built as a host program
against the offsets and region sizes the kernels use and linked to the library's geometry rules, and checks every line
length; the geometries in use are compared with the kernels the launch switches name. Skipped without hipcc or the
built library."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_1806_10550_amd")


def source(name):
    return open(os.path.join(PKG, "csrc", name)).read()


def switch_cases(text, macro, args):
    """Argument tuples of the uses of a launch macro (its definition has names instead of numbers)."""
    return {tuple(map(int, re.findall(r"\d+", m)))
            for m in re.findall(macro + r"\((" + r",\s*".join([r"\d+"] * args) + r")\)", text)}


def test_whole_line_layout_stays_in_bounds(tmp_path):
    hipcc = shutil.which("hipcc")
    if hipcc is None or not os.path.exists(os.path.join(PKG, "libthinfilm.so")):
        pytest.skip("hipcc or libthinfilm.so not available")
    exe = str(tmp_path / "line_geometry_check")
    b = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", os.path.join(HERE, "line_geometry_check.hip"), "-L" + PKG, "-lthinfilm",
                        "-Wl,-rpath," + PKG, "-o", exe], capture_output=True, text=True, timeout=600)
    assert b.returncode == 0, b.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "line geometry check: ok" in r.stdout, r.stdout[-3000:]
    used = {k: {tuple(map(int, m.split())) for m in re.findall(rf"^{k} (.*)$", r.stdout, re.M)} for k in "xys"}
    line = source("tf_line.hip")
    assert used["x"] == switch_cases(line, "TF_XL", 2)
    assert used["y"] == switch_cases(line, "TF_YL", 2)
    assert used["s"] == switch_cases(source("tf_xrow.hip"), "TF_SB", 3)
    # the ensemble's kernels: per number of waves the cases of a switch and 16 by default
    ens = source("tf_line_ens.hip")
    for kernel, macro, key, most in (("k_xline_ens(", "TF_XC", "x", 4), ("k_yline_ens(", "TF_YC", "y", 2)):
        body = ens[ens.index(kernel):]
        body = body[:body.index("\n}\n")]
        switches = [switch_cases(s, macro, 1) for s in re.findall(r"switch \(cpl\) \{(.*?)\}", body)]
        assert len(switches) == most
        assert {(c, w + 1) for w, s in enumerate(switches) for (c,) in s} == {g for g in used[key] if g[1] <= most}
