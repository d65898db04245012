"""The profiling builds' phase names belong to the kernels' phase indices."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2605_17913_amd", "csrc")


def _marks():
    """Phases that the kernels' code marks, QPK_PT(PH_...)."""
    with open(os.path.join(CSRC, "qp_kernel_impl.hpp")) as f:
        return sorted(set(re.findall(r"QPK_PT\((PH_\w+)\)", f.read())))


def test_every_mark_is_reported_under_its_own_name(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    marks = _marks()
    assert len(marks) >= 20
    src = tmp_path / "names.cpp"
    src.write_text('#include <cstdio>\n#include "qp_phase.h"\nint main() {\n'
                   + "".join(f'  std::printf("{m} %s\\n", kPhaseNames[{m}]);\n' for m in marks)
                   + "  return 0;\n}\n")
    exe = tmp_path / "names"
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    got = dict(line.split() for line in out.splitlines())
    assert got == {m: m[len("PH_"):].lower() for m in marks}
