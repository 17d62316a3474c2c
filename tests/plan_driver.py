"""Builds a small host program around the library's own planning functions, so
that the plans of many sizes can be checked without a GPU: the program includes
the internal header and is linked with the built library."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest


def run_plan_program(tmp_path, body: str, headers=()) -> str:
    """Output of a C++ main() whose body is `body`, compiled for the host only,
    after the internal headers named."""
    from paper_2503_01582_amd import _lib
    from paper_2503_01582_amd.build import CSRC, HIPCC, ROOT
    if shutil.which(HIPCC) is None:
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include <vector>\n#include "common.h"\n'
                   + "".join(f'#include "{h}"\n' for h in headers) +
                   "using namespace prenom;\n"
                   "#define CHECK(c, ...) do { if (!(c)) { printf(__VA_ARGS__); return 1; } } while (0)\n"
                   "int main()\n{\n" + body + "\n    printf(\"ok\\n\");\n    return 0;\n}\n")
    lib = _lib.LIB_PATH
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", CSRC, str(src), "-o", str(exe), "-x", "none", lib, f"-Wl,-rpath,{os.path.dirname(lib)}"],
                   check=True, capture_output=True, text=True)
    return subprocess.run([str(exe)], capture_output=True, text=True).stdout
