"""Builds and runs a piece of host C++ against the library's sizing headers."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run(tmp_path, headers, body):
    """Output lines of main() { body }, which sees the given headers of csrc/."""
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    src, exe = str(tmp_path / "t.cpp"), str(tmp_path / "t")
    with open(src, "w") as f:
        f.write("#include <stdio.h>\n" + "".join(f'#include "{h}"\n' for h in headers) +
                "using namespace fz;\nint main()\n{\n" + body + "\nreturn 0;\n}\n")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror=return-type", "-fsanitize=undefined",
                           "-fno-sanitize-recover=all", f"-I{ROOT}/include", f"-I{ROOT}/paper_1509_04394_amd/csrc",
                           src, "-o", exe])
    return subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout.splitlines()
