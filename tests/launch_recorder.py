"""What the library asks of the HIP runtime, without a GPU (tests/launch_recorder.cpp)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2510_25590_amd", "libregione.so")


def build(folder):
    """Builds the stand-in; returns run(commands) -> one (grants, launches) per command: [(bytes, kernel)] and [(grid, dynamic LDS, kernel)].
    refused: commands may fail; one (grants, launches, code and message) each."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler here")
    exe = os.path.join(str(folder), "launch_recorder")
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-isystem", "/opt/rocm/include", os.path.join(ROOT, "tests", "launch_recorder.cpp"),
                    "-rdynamic", "-ldl", "-o", exe], check=True)

    def run(commands, refused=False):
        p = subprocess.run([exe, LIB], input="\n".join(commands) + "\n", capture_output=True, text=True, timeout=120)
        assert p.returncode == 0, p.stderr
        out, grants, launches = [], [], []
        for line in p.stdout.splitlines():
            word, rest = line.split(" ", 1)
            if word == "grant":
                n, kernel = rest.split(" ", 1)
                grants.append((int(n), kernel))
            elif word == "launch":
                x, y, z, lds, kernel = rest.split(" ", 4)
                launches.append(((int(x), int(y), int(z)), int(lds), kernel))
            else:
                assert refused or re.match(r"0\b", rest), rest
                out.append((grants, launches, rest) if refused else (grants, launches))
                grants, launches = [], []
        assert len(out) == len(commands)
        return out
    return run
