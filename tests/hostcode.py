"""Runs host code of the library's headers: a C++ main() over csrc/, compiled for the host alone."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run(body, tmp_path):
    """The lines that `body` (declarations and a main()) prints."""
    src, exe = os.path.join(str(tmp_path), "host.hip"), os.path.join(str(tmp_path), "host")
    with open(src, "w") as f:
        f.write(body)
    subprocess.run(["hipcc", "--offload-host-only", "-O1", "-std=c++17", "-ffp-contract=off", "-Wno-unused-command-line-argument",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2510_16028_amd", "csrc"), src, "-o", exe], check=True)
    return subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
