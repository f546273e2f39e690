"""Builds a host-only program against the library's internal header (the
functions that host and device code share)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def build_host(source: str, out_path: str) -> None:
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-Wno-unused-function",
           "-I", os.path.join(ROOT, "paper_2608_27384_amd", "csrc"),
           os.path.join(HERE, source), "-o", out_path]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
