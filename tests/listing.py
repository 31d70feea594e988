"""The assembly listing of a source file's kernels, compiled here and kept for the tests that scan it."""
import functools
import os
import subprocess
import tempfile

from paper_2409_15520_amd import build

_DIR = tempfile.TemporaryDirectory()


@functools.lru_cache(maxsize=None)
def listing(name):
    out = os.path.join(_DIR.name, f"{name}.s")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.COMMON, "-S", "--cuda-device-only", "-o", out,
                    os.path.join(build.CSRC, f"{name}.hip")], check=True, capture_output=True)
    with open(out) as f:
        return f.read()
