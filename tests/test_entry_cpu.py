"""The edge kernels' entry code on byte vectors against the step-by-step form of
the same method (sanitize/steps.h), compiled for the host under AddressSanitizer and
UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2301_04285_amd", "csrc")


def test_byte_vector_entries_equal_the_steps(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "byte_vectors")
    subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-g",
                    "-std=c++17", "-Xarch_host", "-fsanitize=address", "-Xarch_host",
                    "-fsanitize=undefined", "-Xarch_host", "-fno-sanitize-recover=undefined",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(HERE, "sanitize", "byte_vectors.cpp"), "-o", exe],
                   check=True, capture_output=True, timeout=600)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0"))
    assert p.returncode == 0, p.stdout + p.stderr
    assert "runtime error" not in p.stderr and "Sanitizer" not in p.stderr, p.stderr
    assert " 0 mismatches" in p.stdout and int(p.stdout.split()[0]) > 740_000, p.stdout


@pytest.mark.parametrize("nd", range(1, 64))
def test_short_rows_divide_exactly(nd):
    """A lane's row among rows shorter than a wavefront: column j < nd + 64 by one
    multiplication, as the kernels compute it."""
    mul = 65535 // nd + 1
    assert all((j * mul) >> 16 == j // nd for j in range(nd + 64))
