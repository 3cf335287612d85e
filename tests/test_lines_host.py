"""Lines and nodes of the table hierarchy (csrc/fdy_lines.hpp) on the CPU, in their own source
compiled for the host under AddressSanitizer, against the definition."""
import os
import subprocess

from paper_2604_06664_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_lines_and_nodes_against_the_definition(tmp_path):
    exe = str(tmp_path / "lines_host")
    subprocess.check_call([build.hipcc(), "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-g",
                           "-Xarch_host", "-fsanitize=address", "-fno-gpu-sanitize",
                           "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                           os.path.join(HERE, "level0", "lines_host.hip"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    assert ", 0 wrong" in r.stdout
