"""What the states of the ordered scan hold, over sequences of launches, on the CPU in the kernel's own source."""
import os
import subprocess

from paper_2604_06664_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_fields_and_sums_of_launches_in_turn(tmp_path):
    exe = str(tmp_path / "scan_states_host")
    subprocess.check_call([build.hipcc(), "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-g",
                           "-Xarch_host", "-fsanitize=address", "-fno-gpu-sanitize",
                           "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                           os.path.join(HERE, "level0", "scan_states_host.hip"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0 and ", 0 wrong" in r.stdout, (r.stdout + r.stderr)[-3000:]
