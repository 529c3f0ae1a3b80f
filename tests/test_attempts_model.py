"""The bounds at which searches with send times, or with forward and backward maxima apart, are asked one after the other
(tests/attempts_model.hip, on the library's own rule): none twice, none below the least value, and an end."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_no_bound_is_asked_twice(tmp_path):
    exe = str(tmp_path / "attempts_model")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
                    "-o", exe, os.path.join(HERE, "attempts_model.hip")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert (r.returncode, r.stdout.strip()) == (0, "ok"), r.stdout
