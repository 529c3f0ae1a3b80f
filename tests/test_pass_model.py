"""The recomputing level kernel's pass list on the CPU: the closed form that numbers a chunk's stages, and the
room of the list (tests/pass_model.hip, on the library's own functions)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_stages_are_numbered_through_and_fit_their_list(tmp_path):
    exe = str(tmp_path / "pass_model")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
                    "-o", exe, os.path.join(HERE, "pass_model.hip")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert (r.returncode, r.stdout.strip()) == (0, "ok"), r.stdout
