"""The level kernel's work list on the CPU: the functions that cut it (shared by the kernel that writes the
list and the host that sizes the grid) compiled into a small host program that goes over chain lengths,
windows and item sizes (tests/worklist_model.hip)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_items_fit_the_kernel_their_list_and_the_grid(tmp_path):
    exe = str(tmp_path / "worklist_model")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
                    "-o", exe, os.path.join(HERE, "worklist_model.hip")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert (r.returncode, r.stdout.strip()) == (0, "ok"), r.stdout
