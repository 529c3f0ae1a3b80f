"""What the library asks of the runtime once per device (more than 64 KiB of dynamic LDS for a kernel), on the CPU
with devices and answers of the test's own (tests/once_model.hip)."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2103_16063_amd", "csrc")


def test_every_device_is_asked_and_a_failure_is_not_kept(tmp_path):
    exe = str(tmp_path / "once_model")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
                    "-o", exe, os.path.join(HERE, "once_model.hip")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert (r.returncode, r.stdout.strip()) == (0, "ok"), r.stdout


def test_function_attributes_are_set_through_it_only():
    for name in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, name)) as f:
            calls = len(re.findall(r"hipFuncSetAttribute\(", f.read()))
        assert calls == (1 if name == "rannc_dp_once.h" else 0), name
