"""What the built kernels take of a compute unit, from the metadata that the compiler put beside their code: the
occupancy that the rules for launches count on is the one that the kernels have."""
import os
import re
import struct
import subprocess

import pytest

from paper_2103_16063_amd import binding

HERE = os.path.dirname(os.path.abspath(__file__))
LLVM = "/opt/rocm/llvm/bin"
SIMDS, REGISTERS, LDS = 4, 512, 160 * 1024  # of a compute unit; vector registers of a lane on a SIMD


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> metadata of every kernel in the library's own gfx950 code objects."""
    tmp = tmp_path_factory.mktemp("code")
    data = open(binding.LIB_PATH, "rb").read()
    out, at = {}, data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + length].decode()
            p += 24 + length
            if "gfx950" not in target or size == 0:
                continue
            path = str(tmp / f"{at}.co")
            with open(path, "wb") as f:
                f.write(data[at + off:at + off + size])
            notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", path], capture_output=True, text=True, check=True).stdout
            for block in re.split(r"\n  - (?=\.)", notes):
                name = re.search(r"^\s+\.name:\s+(_Z\S+)", block, re.M)
                if name:
                    out[name.group(1)] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\s*$", block, re.M)}
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)
    assert len(out) > 50, "no kernels found in the library"
    return out


def waves_per_simd(k):
    vector = max(8, (k["vgpr_count"] + 7) // 8 * 8)
    return min(8, REGISTERS // vector, 8 if k["sgpr_count"] <= 100 else 7)


def workgroups_per_cu(k, threads):
    by_waves = waves_per_simd(k) * SIMDS // (threads // 64)
    lds = k["group_segment_fixed_size"]
    return min(by_waves, LDS // lds if lds else by_waves)


def test_dynamic_lds_beyond_64_kib_is_asked_for(kernels):
    """Every kernel that needs more than 64 KiB of a compute unit's LDS at some size is asked for at every size: how much a kernel has of
    its own changes with its code.  (prepare_kernel holds 60 KiB at most, which its launch asserts.)"""
    csrc = os.path.join(os.path.dirname(HERE), "paper_2103_16063_amd", "csrc")
    assert all(k["group_segment_fixed_size"] <= 4 * 1024 for n, k in kernels.items() if "prepare_kernel" in n)
    launched = set()
    for file in sorted(os.listdir(csrc)):
        text = open(os.path.join(csrc, file)).read()
        asked = {m.replace(" ", "") for m in re.findall(r"allow_lds\(\w+(?:\[\d\])?, \(const void \*\)([\w<>, ]+),", text)}
        assert not re.search(r"if \(lds[^;{]*> [\d* ]+\) \{[^}]*allow_lds", text), file
        for kernel, lds in re.findall(r"hipLaunchKernelGGL\(\(?(\w+_kernel(?:<[^;]*?>)?)\)?, dim3\([^;]*?dim3\([^;]*?\), (?!dim3)([^;]*?), st, ", text):
            if lds != "0":
                launched.add(kernel.replace(" ", ""))
                assert kernel.replace(" ", "") in asked, (file, kernel)
    assert len(launched) >= 8


def test_level_kernels_fit_the_workgroups_that_size_their_items(kernels, tmp_path):
    exe = str(tmp_path / "occupancy_model")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
                    "-o", exe, os.path.join(HERE, "occupancy_model.hip")], check=True)
    table = {}
    for line in subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split("\n"):
        if line:
            bits, cls, recompute, groups = map(int, line.split())
            table[bits, cls, recompute] = groups
    seen, wrong = 0, []
    for name, k in kernels.items():
        m = re.search(r"level_merge(?:_one)?_kernelI([jm])Li(\d+)ELb([01])E", name)
        if not m:
            continue
        seen += 1
        cls = int(m.group(2))  # (the kernel of 48 values takes the narrower levels of 64 devices)
        expected = table[32 if m.group(1) == "j" else 64, 64 if cls == 48 else cls, int(m.group(3))]
        if workgroups_per_cu(k, 256) < expected:
            wrong.append((name, k["vgpr_count"], k["sgpr_count"], workgroups_per_cu(k, 256), expected))
    assert seen == 2 * 2 * (5 + 3) and not wrong, wrong


def test_split_kernels_fit_the_workgroups_their_form_was_chosen_for(kernels):
    # (bits, class) -> workgroups of eight waves on a compute unit, winners unpacked in the launch or apart
    expected = {(32, 8): 4, (32, 16): 4, (32, 32): 3, (32, 64): 2, (64, 8): 4, (64, 16): 3, (64, 32): 2, (64, 64): 1}
    seen, wrong = 0, []
    for name, k in kernels.items():
        m = re.search(r"level_split_fast_kernelI([jm])Li(\d+)E", name)
        if not m:
            continue
        seen += 1
        if workgroups_per_cu(k, 512) < expected[32 if m.group(1) == "j" else 64, int(m.group(2))]:
            wrong.append((name, k["vgpr_count"], workgroups_per_cu(k, 512)))
    assert seen == 2 * 2 * 4 and not wrong, wrong


def test_one_launch_kernels_of_batches_fit_twice_on_a_compute_unit(kernels):
    # (bits, class, times recomputed): sixteen waves each, 64 registers
    twice = {(32, 8, 0), (32, 8, 1), (64, 8, 0), (64, 8, 1), (32, 16, 0), (32, 16, 1)}
    fits = set()
    for name, k in kernels.items():
        m = re.search(r"solve_small_kernelI([jm])Li(\d+)ELb([01])E", name)
        if m and workgroups_per_cu(k, 1024) >= 2:
            fits.add((32 if m.group(1) == "j" else 64, int(m.group(2)), int(m.group(3))))
    assert twice <= fits, twice - fits


def test_kernels_without_tables_fit_as_their_launches_count_on(kernels):
    """Workgroups of a search to a compute unit, by registers, and with the LDS that their launches take: three of four waves
    (1536 cells, 256 sources, 1024 records and the sums of 600 blocks), one of eight or sixteen."""
    sums, levels = lambda n: (n + 6) * 24, lambda cells, sources, records: cells * 12 + sources * 24 + records * 8
    seen = set()
    for name, k in kernels.items():
        m = re.search(r"(reach|bound|form)_kernelI(?:Li(\d+)E|L)", name)
        if not m:
            continue
        seen.add((m.group(1), m.group(2)))
        if m.group(2) == "4":
            assert workgroups_per_cu(k, 256) >= 3, name
            assert 3 * (k["group_segment_fixed_size"] + sums(600) + levels(1536, 256, 1024)) <= LDS, name
        else:
            assert workgroups_per_cu(k, 512 if m.group(2) == "8" else 1024) >= 1, name
        # at sixteen waves to a workgroup 128 registers are all there are
        assert k.get("vgpr_spill_count", 0) <= 3, (name, k["vgpr_spill_count"])
    assert seen == {("reach", "4"), ("reach", "8"), ("reach", "16"), ("bound", None), ("form", None)}, seen
