"""The solver's kernels on the host, with `done` stored between the starts of a workgroup's waves."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1911_09220_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
CLANG = os.path.join(ROCM, "llvm", "bin", "clang++")


@pytest.mark.skipif(not os.path.exists(CLANG), reason="no clang")
def test_workgroup_stops_as_a_whole(tmp_path):
    # device.hpp names a scalar register in asm, which the host has not
    for f in ("k_solver.hip", "direction.hpp", "solver.hpp", "internal.hpp", "device.hpp"):
        with open(os.path.join(CSRC, f)) as src, open(tmp_path / f, "w") as dst:
            dst.write(src.read().replace('"+s"', '"+r"'))
    exe = str(tmp_path / "stop")
    build = subprocess.run(
        [CLANG, "-x", "c++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__",
         f"-I{os.path.join(HERE, 'emulate')}", f"-I{tmp_path}", f"-I{ROCM}/include",
         f"-I{os.path.join(ROOT, 'include')}", os.path.join(HERE, "emulate", "stop_inside_launch.cpp"),
         "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout
