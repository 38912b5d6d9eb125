"""The launchers' own argument checks, through a small host program linked to the library: what a kernel has no form for is refused, not
launched as something else."""
import os
import subprocess

from paper_2506_03700_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_forms_that_no_kernel_has_are_refused(tmp_path):
    build.build_hip(force=False)
    exe = str(tmp_path / "launchers")
    p = subprocess.run(["g++", "-std=c++17", "-Wall", "-I", build.CSRC, "-I", os.path.join(ROOT, "include"), "-o", exe,
                        os.path.join(ROOT, "tests", "launchers_driver.cpp"), binding.LIB_PATH, "-Wl,-rpath," + os.path.dirname(binding.LIB_PATH),
                        "-Wl,--unresolved-symbols=ignore-in-shared-libs"], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and "all refused" in r.stdout, r.stdout


def test_kernels_are_those_of_the_stream_s_device(tmp_path):
    build.build_hip(force=False)
    exe = str(tmp_path / "devices")
    p = subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-std=c++17", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-o", exe,
                        os.path.join(ROOT, "tests", "devices_driver.cpp"), "-Wl," + binding.LIB_PATH, "-Wl,-rpath," + os.path.dirname(binding.LIB_PATH),
                        "-Wl,--unresolved-symbols=ignore-in-shared-libs"], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and "every launch on its stream's device" in r.stdout, r.stdout
