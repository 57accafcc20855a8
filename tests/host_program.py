"""Programs under tests/host: the library's host arithmetic driven directly, linked with the built library (no device)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def build(tmp_path, name):
    from paper_2601_11546_amd import binding
    exe, lib_dir = str(tmp_path / name), os.path.dirname(binding.LIB_PATH)
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2601_11546_amd", "csrc"), os.path.join(ROOT, "tests", "host", f"{name}.cpp"),
           "-o", exe, "-L", lib_dir, "-lrelserve", f"-Wl,-rpath,{lib_dir}", "-L", "/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def run(exe, text):
    r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-500:] + r.stderr[-500:]
    return [tuple(map(int, line.split())) for line in r.stdout.splitlines()]
