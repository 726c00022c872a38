"""Small C++ programs against the library's own headers and host functions, built with g++ and run on the CPU."""
import os
import subprocess

import paper_2502_05507_amd as P

PKG = os.path.dirname(os.path.abspath(P.__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def run(tmp_path, source):
    """Compile `source` (it may include the headers of csrc/ and call what libbae.so exports); its output's lines."""
    src, exe = tmp_path / "program.cpp", tmp_path / "program"
    src.write_text(source)
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", f"-I{os.path.join(PKG, 'csrc')}", f"-I{ROCM}/include",
           str(src), "-o", str(exe), f"-L{PKG}", "-l:libbae.so", f"-Wl,-rpath,{PKG}", f"-L{ROCM}/lib",
           f"-Wl,-rpath,{ROCM}/lib", "-lamdhip64"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout.splitlines()
