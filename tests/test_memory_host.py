"""What the library keeps between calls and handles (csrc/memory.cpp), on a runtime made of
counters: workspaces by stream and by the end of their calls, bounds, what goes back with
the last handle, after the time and when memory runs out, threads, and the thread's end at
exit."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_memory_on_a_counting_runtime(tmp_path):
    exe = str(tmp_path / "memory_host")
    src = [os.path.join(ROOT, "tests", "memory_host.cpp"), os.path.join(ROOT, "paper_2505_08985_amd", "csrc", "memory.cpp")]
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-DPNDF_BLOCK_KEEP_SECONDS=0.3", "-w",
           "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "paper_2505_08985_amd", "csrc"),
           "-I" + os.path.join(ROOT, "include")] + src + ["-o", exe, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.returncode, r.stdout, r.stderr[-3000:])
