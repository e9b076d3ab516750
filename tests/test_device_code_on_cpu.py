"""Parts of the device code that are plain arithmetic and loads, compiled for the host and run on the CPU under
sanitizers: no GPU needed, and an access out of range ends the test instead of the GPU's work."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def run_on_cpu(source, tmp_path, *sanitizers):
    exe = tmp_path / "main"
    # the host half alone (no kernel is launched); the symbol of the missing device half is any address
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-fuse-cuid=none", "-Wl,--defsym=__hip_fatbin=main", "-O1", "-g",
           "-std=c++17", "-w"]
    for s in sanitizers:
        cmd += ["-Xarch_host", "-fsanitize=" + s, "-Xarch_host", "-fno-sanitize-recover=" + s]
    build = subprocess.run(cmd + ["-o", str(exe), os.path.join(HERE, source)], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    env = dict(os.environ)
    # (another library may already be preloaded into every process; leak checking needs ptrace)
    env["ASAN_OPTIONS"] = "verify_asan_link_order=0:detect_leaks=0:abort_on_error=0"
    env["UBSAN_OPTIONS"] = "print_stacktrace=1"
    run = subprocess.run([str(exe)], capture_output=True, text=True, env=env, timeout=600)
    assert run.returncode == 0, (run.stdout[-1000:], run.stderr[-3000:])
    assert "runtime error" not in run.stderr and "AddressSanitizer" not in run.stderr, run.stderr[-3000:]
    return run.stdout


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_the_walk_reads_rows_and_nothing_around_them(tmp_path):
    out = run_on_cpu("walk_loads_main.hip", tmp_path, "address", "alignment")
    assert " 0 failed" in out, out
