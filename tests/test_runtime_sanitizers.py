"""The library's runtime (runtime.cpp: sessions, the ready record, the gate's waits, the
idle-window yield, the session registry) built for the CPU with g++ over host stand-ins
for HIP and the kernels (tests/cpu_runtime/), and run under AddressSanitizer (+ UBSan)
and ThreadSanitizer.  The driver covers the session state machine (Sec. 3.6, Alg. 1),
Alg. 2's gate while the pre-position is still pending, the idle pass of Sec. 3.1 yielding
to a flag set by another thread, gates racing mutations and session destruction, and the
batched and allocation-free gates, and a gate giving up on a scan still queued.  A last test plants an unsynchronized read of the
yield flag in a copy of the runtime and checks that ThreadSanitizer reports it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STUB = os.path.join(ROOT, "tests", "cpu_runtime")
CSRC = os.path.join(ROOT, "paper_2606_29565_amd", "csrc")
RUNTIME = os.path.join(CSRC, "runtime.cpp")
OTHERS = [os.path.join(STUB, f) for f in ("stub_hip.cpp", "stub_kernels.cpp", "driver.cpp")]
SANITIZERS = {"asan": ["-fsanitize=address,undefined", "-fno-omit-frame-pointer"],
              "tsan": ["-fsanitize=thread"]}

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")


def _build(out, flags, runtime=RUNTIME):
    cmd = ["g++", "-std=c++17", "-O1", "-g", *flags, "-I", STUB,
           "-DSPP_GATE_WAIT_MS=stub::gate_wait_ms",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, runtime, *OTHERS, "-o", out,
           "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]


def _run(exe):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:halt_on_error=1",
               UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1",
               TSAN_OPTIONS="halt_on_error=0:exitcode=66")
    return subprocess.run([exe], capture_output=True, text=True, timeout=600, env=env)


@pytest.mark.parametrize("san", sorted(SANITIZERS))
def test_runtime_scenarios_clean_under_sanitizer(tmp_path, san):
    exe = str(tmp_path / f"driver_{san}")
    _build(exe, SANITIZERS[san])
    r = _run(exe)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), (r.stdout + r.stderr)[-6000:]
    for marker in ("WARNING: ThreadSanitizer", "ERROR: AddressSanitizer", "runtime error:"):
        assert marker not in r.stderr, r.stderr[-6000:]


def test_thread_sanitizer_reports_a_planted_unsynchronized_flag_read(tmp_path):
    src = open(RUNTIME).read()
    acquire = "stop = __atomic_load_n(y.flag, __ATOMIC_ACQUIRE) != 0;"
    assert src.count(acquire) == 2
    planted = tmp_path / "runtime_planted.cpp"
    planted.write_text(src.replace(acquire, "stop = *y.flag != 0;"))
    exe = str(tmp_path / "driver_planted")
    _build(exe, SANITIZERS["tsan"], runtime=str(planted))
    r = _run(exe)
    assert r.returncode == 66 and "WARNING: ThreadSanitizer: data race" in r.stderr
