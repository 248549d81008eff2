"""Host code under AddressSanitizer and UndefinedBehaviorSanitizer (CPU only).

Two drivers, built here with the sanitizers and -fno-sanitize-recover
and run in child processes:
  * tests/sanitize/oracle_driver.c with oracle/gt_oracle.c and synth/synth.c
    (gcc, no OpenMP): every generator and every oracle function on small
    graphs with empty rows, repeated entries, a single row and row subsets;
  * tests/sanitize/abi_driver.cpp with the library source (hipcc, sanitizers
    on the host compilation only): every entry point's host validation,
    status strings, per-thread error messages, and the pool and profiler
    calls that need no device.
A third run takes the stand-alone C program of the GPU tests (tests/c_caller_gpu.c)
and the library's host code through the program's whole call sequence, release
and process exit included, over tests/sanitize/hip_stub.cpp: a runtime whose
device memory is host memory of the exact size, whose kernels do nothing and
whose handles are checked against a second free or destroy.
Builds are kept under _build/sanitize/, keyed by a hash of their sources."""
import hashlib
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "_build", "sanitize")
SAN = os.path.join(ROOT, "tests", "sanitize")


def cached_build(name, sources, cmd_of):
    h = hashlib.sha256()
    for src in sources:
        h.update(open(src, "rb").read())
    h.update(" ".join(cmd_of("X")).encode())
    exe = os.path.join(BUILD, "%s-%s" % (name, h.hexdigest()[:12]))
    if not os.path.exists(exe):
        os.makedirs(BUILD, exist_ok=True)
        tmp = exe + ".tmp%d" % os.getpid()
        r = subprocess.run(cmd_of(tmp), capture_output=True, text=True, timeout=900)
        if r.returncode != 0:
            raise AssertionError("build failed:\n" + (r.stdout + r.stderr)[-4000:])
        os.replace(tmp, exe)
    return exe


def run_clean(exe):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0",
               UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env)
    out = r.stdout + r.stderr
    assert r.returncode == 0, out[-4000:]
    assert "runtime error" not in out and "AddressSanitizer" not in out, out[-4000:]
    assert "0 failure(s)" in out


def test_oracle_and_generator_under_asan_ubsan():
    if not shutil.which("gcc"):
        pytest.skip("gcc not available")
    srcs = [os.path.join(SAN, "oracle_driver.c"), os.path.join(ROOT, "oracle", "gt_oracle.c"),
            os.path.join(ROOT, "synth", "synth.c")]
    exe = cached_build("oracle_driver", srcs, lambda out: [
        "gcc", "-O1", "-g", "-std=c11", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
        "-fno-sanitize-recover=all"] + srcs + ["-lm", "-o", out])
    run_clean(exe)


def test_library_host_code_under_asan_ubsan():
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    csrc = os.path.join(ROOT, "paper_2605_31500_amd", "csrc")
    srcs = [os.path.join(csrc, n) for n in sorted(os.listdir(csrc)) if n.endswith((".hip", ".hpp"))]
    srcs += [os.path.join(ROOT, "include", "gt_attn.h"), os.path.join(SAN, "abi_driver.cpp")]
    exe = cached_build("abi_driver", srcs, lambda out: [
        hipcc, "--offload-arch=gfx950", "-O0", "-std=c++17",
        "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
        "-Xarch_host", "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"),
        os.path.join(csrc, "gt_attn.hip"), os.path.join(SAN, "abi_driver.cpp"), "-o", out])
    run_clean(exe)


def test_c_program_host_side_under_asan(tmp_path):
    llvm = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "lib", "llvm", "bin")
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    if not os.path.exists(hipcc) or not os.path.exists(os.path.join(llvm, "clang")):
        pytest.skip("hipcc not available")
    rocm_inc = ["-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"),
                "-I", os.path.join(ROOT, "include")]
    csrc = os.path.join(ROOT, "paper_2605_31500_amd", "csrc", "gt_attn.hip")

    def run(cmd):
        r = subprocess.run(cmd, capture_output=True, text=True, timeout=900, cwd=tmp_path)
        assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
        return r.stdout

    asan = ["-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address"]
    run([hipcc, "--offload-arch=gfx950", "--offload-host-only", "-O1", "-g", "-std=c++17",
         "-Xarch_host", "-fsanitize=address", "-I", os.path.join(ROOT, "include"), "-c", csrc, "-o", "lib.o"])
    run([os.path.join(llvm, "clang++"), "-std=c++17"] + asan + rocm_inc + ["-c", os.path.join(SAN, "hip_stub.cpp"), "-o", "stub.o"])
    for src, obj in ((os.path.join(ROOT, "tests", "c_caller_gpu.c"), "prog.o"),
                     (os.path.join(ROOT, "oracle", "gt_oracle.c"), "oracle.o")):
        run([os.path.join(llvm, "clang"), "-std=gnu11"] + asan + rocm_inc + ["-c", src, "-o", obj])
    # (the device code's image, which a host-only compilation leaves out)
    image = [l.split()[-1] for l in run(["nm", "lib.o"]).splitlines() if "__hip_fatbin_" in l and " U " in l and "wrapper" not in l]
    run([os.path.join(llvm, "clang++"), "-fsanitize=address", "lib.o", "stub.o", "prog.o", "oracle.o", "-lm", "-lpthread",
         "-o", "prog"] + ["-Wl,--defsym=%s=0" % s for s in image])
    r = subprocess.run([str(tmp_path / "prog")], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=1"))
    out = r.stdout + r.stderr
    # the four calls return, no kernel has run (their outputs are as they were: NaN), the release and the exit are clean
    assert r.returncode == 1 and out.count("gate error nan") == 4, out[-4000:]
    # (the scratch array stays)
    assert "AddressSanitizer" not in out and re.search(r"hip stub: [1-9]\d* launches, 1 allocations left", out), out[-4000:]
