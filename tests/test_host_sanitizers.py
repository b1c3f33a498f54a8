"""The library's host code (validation, grouping, planner, scheduler) and the oracle
built with AddressSanitizer and UndefinedBehaviorSanitizer, exercised on
random batches by tests/sanitize/host_check.cpp, and the plan calls against a
stand-in HIP runtime by tests/sanitize/plan_calls.cpp.  CPU only: nothing is
launched on a GPU (the device code is compiled as usual and never run)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2401_11240_amd", "csrc")
SAN = os.path.join(ROOT, "tests", "sanitize")
CLANG = "/opt/rocm/llvm/bin/clang"
CLANGXX = "/opt/rocm/llvm/bin/clang++"
HIPCC = "/opt/rocm/bin/hipcc"


SANITIZE = ["-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-fno-omit-frame-pointer"]

pytestmark = pytest.mark.skipif(not all(os.path.exists(c) for c in (HIPCC, CLANG, CLANGXX)),
                                reason="ROCm compilers missing")


def hip_object(src, out):
    """A HIP source with the sanitizers on its host side only."""
    from paper_2401_11240_amd import build as B
    host_san = []
    for f in SANITIZE:
        host_san += ["-Xarch_host", f]
    res = subprocess.run([HIPCC, "-x", "hip", f"--offload-arch={B.ARCH}", "-O1", "-g", "-std=c++17", "-c",
                          f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}"] + B.DEVICE_FLAGS + host_san +
                         [src, "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    return out


def link_and_run(objs, exe):
    res = subprocess.run([CLANGXX] + SANITIZE + objs + ["-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib", "-lamdhip64",
                                                        "-o", exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1",
               UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1")
    run = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=600)
    assert run.returncode == 0, (run.stdout[-2000:], run.stderr[-6000:])
    assert "all checks passed" in run.stdout


@pytest.fixture(scope="module")
def api_object(tmp_path_factory):
    return hip_object(os.path.join(CSRC, "lora_api.hip"), str(tmp_path_factory.mktemp("api") / "lora_api.o"))


def test_planner_and_oracle_under_asan_ubsan(tmp_path, api_object):
    # the library's host code and the driver, which stands in for the launch functions
    objs = [api_object, hip_object(os.path.join(SAN, "host_check.cpp"), str(tmp_path / "host_check.o"))]
    # the oracle: plain C, no OpenMP here (its pragmas are then ignored)
    objs.append(str(tmp_path / "oracle.o"))
    subprocess.run([CLANG, "-c", "-O1", "-g", "-std=c11", "-ffp-contract=off"] + SANITIZE +
                   [os.path.join(ROOT, "oracle", "lora_oracle.c"), "-o", objs[-1]], check=True)
    # the scheduler and the CPU LoRA kernel: plain C++
    for src in ("lora_sched.cpp", "lora_cpu.cpp"):
        objs.append(str(tmp_path / (src + ".o")))
        res = subprocess.run([CLANGXX, "-c", "-O1", "-g", "-std=c++17", f"-I{os.path.join(ROOT, 'include')}"] +
                             SANITIZE + [os.path.join(CSRC, src), "-o", objs[-1]], capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-4000:]
    link_and_run(objs, str(tmp_path / "host_check"))


def test_plan_calls_on_a_stand_in_runtime(tmp_path, api_object):
    objs = [api_object, hip_object(os.path.join(SAN, "plan_calls.cpp"), str(tmp_path / "plan_calls.o"))]
    link_and_run(objs, str(tmp_path / "plan_calls"))
