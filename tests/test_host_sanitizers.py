"""The host runtime (paper_1712_06139_amd/csrc/runtime.cpp) built for its
host-only paths with the compiler's sanitizers and driven through the C ABI
without a GPU (tests/sanitize/host_paths.cpp): address and undefined-behaviour
checks over model and queue life cycles, trace replays with launch windows,
the serving calls, version transitions and queues replaced while serving;
thread checks over models created and destroyed on loader threads while the
main thread serves and swaps them in. The device runtime and the kernels are
replaced by stand-ins that stop the program if a host-only path reaches them
(tests/sanitize/hip_absent.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = [os.path.join(ROOT, "paper_1712_06139_amd", "csrc", "runtime.cpp"),
       os.path.join(ROOT, "tests", "sanitize", "hip_absent.cpp"),
       os.path.join(ROOT, "tests", "sanitize", "host_paths.cpp")]
FLAGS = ["-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__",
         "-I/opt/rocm/include", f"-I{os.path.join(ROOT, 'include')}"]

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                                reason="needs g++ and the HIP headers")


def _build_and_run(tmp_path, sanitize, args):
    exe = str(tmp_path / "host_paths")
    subprocess.run(["g++", *FLAGS, *sanitize, *SRC, "-o", exe, "-lpthread"], check=True, capture_output=True,
                   timeout=300)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=1", UBSAN_OPTIONS="halt_on_error=1",
               TSAN_OPTIONS="halt_on_error=1")
    r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "host paths ok" in r.stdout
    return r.stdout


def test_host_runtime_under_address_and_undefined_behaviour_sanitizers(tmp_path):
    out = _build_and_run(tmp_path, ["-fsanitize=address,undefined", "-fno-sanitize-recover=undefined"], [])
    print(out)


def test_host_runtime_loader_threads_under_thread_sanitizer(tmp_path):
    out = _build_and_run(tmp_path, ["-fsanitize=thread"], ["--threads"])
    print(out)


def test_runtime_links_only_with_every_kernel_launcher(tmp_path):
    # no reference of the runtime to a kernel launcher is weak (a missing one
    # would then load as a call of address 0), and the stand-ins cover them all
    syms = {}
    for src in SRC[:2]:
        obj = str(tmp_path / (os.path.basename(src) + ".o"))
        subprocess.run(["g++", *FLAGS, "-c", src, "-o", obj], check=True, capture_output=True, timeout=300)
        out = subprocess.run(["nm", "-C", obj], check=True, capture_output=True, text=True).stdout
        syms[src] = [line[17:].split(" ", 1) for line in out.splitlines()]
    names = {t: {n for k, n in syms[SRC[0]] if k == t and n.startswith("rb_")} for t in "Uwv"}
    assert not names["w"] and not names["v"]
    assert any(n.startswith("rb_gemm_f32_split(") for n in names["U"]) and "rb_route_bags" in names["U"]
    assert names["U"] <= {n for k, n in syms[SRC[1]] if k == "T"}
