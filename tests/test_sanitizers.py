"""Host code under AddressSanitizer and UndefinedBehaviorSanitizer (CPU only; GPU code is never
instrumented): the C oracle runs its pins once as a sanitizer build, and the host side of
libtide_route -- argument checks, the prefill plan, the persistent kernels' tile schedule, the
workspace arithmetic -- runs the plan and boundary tests as a sanitizer build of the same sources, and what it
looks up without its lock (the device's number of CUs) is called from several threads at once."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SAN_FLAGS = "-fsanitize=address,undefined -fno-sanitize-recover=undefined -fno-omit-frame-pointer -g -O1"


def _tool_file(tool, name):
    out = subprocess.run([tool, f"-print-file-name={name}"], capture_output=True, text=True).stdout.strip()
    return out if os.path.isabs(out) and os.path.exists(out) else None


def _sanitizer_env(runtime, log_dir, **extra):
    """The sanitizer runtime must be the first library the interpreter loads; whatever is preloaded already stays.
    Reports go to files under log_dir (pytest captures the child's stderr and a report dies with the process)."""
    preload = runtime + (":" + os.environ["LD_PRELOAD"] if os.environ.get("LD_PRELOAD") else "")
    log = os.path.join(str(log_dir), "sanitizer")
    return dict(os.environ, LD_PRELOAD=preload, ASAN_OPTIONS=f"detect_leaks=0:verify_asan_link_order=0:log_path={log}",
                UBSAN_OPTIONS=f"halt_on_error=1:print_stacktrace=1:log_path={log}", PYTHONDONTWRITEBYTECODE="1", **extra)


def _reports(log_dir):
    return "".join(open(os.path.join(str(log_dir), f)).read() for f in sorted(os.listdir(str(log_dir))) if f.startswith("sanitizer"))


def _pytest(files, env, timeout):
    return subprocess.run([sys.executable, "-m", "pytest", "-q", "-x", "-p", "no:cacheprovider", *files], cwd=ROOT, env=env,
                          capture_output=True, text=True, timeout=timeout)


def _clean(run, log_dir):
    text = run.stdout + run.stderr + _reports(log_dir)
    return run.returncode == 0 and "AddressSanitizer" not in text and "runtime error:" not in text


@pytest.fixture(scope="module")
def gcc_asan():
    lib = _tool_file("gcc", "libasan.so")
    if lib is None:
        pytest.skip("gcc's AddressSanitizer runtime is not installed")
    return lib


def _oracle_copy(tmp_path, name):
    parent = tmp_path / name
    shutil.copytree(os.path.join(ROOT, "oracle"), parent / "oracle", ignore=shutil.ignore_patterns("*.so", "__pycache__"))
    return parent


def test_oracle_pins_under_sanitizers(gcc_asan, tmp_path):
    parent = _oracle_copy(tmp_path, "san")
    env = _sanitizer_env(gcc_asan, tmp_path, TIDE_ORACLE_PARENT=str(parent), TIDE_ORACLE_CFLAGS=SAN_FLAGS)
    run = _pytest([os.path.join(ROOT, "tests", "test_oracle_pins.py")], env, 900)
    assert _clean(run, tmp_path), run.stdout[-3000:] + run.stderr[-3000:] + _reports(tmp_path)[-3000:]
    assert (parent / "oracle" / "libtide_oracle.so").exists()          # the instrumented copy is what ran


def test_sanitizer_build_catches_a_planted_overflow(gcc_asan, tmp_path):
    """Control: the same mechanism fails when the oracle copy allocates one element too few for a heap array."""
    parent = _oracle_copy(tmp_path, "ovf")
    src = parent / "oracle" / "tide_oracle.c"
    text = src.read_text()
    site = "double* act = (double*)malloc(sizeof(double) * (size_t)b);"
    assert site in text
    src.write_text(text.replace(site, "double* act = (double*)malloc(sizeof(double) * (size_t)(b - 1));"))
    env = _sanitizer_env(gcc_asan, tmp_path, TIDE_ORACLE_PARENT=str(parent), TIDE_ORACLE_CFLAGS=SAN_FLAGS)
    run = _pytest([os.path.join(ROOT, "tests", "test_oracle_pins.py")], env, 900)
    assert run.returncode != 0 and "heap-buffer-overflow" in _reports(tmp_path), run.stdout[-2000:] + _reports(tmp_path)[-2000:]


def test_host_side_of_the_library_under_sanitizers(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    runtime = _tool_file(hipcc, "libclang_rt.asan-x86_64.so") if os.path.exists(hipcc) else None
    if runtime is None:
        pytest.skip("hipcc or clang's AddressSanitizer runtime is not installed")
    from paper_2603_21365_amd.build import CSRC, HIPCC_FLAGS, INCLUDE
    lib = str(tmp_path / "libtide_route_hostsan.so")
    flags = [f for f in HIPCC_FLAGS if f != "-O3"]
    host_san = []
    for f in ("-fsanitize=address", "-fsanitize=undefined", "-fno-sanitize-recover=undefined"):
        host_san += ["-Xarch_host", f]                               # host pass only: device code stays uninstrumented
    cmd = [hipcc, *flags, "-O1", "-g", *host_san, "-shared-libsan", "-I", INCLUDE, "-o", lib, os.path.join(CSRC, "tide_route.hip")]
    build = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    assert build.returncode == 0, build.stderr[-3000:]
    env = _sanitizer_env(runtime, tmp_path, TIDE_ROUTE_LIB=lib)
    run = _pytest([os.path.join(ROOT, "tests", "test_plan.py"), os.path.join(ROOT, "tests", "test_abi.py")], env, 900)
    assert _clean(run, tmp_path), run.stdout[-3000:] + run.stderr[-3000:] + _reports(tmp_path)[-3000:]
    assert " passed" in run.stdout


_THREADS = r"""
#include <dlfcn.h>
#include <atomic>
#include <cstdint>
#include <cstdio>
#include <thread>
#include <vector>
static thread_local int g_dev = 0;                       // in place of the HIP runtime: a device per thread, no GPU
extern "C" int hipGetDevice(int* d) { *d = g_dev; return 0; }
extern "C" int hipDeviceGetAttribute(int* v, int, int) { *v = 304; return 0; }
int main(int, char** argv) {
    void* lib = dlopen(argv[1], RTLD_NOW);
    if (!lib) { puts(dlerror()); return 3; }
    auto need = (size_t(*)(int, int64_t, int64_t, int64_t, int64_t, int))dlsym(lib, "tide_workspace_bytes");
    for (int first : {3, 40}) {                          // one device's entry; devices beyond the table
        std::atomic<int> ready{0};
        std::vector<size_t> got(8);
        std::vector<std::thread> threads;
        for (int i = 0; i < 8; ++i)
            threads.emplace_back([&, i] {
                g_dev = first;
                ready.fetch_add(1, std::memory_order_relaxed);
                while (ready.load(std::memory_order_relaxed) < 8) std::this_thread::yield();
                got[i] = need(2, 8, 100, 4096, 128, 0);
            });
        for (auto& t : threads) t.join();
        for (size_t g : got)
            if (g != got[0] || g == 0) { printf("%zu\n", g); return 4; }
    }
    puts("same answer");
}
"""


def test_first_calls_from_several_threads(tmp_path):
    """The number of CUs is cached per device and read without the library's lock (by the exit projection, which needs no
    workspace and runs on any device index, and by tide_workspace_bytes): no race on it, no index beyond the cache."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    clang = "/opt/rocm/lib/llvm/bin/clang++"
    runtime = _tool_file(clang, "libclang_rt.tsan-x86_64.so") if os.path.exists(hipcc) and os.path.exists(clang) else None
    if runtime is None:
        pytest.skip("hipcc or clang's ThreadSanitizer runtime is not installed")
    from paper_2603_21365_amd.build import CSRC, HIPCC_FLAGS, INCLUDE
    lib, driver, source = (str(tmp_path / n) for n in ("libtide_route_tsan.so", "threads", "threads.cpp"))
    with open(source, "w") as f:
        f.write(_THREADS)
    host_san = []
    for f in ("-fsanitize=thread", "-fsanitize=bounds", "-fno-sanitize-recover=bounds"):
        host_san += ["-Xarch_host", f]                               # host pass only
    builds = ([hipcc, *[f for f in HIPCC_FLAGS if f != "-O3"], "-O1", "-g", *host_san, "-shared-libsan", "-I", INCLUDE, "-o", lib, os.path.join(CSRC, "tide_route.hip")],
              [clang, "-std=c++17", "-O1", "-g", "-fsanitize=thread", "-shared-libsan", "-rdynamic", "-o", driver, source, "-ldl", "-pthread"])
    for cmd in builds:
        build = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
        assert build.returncode == 0, build.stderr[-3000:]
    run = subprocess.run([driver, lib], capture_output=True, text=True, timeout=300,
                         env=dict(os.environ, LD_LIBRARY_PATH=os.path.dirname(runtime) + ":" + os.environ.get("LD_LIBRARY_PATH", "")))
    text = run.stdout + run.stderr
    assert run.returncode == 0 and "ThreadSanitizer" not in text and "same answer" in text, text[-3000:]
