"""The library's host runtime on a HIP runtime of host memory: what it
uploads, which layouts and kernels it launches with, and what a failing
allocation leaves behind, with the address and undefined-behaviour sanitizers
on (no device; scenarios in native/host_scenarios.py)."""
import concurrent.futures as cf
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1601_00221_amd", "csrc")
SOURCES = [os.path.join(CSRC, s) for s in
           ("lower.cpp", "runtime.cpp", "batch.cpp", "serve.cpp", "core_host.cpp", "evolve.cpp", "blockgp.cpp")]
SOURCES.append(os.path.join(HERE, "native", "fake_hip.cpp"))
SAN = ["-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-fno-omit-frame-pointer"]


def _runtime(name):
    p = subprocess.run(["gcc", "-print-file-name=" + name], capture_output=True, text=True).stdout.strip()
    return p if os.path.isabs(p) and os.path.exists(p) else None


pytestmark = pytest.mark.skipif(not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h") or
                                _runtime("libasan.so") is None,
                                reason="needs the HIP headers and the gcc sanitizer runtimes")


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_runtime")
    sys.path.insert(0, CSRC)
    import gen_core
    gen_core.main(str(d / "gen"))
    flags = ["-std=c++17", "-O1", "-g", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-D__device__=", "-D__forceinline__=inline",
             "-I/opt/rocm/include", "-I%s" % (d / "gen"), "-I" + CSRC, "-I" + os.path.join(ROOT, "include")] + SAN

    def compile_one(src):
        o = str(d / (os.path.basename(src) + ".o"))
        count = ["-Dlower_tree=real_lower_tree", "-Dneeded_linear=real_needed_linear"] if src.endswith("lower.cpp") else []
        subprocess.run(["g++", *flags, *count, "-c", src, "-o", o], check=True)
        return o
    with cf.ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    lib = str(d / "libgp_host.so")
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", *SAN, "-o", lib, *objs, "-lpthread"], check=True)
    return lib


def run(library, scenario, *args, **env):
    e = dict(os.environ, **env)
    pre = [p for p in (_runtime("libasan.so"), _runtime("libubsan.so"), e.get("LD_PRELOAD")) if p]
    e["LD_PRELOAD"] = " ".join(pre)
    e["ASAN_OPTIONS"] = "detect_leaks=0:abort_on_error=0:exitcode=23"
    e["UBSAN_OPTIONS"] = "halt_on_error=1:print_stacktrace=1:exitcode=24"
    r = subprocess.run([sys.executable, os.path.join(HERE, "native", "host_scenarios.py"), library, scenario, *args],
                       env=e, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), (r.returncode, r.stdout[-2000:], r.stderr[-4000:])
    return r.stdout.split()


def test_failed_allocation_leaves_no_layout(library):
    run(library, "failed_allocation_leaves_no_layout")


def test_a_batch_is_lowered_once(library, tmp_path):
    run(library, "batch_is_lowered_once")
    # the same where configurations of other shapes are stored
    cache = tmp_path / "tuned.json"
    cache.write_text('{\n"d7x1;j0,0,1,1,1,1;": [0, 8, 1]\n}\n')
    run(library, "batch_is_lowered_once", GP2D_TUNE_CACHE=str(cache))


def test_stored_configurations_go_by_kernel_name(library, tmp_path):
    cache = tmp_path / "tuned.json"
    env = {"GP2D_TUNE_CACHE": str(cache)}
    default = run(library, "evaluated_with", "-")[0]
    kernel, number = run(library, "tune", **env)[:2]
    stored = cache.read_text()
    assert '["%s", ' % kernel in stored and kernel != default
    run(library, "evaluated_with", kernel, **env)
    # a file of an earlier release: the kernel's number
    cache.write_text(stored.replace('"%s"' % kernel, number))
    run(library, "evaluated_with", kernel, **env)
    # kernels that do not exist, or cannot hold the batch (trees only; no sin/cos/exp/log; Boolean): the default
    for other in ('"k_core_9_9_9_9"', '"k_core_4_8_8_64_t"', '"k_core_8_6_8_40_a"', '"k_core_4_6_20_16_b"', "16", "22", "-1",
                  "4000"):
        cache.write_text(stored.replace('"%s"' % kernel, other))
        run(library, "evaluated_with", default, **env)


@pytest.mark.parametrize("launch,table,copy,table_kept", [(1, 3, 0, 0), (2, 3, 0, 1), (0.5, 3, 1, 0), (0.5, 1.5, 1, 0),
                                                          (4, 3, 1, 1)])
def test_tuning_compares_whole_calls(library, launch, table, copy, table_kept):
    run(library, "tuning_keeps_the_faster", *(str(x) for x in (launch, table, copy, table_kept)))


def test_every_evaluation_takes_the_translation_that_suits_it(library):
    run(library, "every_evaluation_takes_the_translation_that_suits_it")


def test_tuning_does_without_the_default(library):
    run(library, "tuning_does_without_the_default")
