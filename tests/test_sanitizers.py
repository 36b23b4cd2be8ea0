"""Host code under AddressSanitizer and UndefinedBehaviorSanitizer (CPU only, no GPU code is
instrumented): the C oracle, and the library's host side (dictionary, encoder, validation,
argument checks, launch planning).  Each leg builds a sanitized copy and re-runs the existing
host tests against it in a child process that preloads the sanitizer's runtime; any report
makes the child exit non-zero.  The host encoder's threads run under ThreadSanitizer, too, in a program of their own.
"""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2310_16795_amd", "csrc")


def _run_child(files, env_extra, preload):
    env = dict(os.environ)
    env.update(env_extra)
    env["LD_PRELOAD"] = " ".join(x for x in (env.get("LD_PRELOAD"), preload) if x)
    env["ASAN_OPTIONS"] = "detect_leaks=0:verify_asan_link_order=0:abort_on_error=0:exitcode=23"
    env["UBSAN_OPTIONS"] = "halt_on_error=1:print_stacktrace=1:exitcode=23"
    cmd = [sys.executable, "-m", "pytest", "-x", "-q", "-m", "not gpu", "-p", "no:cacheprovider", *files]
    r = subprocess.run(cmd, cwd=ROOT, env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-4000:]
    assert "passed" in r.stdout


def test_oracle_under_asan_and_ubsan():
    rt = subprocess.check_output(["gcc", "-print-file-name=libasan.so"], text=True).strip()
    if not os.path.isabs(rt) or not os.path.exists(rt):
        pytest.skip("gcc's libasan is not installed")
    env = {"ORACLE_SANITIZE": "1"}
    subprocess.check_call([sys.executable, "-c", "import oracle; oracle.build()"], cwd=ROOT, env={**os.environ, **env})
    _run_child(["tests/test_oracle_codec.py", "tests/test_oracle_dictionary.py", "tests/test_oracle_matvec.py"], env, rt)


def test_library_host_side_under_asan_and_ubsan():
    from paper_2310_16795_amd import build as B

    cands = []
    for base, _, files in os.walk("/opt/rocm/lib/llvm/lib/clang"):
        cands += [os.path.join(base, f) for f in files if f == "libclang_rt.asan-x86_64.so"]
    if not cands:
        pytest.skip("clang's shared ASan runtime is not installed")
    B.build_library(incremental=True)  # the device objects the sanitized host objects are linked with
    san = os.path.join(B.OBJ, "san")
    os.makedirs(san, exist_ok=True)
    host_flags = ["-O1", "-g", "-std=c++17", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    subprocess.check_call(["hipcc", *host_flags, "-fsanitize=address", "-fsanitize=undefined",
                           "-fno-sanitize-recover=undefined", "-fno-gpu-sanitize",
                           "-c", os.path.join(CSRC, "qmoe_host.cpp"), "-o", os.path.join(san, "qmoe_host.o")])
    subprocess.check_call(["hipcc", *host_flags, "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                           "-packed-fp32-ops", "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                           "-Xarch_host", "-fno-sanitize-recover=undefined",
                           "-c", os.path.join(CSRC, "qmoe_api.hip"), "-o", os.path.join(san, "qmoe_api.o")],
                          stderr=subprocess.DEVNULL)
    others = [os.path.join(B.OBJ, os.path.splitext(u)[0] + ".o") for u in B.UNITS
              if u not in ("qmoe_host.cpp", "qmoe_api.hip")]
    lib = os.path.join(san, "libqmoe_san.so")
    subprocess.check_call(["hipcc", "-shared", "-fPIC", "--offload-arch=gfx950", "-fsanitize=address",
                           "-fsanitize=undefined", "-shared-libsan", "-fno-gpu-sanitize", "-o", lib,
                           os.path.join(san, "qmoe_host.o"), os.path.join(san, "qmoe_api.o"), *others])
    _run_child(["tests/test_lib_host.py"], {"QMOE_LIBRARY": lib}, cands[0])


ENCODER_THREADS = r"""
#include <cstdio>
#include <cstring>
#include <vector>
#include "qmoe.h"

static int fail(const char *what, int rows, int threads)
{
    std::printf("%s: %d rows, %d threads\n", what, rows, threads);
    return 1;
}

int main()
{
    qmoe_dict *full, *small;  // (the small one lacks the pair -1 -1)
    if (qmoe_dict_create(0.885, 14, 65536, &full) || qmoe_dict_create(0.5, 1, 8, &small)) return 1;
    const int cols = 66;
    for (int rows : {1, 70, 1029})
        for (int kind = 0; kind < 5; kind++) {  // streams of both dictionaries, a bad symbol, a buffer that is too small, a size only
            const qmoe_dict *d = kind == 1 ? small : full;
            std::vector<int8_t> t((size_t)rows * cols);
            uint32_t state = 12345u + (uint32_t)rows;
            for (size_t i = 0; i < t.size(); i += 2) {
                state = state * 1664525u + 1013904223u;
                t[i] = state >> 28 == 0 ? 1 : state >> 28 == 1 ? -1 : 0;
            }
            if (kind == 2) t[t.size() / 2] = 2;
            std::vector<uint16_t> one(t.size()), out(t.size());
            std::vector<uint32_t> one_off(rows + 1), off(rows + 1);
            size_t one_n = 0, n = 0;
            qmoe_set_tuning("host_threads", 1);
            const int want = qmoe_encode_host(d, t.data(), rows, cols, kind == 4 ? nullptr : one.data(), kind == 3 ? 1 : one.size(), one_off.data(), &one_n);
            if (want != (kind == 2 ? QMOE_E_BAD_SYMBOL : kind == 3 ? QMOE_E_BUFFER_TOO_SMALL : QMOE_OK)) return fail("status", rows, 1);
            for (int threads : {2, 5, 16})
                for (int again = 0; again < 5; again++) {
                    qmoe_set_tuning("host_threads", threads);
                    if (qmoe_encode_host(d, t.data(), rows, cols, kind == 4 ? nullptr : out.data(), kind == 3 ? 1 : out.size(), off.data(), &n) != want)
                        return fail("status", rows, threads);
                    if (want == QMOE_OK && (n != one_n || off != one_off || (kind != 4 && std::memcmp(out.data(), one.data(), 2 * n) != 0)))
                        return fail("stream", rows, threads);
                }
        }
    qmoe_dict_destroy(full);
    qmoe_dict_destroy(small);
    std::puts("done");
    return 0;
}
"""


def test_host_encoder_threads_under_tsan(tmp_path):
    rt = subprocess.check_output(["g++", "-print-file-name=libtsan.so"], text=True).strip()
    if not os.path.isabs(rt) or not os.path.exists(rt):
        pytest.skip("gcc's libtsan is not installed")
    (tmp_path / "threads.cpp").write_text(ENCODER_THREADS)
    program = str(tmp_path / "threads")
    subprocess.check_call(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=thread", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                           str(tmp_path / "threads.cpp"), os.path.join(CSRC, "qmoe_host.cpp"), "-o", program, "-lpthread"])
    r = subprocess.run([program], env={**os.environ, "TSAN_OPTIONS": "exitcode=23:halt_on_error=1"}, stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.rstrip().endswith("done"), r.stdout[-4000:]
