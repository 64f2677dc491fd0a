"""The host side of the library under AddressSanitizer and UndefinedBehaviorSanitizer: tests/host_sanitize_driver.cpp
is built with the library's sources into one executable whose host code is instrumented (__graft_entry__.
build_sanitize_driver; device code is not instrumented) and exercises the C ABI directly.  Without a GPU it runs the
argument checks and host-only routines of every entry point; with one, every kind of call on tiny random models.
A sanitizer report aborts the run, a failed check makes the exit status 1."""
import os
import subprocess

import pytest

import __graft_entry__ as entry

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCES = [os.path.join(ROOT, "paper_2407_19947_amd", "csrc", n) for n in
           ("stairs_kernels.hip", "stairs_block.hip", "stairs_api.hip", "stairs_kernels.h", "stairs_device.h")] + \
          [os.path.join(ROOT, "include", "stairs.h"), entry.SANITIZE_DRIVER + ".cpp"]
ENV = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1")


def _build_if_stale():
    exe = entry.SANITIZE_DRIVER
    if not os.path.exists(exe) or any(os.path.getmtime(s) > os.path.getmtime(exe) for s in SOURCES):
        entry.build_sanitize_driver()


def _run(timeout):
    res = subprocess.run([entry.SANITIZE_DRIVER], capture_output=True, text=True, env=ENV, timeout=timeout)
    print(res.stdout[-2000:], res.stderr[-6000:], flush=True)
    return res


def test_argument_checks_under_host_sanitizers():
    """No GPU: (re)build the instrumented driver when it is missing or older than a source, run part 1."""
    _build_if_stale()
    res = _run(120)
    assert res.returncode == 0
    assert "part 1 (no GPU): 0 failed checks" in res.stdout


@pytest.mark.parametrize("forced,qkv,down", [
    (None, "3/4 3/4 3/4 3/4 shared shared shared", "split split shared shared shared shared shared"),
    ("2/3", "2/3 2/3 2/3 2/3 2/3 2/3 1/3", "2/3 2/3 2/3 2/3 2/3 2/3 1/3"),
    ("0/5", "split split split split 1/8 1/8 1/8", "split split split split 1/8 1/8 1/8"),
])
def test_forced_launch_shapes_reach_every_row_count(forced, qkv, down):
    """STAIRS_WIDE_CFG sends projections of 8, 16, 17, 32, 33, 48 and 64 rows to the fragment-reading GEMM with its tiles per wave
    and waves, whichever kernel they take without it (768 tiles, 8 chunks; 256 tiles, 22 chunks).  Beyond 32 rows a wave has at
    most two tiles, beyond 48 one, and there is no split-K (0)."""
    _build_if_stale()
    env = dict(ENV)
    env.pop("STAIRS_WIDE_CFG", None)
    if forced:
        env["STAIRS_WIDE_CFG"] = ",".join([forced] * 5)
    out = subprocess.run([entry.SANITIZE_DRIVER, "wide-cfg"], capture_output=True, text=True, env=env, timeout=60).stdout
    assert out.split("\n")[:-1] == ["768 x 4096: " + qkv, "256 x 11008: " + down]


@pytest.mark.parametrize("limit,want", [(None, 7), ("4", 4), ("2", 2)])
def test_row_limit_of_the_lds_resident_gemm(limit, want):
    """STAIRS_ROWS_MAX limits the rows of the GEMM with the activations in LDS for every projection: few tiles and many with a
    short k, a long k."""
    _build_if_stale()
    env = dict(ENV)
    env.pop("STAIRS_ROWS_MAX", None)
    if limit:
        env["STAIRS_ROWS_MAX"] = limit
    out = subprocess.run([entry.SANITIZE_DRIVER, "rows-max"], capture_output=True, text=True, env=env, timeout=60).stdout
    assert out.split("\n")[:-1] == [f"{shape}: {want}" for shape in ("2304 x 768", "32000 x 1024", "22016 x 4096")]


@pytest.mark.gpu
def test_every_kind_of_call_under_host_sanitizers():
    """GPU: the prebuilt driver (built on the CPU beforehand, never here) through prefill, generation, batches,
    sampling, end token, encoder-decoder and the diagnostics."""
    if not os.path.exists(entry.SANITIZE_DRIVER):
        pytest.skip("instrumented driver not built (python -c 'import __graft_entry__ as g; g.build()' builds it)")
    res = _run(300)
    assert res.returncode == 0
    assert "part 2 (encoder-decoder): 0 failed checks in all" in res.stdout
