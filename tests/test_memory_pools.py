"""The library's device-memory code on the CPU: api.hip as host C++ with a counted heap in place of
the device (tests/memory/driver.cpp), under the address sanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("memory") / "driver")
    cmd = ["g++", "-std=c++17", "-g", "-O1", "-fsanitize=address", "-no-pie", "-w",
           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           os.path.join(ROOT, "tests", "memory", "driver.cpp"), "-o", exe,
           "-Wl,--unresolved-symbols=ignore-all", "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def _run(driver, what):
    r = subprocess.run([driver, what], capture_output=True, text=True, timeout=20,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0 and r.stdout == "ok\n", (r.stdout + r.stderr)[-3000:]


@pytest.mark.parametrize("what", ["refusal", "hook_refusal"])
def test_idle_memory_goes_back_before_a_refusal(driver, what):
    _run(driver, what)


@pytest.mark.parametrize("what", ["no_host_memory", "idle_at_exit"])
def test_idle_checkpoints(driver, what):
    _run(driver, what)


def test_full_lists_follow_the_sizes_in_use(driver):
    _run(driver, "full_lists")


def test_failed_calls_give_nothing_back_that_is_in_use(driver):
    _run(driver, "failed_call")


def test_trim_gives_everything_back(driver):
    _run(driver, "trim")
