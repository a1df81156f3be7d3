"""Host code of libvgicp.so on a HIP runtime of host memory (tests/host_runtime/driver.cpp): ownership
of the device blocks that outlive a call, refused allocations, devices, threads. CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2202_00242_amd")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(os.path.join(PKG, "libvgicp.so")):
        from paper_2202_00242_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("host_runtime") / "driver")
    src = os.path.join(ROOT, "tests", "host_runtime", "driver.cpp")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-rdynamic", "-pthread", "-o", exe, src,
                        f"-L{PKG}", "-l:libvgicp.so", f"-Wl,-rpath,{PKG}",
                        "-Wl,--allow-shlib-undefined"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def run(driver, name, **env):
    r = subprocess.run([driver, name], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, **env))
    assert r.returncode == 0 and f"{name} ok" in r.stdout, (r.returncode, r.stdout + r.stderr)


def test_refused_allocation_fails_its_own_call_only(driver):
    run(driver, "refusal_is_forgotten")


def test_refused_schedule_leaves_the_batch_as_it_was(driver):
    run(driver, "schedule_refused")


def test_batch_calls_with_another_device_current(driver):
    run(driver, "other_device_current")


def test_memory_of_ordering_small_clouds_beside_large_ones(driver):
    run(driver, "order_memory")


def test_workspace_checks(driver):
    run(driver, "workspace_checks")


def test_kept_blocks_of_many_threads_are_bounded_and_released(driver):
    run(driver, "threads")


def test_memory_that_was_not_waited_for_is_not_kept(driver):
    run(driver, "refused_waits")


def test_copies_of_a_refused_call_are_over_when_it_returns(driver):
    run(driver, "copies_of_a_refused_call")


def test_autotune_times_each_launch_once(driver, tmp_path):
    run(driver, "tuned_once", VGICP_AUTOTUNE_LOG=str(tmp_path / "log"))
