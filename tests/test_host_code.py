"""Host code of libhyperim.so on the CPU, over a stand-in HIP runtime
(tests/host): which stream the shared workspaces belong to, and what a call
leaves behind when memory runs out."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host")
LIB_DIR = os.path.join(ROOT, "paper_2406_01911_amd")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    lib = os.path.join(LIB_DIR, "libhyperim.so")
    if not os.path.exists(lib):
        from paper_2406_01911_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("host") / "driver")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.check_call(["g++", "-O1", "-g", "-std=c++17", "-pthread", "-rdynamic", "-D__HIP_PLATFORM_AMD__=1",
                           "-isystem", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"),
                           os.path.join(HERE, "driver.cpp"), os.path.join(HERE, "fake_hip.cpp"), lib, "-o", exe,
                           "-Wl,-rpath," + LIB_DIR, "-Wl,-rpath-link," + os.path.join(rocm, "lib")])
    return exe


def _run(exe, scenario):
    r = subprocess.run([exe, scenario], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok "), r.stdout[-2000:]


def test_workspace_belongs_to_one_stream_at_a_time(driver):
    _run(driver, "streams")


def test_workspace_after_memory_ran_out(driver):
    _run(driver, "workspace_nomem")


def test_pool_after_memory_ran_out(driver):
    _run(driver, "pool_nomem")


def test_layer_tables_after_memory_ran_out(driver):
    _run(driver, "tables_nomem")


def test_small_graph_within_a_small_budget(driver):
    _run(driver, "small_budget")


def test_freed_blocks(driver):
    _run(driver, "blocks")


def test_work_that_does_not_finish(driver):
    _run(driver, "wait_limit")
