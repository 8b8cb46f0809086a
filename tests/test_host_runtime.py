"""The library's host runtime without a GPU: paths that an ordinary run does not
take (a failed allocation, a reused address, a second thread), in a host build
against a stand-in HIP runtime (host/runtime_test.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")


@pytest.fixture(scope="module")
def build(tmp_path_factory):
    """Path of the test program built with extra compiler flags."""
    out = tmp_path_factory.mktemp("host")
    built = {}

    def get(*flags):
        if flags not in built:
            exe = str(out / ("runtime_test%d" % len(built)))
            cmd = ["g++", "-std=c++17", "-O1", "-g", "-w", "-pthread", *flags, "-I", HERE,
                   os.path.join(HERE, "runtime_test.cpp"), "-o", exe]
            r = subprocess.run(cmd, capture_output=True, text=True)
            assert r.returncode == 0, r.stdout + r.stderr
            built[flags] = exe
        return built[flags]
    return get


def _run(exe, name):
    r = subprocess.run([exe, name], capture_output=True, text=True, timeout=120)
    if r.returncode == 77 or "unexpected memory mapping" in r.stderr:  # (the latter: no room for the sanitizer)
        pytest.skip("%s does not apply here" % name)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("name", [
    "captured_search_of_a_released_peakmap",
    "allocation_after_trimming",
    "search_after_a_failed_allocation",
    "search_without_room_for_optional_buffers",
    "kept_memory_makes_room",
    "request_in_a_tight_budget",
    "peakmap_released_during_a_capture",
    "forced_tile_parts",
    "spectra_without_pinned_memory",
    "search_after_a_refused_call",
    "option_changed_behind_a_queued_request",
])
def test_host_runtime(build, name):
    _run(build(), name)


def test_host_runtime_threads(build):
    _run(build("-fsanitize=thread"), "peakmaps_released_on_another_thread")
