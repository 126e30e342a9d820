"""The pointer tables of a plan on several streams and threads, on the CPU: kt_api.cpp built against a stand-in
for the HIP runtime (host/fake_hip.h) that runs whatever is not ordered in the worst order, with
AddressSanitizer and UBSan."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_10183_amd", "csrc")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include/hip"),
                                reason="needs g++ and the HIP headers")


def build(out, *flags):
    subprocess.check_call(
        ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan",
         "-static-libubsan", *flags, "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
         os.path.join(ROOT, "tests", "host", "pointer_tables.cpp"), os.path.join(CSRC, "kt_api.cpp"),
         os.path.join(CSRC, "kt_plan.cpp"), "-rdynamic", "-ldl", "-pthread", "-o", out])
    return out


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    """With the runtime's ids of streams."""
    return build(str(tmp_path_factory.mktemp("tables") / "pointer_tables"), "-DFAKE_STREAM_IDS")


@pytest.fixture(scope="module")
def exe_no_ids(tmp_path_factory):
    return build(str(tmp_path_factory.mktemp("tables_no_ids") / "pointer_tables"))


def run(exe, case):
    got = subprocess.run([exe, case], capture_output=True, text=True, timeout=120)
    assert got.returncode == 0 and got.stdout == "ok\n", got.stdout + got.stderr


@pytest.mark.parametrize("case", ["per_thread_hit", "per_thread_eviction", "per_thread_new_pointers"])
def test_the_per_thread_stream(exe, case):
    run(exe, case)


@pytest.mark.parametrize("case", ["destroyed_stream_undrained", "destroyed_stream_drained", "destroyed_stream_later_upload"])
def test_a_destroyed_streams_handle_given_again(exe, case):
    run(exe, case)


@pytest.mark.parametrize("case", ["other_streams_queue", "one_stream_marks_nothing"])
def test_what_a_new_table_waits_for(exe, case):
    run(exe, case)


@pytest.mark.parametrize("where", ["captured", "other", "null"])
def test_a_call_recorded_after_the_same_call_on(exe, exe_no_ids, where):
    run(exe, "recorded_after_%s_stream" % where)
    run(exe_no_ids, "recorded_after_%s_stream" % where)


def test_new_pointers_beside_a_capture(exe, exe_no_ids):
    run(exe, "new_pointers_beside_a_capture")
    run(exe_no_ids, "new_pointers_beside_a_capture")


def test_a_runtime_without_stream_ids(exe_no_ids):
    for case in ("per_thread_hit", "per_thread_eviction", "destroyed_stream_drained", "other_streams_queue"):
        run(exe_no_ids, case)
