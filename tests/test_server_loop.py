"""The request loop (csrc/server.cpp) built for the host with its launches replaced by events that
end when the scenario says so (native/server_loop.cpp), under the address sanitizer: requests that
finish out of line, a reset while others run, launches that fail, a client that polls."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2305_02678_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("server_loop") / "server_loop")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer", "-D__HIP_PLATFORM_AMD__",
           f"-I{ROCM}/include", f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}",
           os.path.join(HERE, "native", "server_loop.cpp"), os.path.join(CSRC, "server.cpp"), "-pthread", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def _run(program, scenario):
    r = subprocess.run([program, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.stdout + r.stderr)[:4000]


@pytest.mark.parametrize("scenario", ["reset_behind_other_kernel", "reset_after_failed_group",
                                      "reset_with_tile_of_failed_request"])
def test_reset_while_requests_run(program, scenario):
    _run(program, scenario)


def test_submissions_reach_an_idle_worker(program):
    _run(program, "poll_from_idle")
