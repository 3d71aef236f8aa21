"""Host path of a solve without a GPU: the library's host code on a stand-in for the HIP runtime."""
import os
import shutil
import signal
import time

import numpy as np
import pytest

import host_runtime
import mgk_workloads as W

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return host_runtime.build(tmp_path_factory.mktemp("host_runtime"))


@pytest.fixture
def host(so):
    h = host_runtime.Host(so)
    yield h
    if h.ctx is not None:
        h.destroy()


def in_child(f, seconds=20):
    """Exit status of a forked child that calls f; None if it does not end."""
    pid = os.fork()
    if pid == 0:
        try:
            f()
        except BaseException:
            os._exit(1)
        os._exit(0)
    end = time.time() + seconds
    while time.time() < end:
        got, status = os.waitpid(pid, os.WNOHANG)
        if got:
            return status
        time.sleep(0.01)
    os.kill(pid, signal.SIGKILL)
    os.waitpid(pid, 0)
    return None


def test_context_survives_a_fork(so):
    """The threads of a context do not exist in a forked child: loading and destroying work there."""
    h = host_runtime.Host(so, -1)
    wb = W.config1(40)

    def child():
        h.free(h.load(wb, reorder=1))
        h.destroy()

    h.free(h.load(wb, reorder=1))   # starts the threads
    assert in_child(child) == 0
    h.free(h.load(wb, reorder=1))
    h.destroy()
