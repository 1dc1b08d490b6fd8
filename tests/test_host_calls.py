"""What the library's host code asks of the HIP runtime, on the CPU: the calls run in a child
process with the stand-in runtime of tests/fake_hip.c preloaded, which logs them."""
import ctypes as C
import os
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
N = 8


class Handle:
    """A grid handle driven through the C ABI, its workspace in host memory."""

    def __init__(self):
        from paper_2505_17287_amd import ibm
        from paper_2505_17287_amd import inputs as I
        self.ibm, self.L, self.hip = ibm, ibm.lib(), C.CDLL(None)
        f = I.uniform_faces(-1.0, 1.0, N)
        self.h = C.c_void_p()
        assert self.L.ibm_create_grid(N, N, N, *[ibm._dp(f)] * 3, C.byref(self.h)) == 0
        v, t = I.aabb_mesh((-0.4,) * 3, (0.4,) * 3)
        self.v, self.t = np.ascontiguousarray(v, float), np.ascontiguousarray(t, np.int32)
        self.caps = (len(v), len(t), 64)

    def check(self, code):
        assert code >= 0, self.L.ibm_last_error(self.h)

    def bind(self, stream=None):
        n = self.L.ibm_grid_workspace_bytes(self.h, *self.caps, 0)
        self.ws = np.zeros(n + 256, np.uint8)
        p = self.ws.ctypes.data
        self.check(self.L.ibm_bind_workspace(self.h, C.c_void_p(p + -p % 256), n, *self.caps, 0, stream))

    def set_geometry(self, stream=None):
        self.check(self.L.ibm_set_geometry(self.h, self.ibm._dp(self.v), len(self.v), C.c_void_p(self.t.ctypes.data),
                                           len(self.t), stream))

    def classify(self, stream=None):
        counts = np.zeros(8, np.int64)
        counts[0] = N ** 3  # every cell fluid
        self.hip.fake_hip_next_read(C.c_size_t(64), C.c_void_p(counts.ctypes.data))
        self.check(self.L.ibm_classify(self.h, stream, C.c_void_p(np.zeros(3, np.int64).ctypes.data)))

    def stencils(self, stream=None):
        self.check(self.L.ibm_build_ghost_stencils(self.h, stream, None))

    def solve(self, stream=None, method="bicgstab"):
        rhs, p = np.zeros((N, N, N)), np.zeros((N, N, N))
        o = self.ibm.make_opts(method=method)
        self.check(self.L.ibm_poisson_solve(self.h, C.c_void_p(rhs.ctypes.data), C.c_void_p(p.ctypes.data), C.byref(o),
                                            None, stream))


def case_create():
    Handle()


def case_waits():
    H = Handle()
    s = C.c_void_p(0x1000)
    H.bind(s)
    H.hip.fake_hip_mark()
    for call in (H.set_geometry, H.classify, H.stencils, H.solve):
        call(s)
        H.hip.fake_hip_mark()


def case_second_device():
    H = Handle()
    for device in (0, 1, 1, 0):
        H.hip.hipSetDevice(device)
        H.bind()
        for call in (H.set_geometry, H.classify, H.stencils, H.solve):
            call()
        H.solve(method="vcycle")
    H.L.ibm_destroy_grid(H.h)


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("fake_hip")
    so = d / "fake_hip.so"
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", str(so), os.path.join(HERE, "fake_hip.c")], check=True)

    def child(name):
        log = d / (name + ".log")
        log.write_text("")
        env = dict(os.environ, LD_PRELOAD=str(so), FAKE_HIP_LOG=str(log))
        r = subprocess.run([sys.executable, os.path.abspath(__file__), name], env=env, capture_output=True, text=True,
                           timeout=120)
        assert r.returncode == 0, r.stderr[-2000:]
        return [tuple(l.rsplit(" ", 2)) for l in log.read_text().splitlines()]

    return child


def test_grid_creation_does_no_device_work(run):
    """Planning needs no GPU: a process that only sizes a problem does not start the runtime."""
    assert run("create") == []


def test_setup_and_solve_leave_nothing_in_flight(run):
    """set_geometry, classify, build_ghost_stencils and poisson_solve return with their stream
    idle: a program may go on with another stream, and the set-up time is the set-up's."""
    log, calls = run("waits"), []
    marks = [q for q, l in enumerate(log) if l[0] == "mark"]
    for name, a, b in zip(("set_geometry", "classify", "build_ghost_stencils", "poisson_solve"), marks, marks[1:]):
        work = [l for l in log[a + 1:b] if l[0] in ("kernel", "copy", "fill", "wait")]
        assert {l[1] for l in work} == {"0x1000"}
        if work[-1][0] != "wait":
            calls.append(name)
    assert len(marks) == 5 and not calls


def test_events_live_on_the_device_of_the_workspace(run):
    """A handle bound again on another device records none of the first one's events (the runtime
    refuses that) and destroys what it has created."""
    log = run("second_device")
    assert any(l[0] == "record" for l in log)
    assert sum(l[0] == "create" for l in log) == sum(l[0] == "destroy" for l in log)


if __name__ == "__main__":
    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    globals()["case_" + sys.argv[1]]()
