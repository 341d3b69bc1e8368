"""The C ABI on the CPU: the server's host code with HIP and the launches
replaced (tests/host_server.cpp), numpy arrays as device memory."""
import ctypes
import os
import subprocess
from collections import namedtuple

import numpy as np

from paper_1611_06213_amd import ps

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1611_06213_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

Launch = namedtuple("Launch", "kind k r gdt pdt fronts blocks group")
APPLY, SYNC, PULL, STEPS, SYNC_STEPS = range(5)   # Launch.kind
STREAM = 0x1000   # any stream but the null one


def build(out):
    """The shared library at `out`. -Bsymbolic: its own HIP calls, whatever
    else the process has loaded."""
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fPIC", "-shared", "-ffp-contract=off", "-Wall",
           "-Wextra", "-Werror", "-Wno-unused-parameter", "-D__HIP_PLATFORM_AMD__", "-Wl,-Bsymbolic",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-isystem", os.path.join(ROCM, "include"),
           *(os.path.join(CSRC, s) for s in ("ps_server.cpp", "ps_protocol.cpp", "ps_layout.cpp")),
           os.path.join(ROOT, "tests", "host_server.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return ps.load_library(out)


class Host:
    """A server of the host build; `lib` is what build() returned and is the
    library that paper_1611_06213_amd.ps calls."""

    def __init__(self, lib, n, lr=0.01, momentum=0.0, depth=64, run=True, skip=True):
        self.lib, self.n = lib, n
        lib.host_reset(int(run))
        self.h = ps.ps_create(n, lr, momentum)
        assert ps.ps_set_stream(self.h, STREAM) == 0
        assert ps.ps_set_queue_depth(self.h, depth) == 0
        assert ps.ps_set_pull_skip(self.h, skip) == 0

    def launches(self):
        out, v = [], (ctypes.c_int * 8)()
        for i in range(self.lib.host_launches()):
            self.lib.host_launch(i, v)
            out.append(Launch(*v))
        return out

    def clear(self, fail=-1):
        """Empty the launch log; its `fail`-th launch from now on fails."""
        self.lib.host_reset(1)
        self.lib.host_fail_launch(fail)

    def w(self):
        return np.ctypeslib.as_array((ctypes.c_float * self.n).from_address(ps.ps_weights(self.h))).copy()

    def v(self):
        p = ps.ps_velocity(self.h)
        return np.ctypeslib.as_array((ctypes.c_float * self.n).from_address(p)).copy() if p else None

    def state(self):
        """Everything the server says of itself."""
        s = ps.ps_get_stats(self.h)
        return ({f: getattr(s, f) for f, _ in s._fields_ if f != "staleness_hist"}, list(s.staleness_hist),
                ps.ps_pending(self.h), ps.ps_timestamp(self.h), ps.ps_last_applied(self.h),
                ps.ps_last_staleness(self.h))

    def close(self):
        ps.ps_destroy(self.h)


def script(ops, base=0):
    """An OpScript of ("push", learner, offset, dtype), ("apply",), ("sync",), ("pull" |
    "apply_pull", offsets, dtype): offsets count 2-byte units from `base`, and a
    call's i-th replica is learner i's."""
    s = ps.OpScript()
    for op in ops:
        if op[0] == "push":
            s.push(op[1], base + 2 * op[2], op[3])
        elif op[0] == "apply":
            s.apply()
        elif op[0] == "sync":
            s.apply_sync()
        else:
            f = s.pull if op[0] == "pull" else s.apply_pull
            f(list(range(len(op[1]))), [base + 2 * o for o in op[1]], op[2])
    return s.build()
