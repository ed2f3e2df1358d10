"""Host code of the built library without a device: a child process loads the
stand-ins of hip_host.cpp, then libfdbb.so, and runs a test's script with the
names defined here.  No kernel runs."""
import ctypes
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIBRARY = os.path.join(os.path.dirname(HERE), "paper_1809_09851_amd", "libfdbb.so")
EINVAL, EHIP = 1, 4
CONS2PRIM, FLUX, JACOBIAN, CONS2CHAR, FUSED, EIGEN, FLUX_DIR = 0, 3, 4, 6, 8, 11, 16
F64, F32 = 0, 1


class Task(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("op", "dim", "dtype", "dir")] + [
        ("gamma", ctypes.c_double), ("n", ctypes.c_int64)] + [
        f for s in ("in0", "in1", "out0", "out1", "out2")
        for f in ((s, ctypes.c_void_p), ("ld_" + s, ctypes.c_int64))]


_next = [1 << 40]


def address(fields, n, unit=1, es=8, offset=0):
    """A range of its own for `fields` rows of n points."""
    p = _next[0]
    _next[0] += (fields * n * unit * es + offset + 8191) // 4096 * 4096
    return p + offset


def task(op, dim, n, dtype=F64):
    K, es = dim + 2, 4 if dtype == F32 else 8
    t = Task(op=op, dim=dim, dtype=dtype, gamma=1.4, n=n)
    t.in0, t.ld_in0 = address(K, n, es=es), n
    rows = {CONS2PRIM: K, CONS2CHAR: K, FLUX_DIR: K, FLUX: K * dim, FUSED: K * dim}.get(op)
    if rows:
        t.out0, t.ld_out0 = address(rows, n, es=es), n
    if op == JACOBIAN:
        t.out0, t.ld_out0 = address(dim, n, K * K, es), n
    if op == EIGEN:
        t.out0, t.ld_out0 = address(dim, n, K * K, es), n
        t.out1, t.ld_out1 = address(dim, n, K * K, es), n
    if op == FUSED:
        t.out1, t.ld_out1 = address(dim, n, K * K, es), n
        t.out2, t.ld_out2 = address(2 * dim + 1, n, es=es), n
    return t


class Launch:
    def __init__(self, line):
        self.kernel, *v = line.rsplit(None, 5)
        self.grid, self.block, self.lds, self.units, self.replay = map(int, v)

    def __repr__(self):
        return f"{self.kernel} grid {self.grid} block {self.block} lds {self.lds} units {self.units} replay {self.replay}"


class Host:
    """The stand-ins and the library; `launches` empties the log."""

    def __init__(self, stand_ins, library):
        self.hip = ctypes.CDLL(stand_ins, mode=ctypes.RTLD_GLOBAL)
        self.hip.host_log.restype = ctypes.c_char_p
        self.lib = ctypes.CDLL(library)
        self.lib.fdbb_last_error.restype = ctypes.c_char_p

    def launches(self):
        return [Launch(l) for l in self.hip.host_log().decode().splitlines()]

    def fail(self, call, on=True):
        self.hip.host_fail(call.encode(), int(on))

    def stream(self):
        s = ctypes.c_void_p()
        self.hip.hipStreamCreateWithFlags(ctypes.byref(s), 0)
        return s

    def capture(self, stream, body):
        """body() captured on `stream`; the instantiated graph."""
        g, x = ctypes.c_void_p(), ctypes.c_void_p()
        self.hip.hipStreamBeginCapture(stream, 0)
        body()
        self.hip.hipStreamEndCapture(stream, ctypes.byref(g))
        self.hip.hipGraphInstantiate(ctypes.byref(x), g, None, None, ctypes.c_size_t(0))
        return x

    def replay(self, graph, stream):
        self.hip.hipGraphLaunch(graph, stream)

    def plan(self, tasks, capacity=16, block=0, ppt=1, grid=0, nt=1):
        p = ctypes.c_void_p()
        rc = self.lib.fdbb_batch_plan_create(_array(tasks), len(tasks), capacity, block, ppt, grid, nt, ctypes.byref(p))
        assert rc == 0, self.lib.fdbb_last_error()
        return p

    def update(self, plan, tasks, stream):
        return self.lib.fdbb_batch_plan_update(plan, _array(tasks), len(tasks), stream)

    def run(self, plan, stream, graph):
        return self.lib.fdbb_batch_exec(plan, stream, int(graph))


def _array(tasks):
    return (Task * max(1, len(tasks)))(*tasks)


def build(folder):
    out = os.path.join(str(folder), "libhip_host.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I/opt/rocm/include",
                    os.path.join(HERE, "hip_host.cpp"), "-o", out], check=True)
    return out


def run(stand_ins, script):
    """Runs `script` in a child with `h` a Host; its failed assertion fails
    the caller."""
    head = f"import sys; sys.path.insert(0, {HERE!r})\nfrom hip_host import *\nh = Host({stand_ins!r}, {LIBRARY!r})\n"
    r = subprocess.run([sys.executable, "-c", head + script], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
