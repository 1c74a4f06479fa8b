"""The library on the CPU over a HIP runtime that runs nothing (c/hip_stub.cpp):
a test's cases run in a process of their own, where that runtime is loaded
before the library.

A test file's cases are functions of one argument, this module's ``Stub``;
``run_case(__file__, name)`` runs one of them in such a process, and
``main()`` at the end of the file is that process's side.
"""
import ctypes
import os
import re
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "c", "hip_stub.cpp")


def build(directory):
    so = os.path.join(str(directory), "libhipstub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-shared", "-fPIC", "-pthread", "-o", so,
                    SRC], check=True, capture_output=True, text=True)
    return so


def run_case(path, name, so, *args, timeout=120):
    r = subprocess.run([sys.executable, path, name, so, *map(str, args)], capture_output=True,
                       text=True, timeout=timeout, cwd=ROOT)
    assert r.returncode == 0, f"{name}: status {r.returncode}\n{r.stdout}{r.stderr}"


class Stub:
    def __init__(self, so):
        sys.path.insert(0, ROOT)
        sys.modules["torch"] = None  # its own HIP runtime stays out of this process
        self.L = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
        self.L.hs_log.restype = ctypes.c_char_p
        for f in ("hs_pinned_now", "hs_pinned_peak"):
            getattr(self.L, f).restype = ctypes.c_size_t
        self.L.hs_hold.argtypes = [ctypes.c_char_p, ctypes.c_void_p]
        self.L.hs_cost.argtypes = [ctypes.c_char_p, ctypes.c_double]
        self.L.hs_capture.argtypes = [ctypes.c_void_p, ctypes.c_int]
        import paper_1010_1233_amd as flb
        self.flb = flb
        flb.lib()

    def hold(self, fn, obj=None):
        self.L.hs_hold(fn.encode(), obj)

    def held(self, fn, n=1, ms=5000):
        return bool(self.L.hs_held(fn.encode(), n, ms))

    def release(self, fn):
        self.L.hs_release(fn.encode())

    def cost(self, part_of_name, ms):
        self.L.hs_cost(part_of_name.encode(), ms)

    def stream(self, device=0):
        """A stream made on a device (the thread's current one is put back)."""
        old, s = ctypes.c_int(), ctypes.c_void_p()
        self.L.hipGetDevice(ctypes.byref(old))
        self.L.hipSetDevice(device)
        self.L.hipStreamCreateWithFlags(ctypes.byref(s), 1)
        self.L.hipSetDevice(old)
        return s.value

    def take_log(self):
        out = [self.L.hs_log(i).decode() for i in range(self.L.hs_log_size())]
        self.L.hs_log_clear()
        return out

    def take_steps(self):
        """The launches that step from one buffer into another since the last
        call: (kernel, steps, source, destination)."""
        out = []
        for line in self.take_log():
            m = re.match(r"launch (\w+).* src=(\S+) dst=(\S+) steps=(\d+)", line)
            if m and int(m[4]):
                out.append((m[1], int(m[4]), m[2], m[3]))
        return out


def main(cases):
    cases[sys.argv[1]](Stub(sys.argv[2]), *sys.argv[3:])
