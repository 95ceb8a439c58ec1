"""Runs the library against a HIP runtime of host bookkeeping (fake_hip.cpp), in a process of its own.

The fake runtime's symbols go into the process's global scope before libqe.so is loaded, so the library's
calls bind to them; torch, which would bring a real runtime, stays out.  A test names a function of its own
module; `calls` runs it in a child process and returns what it returns (JSON values).

    def scenario(qe, hip): ...          # hip.log(), hip.pending(), hip.drain(stream), hip.fail_launch(n) ..
    def test_it(): assert calls(scenario) == ...
"""
import ctypes as C
import functools
import importlib
import json
import os
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "tests", "fake_hip.cpp")
ADDR = 1 << 20  # a device address: never read


class Hip:
    def __init__(self, path):
        self.so = C.CDLL(path, mode=C.RTLD_GLOBAL)
        self.so.fake_log.restype = C.c_char_p
        self.so.fake_drain.argtypes = [C.c_void_p]
        self.pending, self.drain = self.so.fake_pending, self.so.fake_drain
        self.fail_launch, self.fail_record = self.so.fake_fail_launch, self.so.fake_fail_record
        self.clear = self.so.fake_clear

    def log(self, *kinds):
        """The logged calls as lists of words; with kinds, those that begin with one of them."""
        lines = [s.split() for s in self.so.fake_log().decode().splitlines()]
        return [w for w in lines if not kinds or w[0] in kinds]


@functools.lru_cache(maxsize=None)
def _built():
    """The folder of the built runtime, removed with the process."""
    td = tempfile.TemporaryDirectory()
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", SOURCE, "-o", os.path.join(td.name, "libfakehip.so")], check=True)
    return td


def calls(scenario, *args):
    so = os.path.join(_built().name, "libfakehip.so")
    r = subprocess.run([sys.executable, "-m", "tests.fake_hip", so, scenario.__module__.split(".")[-1],
                        scenario.__name__, json.dumps(args)], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads(r.stdout.splitlines()[-1])


if __name__ == "__main__":
    sys.modules["torch"] = None  # importing it fails
    hip = Hip(sys.argv[1])
    from paper_2609_23536_amd import qe
    scenario = getattr(importlib.import_module("tests." + sys.argv[2]), sys.argv[3])
    print(json.dumps(scenario(qe, hip, *json.loads(sys.argv[4]))))
