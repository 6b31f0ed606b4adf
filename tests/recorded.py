"""What the library asks of the HIP runtime, seen without a GPU: a piece of Python run in a process of its own in which
tests/hip_recorder.cpp stands in for the runtime."""
import ast
import collections
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

Launch = collections.namedtuple("Launch", "kernel stream smem limit groups")  # groups: along the grid's first axis

PRELUDE = """
import ctypes, sys
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rec.recorder_line.restype = ctypes.c_char_p
import paper_1811_01532_amd as wap


class Mem:  # device memory that nothing reads
    def __init__(self, nbytes, at=1 << 40):
        self.nbytes, self.at = nbytes, at
    def data_ptr(self):
        return self.at
    def numel(self):
        return self.nbytes
    def element_size(self):
        return 1
"""
EPILOGUE = """
for i in range(rec.recorder_count()):
    print("#", rec.recorder_line(i).decode())
"""


def build(folder):
    so = os.path.join(str(folder), "hip_recorder.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wall", "-I/opt/rocm/include", os.path.join(HERE, "hip_recorder.cpp"), "-o", so], check=True)
    return so


def run(so, code, printed=None):
    """The calls that `code` (with `wap`, `Mem` and `rec` at hand) makes, as lists of words: launch kernel stream smem limit groups,
    stream handle, record stream, wait stream.  What it prints, a word and a value a line, goes to printed[word]."""
    r = subprocess.run([sys.executable, "-c", PRELUDE + code + EPILOGUE, so], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    for line in r.stdout.splitlines():
        if printed is not None and not line.startswith("# "):
            word, value = line.split(" ", 1)
            printed.setdefault(word, []).append(ast.literal_eval(value))
    return [line[2:].split() for line in r.stdout.splitlines() if line.startswith("# ")]


def launches(calls):
    return [Launch(c[1], c[2], int(c[3]), int(c[4]), int(c[5])) for c in calls if c[0] == "launch"]
