"""Runs the library's host code without a GPU: a child process loads a stand-in
for the HIP runtime (native/fake_hip.cpp) ahead of the library and sees what
each call would have launched or allocated."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = r"""
import ctypes, sys
sys.modules["torch"] = None          # the binding does without it here
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
fake.fake_log.restype = ctypes.c_char_p
fake.fake_graphs.restype = ctypes.c_long
import paper_2209_08241_amd as bn
L = bn.lib()

def frames(shapes, off=0):
    # made-up device addresses, 1 GiB apart; `off` elements into their buffers
    at = lambda k, j: (4 * k + j + 1) << 30
    return (bn.Frame * len(shapes))(*[
        bn.Frame(at(k, 0), H, W, W, 500.0, 500.0, W / 2, H / 2, at(k, 1) + 4 * off,
                 at(k, 2) + off, at(k, 3)) for k, (H, W) in enumerate(shapes)])

def log():
    lines = fake.fake_log().decode().splitlines()
    fake.fake_clear()
    return lines

def launches(lines):
    # (kernel's name, workgroups) of each launch
    out = []
    for line in lines:
        if line.startswith("launch "):
            name, gx = line.split()[1:3]
            out.append((name, int(gx)))
    return out

def create(shapes, params=None):
    p = params or bn.make_params(2)
    h = ctypes.c_void_p()
    assert L.bn_batch_plan_create(frames(shapes), len(shapes), p, ctypes.byref(h)) == 0
    return h

def update(h, shapes):
    return L.bn_batch_plan_update(h, frames(shapes), len(shapes), None)
"""


def build(folder) -> str:
    so = os.path.join(str(folder), "libfakehip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "native", "fake_hip.cpp"), "-o", so], check=True)
    return so


def run(so: str, code: str) -> None:
    res = subprocess.run([sys.executable, "-c", PRELUDE + code, so], cwd=ROOT, timeout=120,
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-3000:]
