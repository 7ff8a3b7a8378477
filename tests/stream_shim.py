"""Child processes whose hipStreamSynchronize is counted, and made to report an
error on request, by a small library loaded before the HIP runtime (the call
itself is always passed on, so that the GPU runs as it would).  The library also
counts stream captures and can refuse hipGraphInstantiate."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
static int (*real)(void*);
static int (*begin)(void*, int);
static int (*instantiate)(void*, void*, void*, char*, unsigned long);
static int calls, failing, refusing, captures;
void shim_init(void* f, void* g, void* h) {
    real = (int (*)(void*))f;
    begin = (int (*)(void*, int))g;
    instantiate = (int (*)(void*, void*, void*, char*, unsigned long))h;
}
void shim_refuse(int on) { refusing = on; }
int shim_captures(void) { return captures; }
int hipStreamBeginCapture(void* stream, int mode) { ++captures; return begin(stream, mode); }
int hipGraphInstantiate(void* x, void* g, void* n, char* log, unsigned long size) {
    return refusing ? 999 : instantiate(x, g, n, log, size);
}
int shim_calls(void) { return calls; }
void shim_fail(int on) { failing = on; }
int hipStreamSynchronize(void* stream) {
    int rc = real(stream);
    ++calls;
    return failing ? 999 : rc;   /* hipErrorUnknown */
}
"""

PRELUDE = r"""
import ctypes, sys
sys.path[:0] = [{root!r}, {tests!r}]
shim = ctypes.CDLL({shim!r}, mode=ctypes.RTLD_GLOBAL)
import numpy as np
import torch
from paper_2602_16312_amd import _ffi as F
from paper_2602_16312_amd import api, problem
from workloads import make_problem
F.lib()
path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
hip = ctypes.CDLL(path)
shim.shim_init(*(ctypes.cast(f, ctypes.c_void_p) for f in (hip.hipStreamSynchronize, hip.hipStreamBeginCapture,
                                                         hip.hipGraphInstantiate)))
"""


def run_child(tmp_path, body):
    """Runs `body` after the prelude; returns what it printed."""
    src, so = tmp_path / "shim.c", tmp_path / "libshim.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    script = tmp_path / "child.py"
    script.write_text(PRELUDE.format(root=ROOT, tests=os.path.join(ROOT, "tests"), shim=str(so)) + body)
    r = subprocess.run([sys.executable, "-u", str(script)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
