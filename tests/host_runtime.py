"""librcx on a stand-in for the HIP runtime (fake_hip.c): tests of its host
code (plans, dispatch, workspaces, failures of device allocations) without a
GPU. ``run(code)`` runs ``code`` in a child process with ``rt`` (the stand-in),
``L`` (librcx) and the helpers below in scope; the child's failed assertions
fail the test. The stand-in is loaded first, so the library's HIP calls bind to it."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes as C, sys
rt = C.CDLL({shim!r}, mode=C.RTLD_GLOBAL)
rt.fake_log.restype = C.c_char_p
rt.fake_live_bytes.restype = C.c_size_t
rt.fake_fail_malloc.argtypes = [C.c_int, C.c_int]
rt.hipMalloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t]
sys.path.insert(0, {root!r})
from paper_2408_14425_amd import rcx
L = rcx.load()

def params(**kw):
    p = rcx.rcx_params_default()
    for k, v in kw.items():
        setattr(p, k, v)
    return p

def plan(nx, nz, n_wave=1, **kw):
    return C.c_void_p(rcx.rcx_plan_create(rcx.rcx_grid(nx, nz, 1.0), params(**kw), n_wave))

def device(n_bytes):
    p = C.c_void_p()
    assert rt.hipMalloc(C.byref(p), n_bytes) == 0
    return p

def launches(clear=True):
    # [(kernel, grid x, grid y, block x)] since the last clear
    out = []
    for line in rt.fake_log().decode().splitlines():
        name, gx, gy, gz, bx = line.split()
        out.append((name, int(gx), int(gy), int(bx)))
    if clear:
        rt.fake_log_clear()
    return out

def mallocs():
    out = (C.c_size_t * 256)()
    return list(out[:rt.fake_sizes(out)])

def count(ls, kernel):
    return sum(kernel in l[0] for l in ls)

def solve(p, nx, nz, n_wave=1):
    f = device(4 * n_wave * nx * nz)
    rt.fake_log_clear()
    rc = L.rcx_formal_solve(p, n_wave, f, f, f, None, 0, None)
    buf = C.create_string_buffer(512)
    L.rcx_last_error(buf, 512)
    assert rc == 0, (rc, buf.value)
    return launches()
"""


def run(tmp_path, code: str) -> str:
    cc = os.environ.get("CC") or shutil.which("gcc") or shutil.which("cc") or "/opt/rocm/llvm/bin/clang"
    shim = os.path.join(str(tmp_path), "libfake_hip.so")
    subprocess.run([cc, "-O1", "-shared", "-fPIC", "-o", shim, os.path.join(HERE, "fake_hip.c")], check=True)
    script = PRELUDE.format(shim=shim, root=ROOT) + textwrap.dedent(code)
    res = subprocess.run([sys.executable, "-c", script], capture_output=True, text=True, timeout=300, cwd=ROOT)
    assert res.returncode == 0, res.stdout + res.stderr
    return res.stdout
