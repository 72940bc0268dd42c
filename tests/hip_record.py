"""Runs libacm on the recorded HIP runtime of hip_record.cpp (no GPU).

run(body, tmp_path) executes the Python statements `body` in a process of its own,
with `acm` (the binding), `np`, the recorder's `rec` library, `launches()`
and the helpers `solver(cfg, force)` and `batch(cfgs, ...)` at hand, and
returns what the body put into `result` (a JSON value)."""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = '''
import ctypes, json, sys
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rec.rec_name.restype = ctypes.c_char_p
rec.rec_count.restype = ctypes.c_long
for f in (rec.rec_name, rec.rec_grid):
    f.argtypes = [ctypes.c_long]
rec.rec_reset.argtypes = [ctypes.c_long]
rec.rec_arg.argtypes = [ctypes.c_long, ctypes.c_int]
sys.path.insert(0, sys.argv[2])
import numpy as np
from paper_2012_03525_amd import acm
keep = []


def reset(fail=-1):
    """forget the launches; the launch after the next `fail` ones fails"""
    rec.rec_reset(fail)


def launches():
    """(name, workgroups, integer arguments) of each recorded launch"""
    return [(rec.rec_name(i).decode(), rec.rec_grid(i), [rec.rec_arg(i, k) for k in range(3)])
            for i in range(rec.rec_count())]


def aligned(n):
    a = np.zeros(n + 256, np.uint8)
    keep.append(a)
    return ctypes.c_void_p(a.ctypes.data + -a.ctypes.data % 256)


def field():
    a = np.zeros(64)
    keep.append(a)
    return a.ctypes.data


def solver(cfg, force=None):
    """a handle; the fields are addresses that no recorded launch reads"""
    sets = [acm.Fields(*[field() for _ in range(5)]) for _ in range(2)]
    n = acm.lib().acm_scratch_bytes(ctypes.byref(cfg))
    h = ctypes.c_void_p()
    acm.check(acm.lib().acm_init(ctypes.byref(cfg), ctypes.byref(sets[0]), ctypes.byref(sets[1]), force, aligned(4096),
                                 ctypes.c_size_t(n), None, ctypes.byref(h)))
    return h


def current(h):
    w, s = ctypes.c_int32(), ctypes.c_int64()
    acm.check(acm.lib().acm_current(h, ctypes.byref(w), ctypes.byref(s)))
    return w.value, s.value


def batch(cfgs, tiles, chunk=20, mode=0, nsteps=20):
    arr = (acm.BatchCase * len(cfgs))()
    for k, c, t in zip(arr, cfgs, tiles):
        k.cfg, k.tile, k.nsteps, k.force_x = c, t, nsteps, None
        k.a, k.b = (acm.Fields(*[field() for _ in range(3)], None, None) for _ in range(2))
    opts = acm.BatchOpts(chunk, 0, 0, 0.0, mode)
    keep.append((arr, opts))
    n = acm.lib().acm_batch_scratch_bytes(arr, len(cfgs), ctypes.byref(opts))
    assert n, acm.lib().acm_last_error()
    h = ctypes.c_void_p()
    acm.check(acm.lib().acm_batch_init(arr, len(cfgs), ctypes.byref(opts), aligned(n), ctypes.c_size_t(n), None,
                                       ctypes.byref(h)))
    return h


result = None
'''


def run(body, tmp_path):
    lib = os.path.join(str(tmp_path), "libhiprecord.so")
    if not os.path.exists(lib):
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "hip_record.cpp"),
                               "-o", lib])
    code = PRELUDE + body + "\nprint('RESULT ' + json.dumps(result), flush=True)\n"
    p = subprocess.run([sys.executable, "-c", code, lib, ROOT], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stderr[-2000:]
    return json.loads([l for l in p.stdout.splitlines() if l.startswith("RESULT ")][-1][7:])
