"""Run a script against libapss.so with no device: the host code as it is, kernels only noted (see fake_hip.c).

The script finds ``fake`` (the stand-in runtime), ``apss``, ``np``, ``index(n)`` (an index of n rows over 64
dimensions) and ``launches()`` (the kernels' names since the last call).
"""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, sys
sys.path.insert(0, %(root)r)
%(before)s
fake = ctypes.CDLL(%(lib)r, ctypes.RTLD_GLOBAL)
fake.fake_launch.restype = ctypes.c_char_p
for f in (fake.fake_mallocs, fake.fake_live):
    f.restype = ctypes.c_long
for f in (fake.fake_fail_mallocs, fake.fake_fail_events):
    f.argtypes = [ctypes.c_long, ctypes.c_long]
import numpy as np
import paper_1402_3010_amd as apss
apss.load()

def launches():
    out = [fake.fake_launch(k).decode() for k in range(fake.fake_launches())]
    fake.fake_forget_launches()
    return out

def rows(n):
    c = (np.arange(2 * n) %% 64).astype(np.int32)
    return np.arange(0, 2 * n + 1, 2), c, np.full(2 * n, np.sqrt(0.5), np.float32)

def index(n, t=0.5, **kw):
    o = apss.default_opts()
    for k, v in kw.items():
        setattr(o, k, v)
    return apss.Index(apss.build_index(n, 64, *rows(n), t, o), n, 64)
"""


def run(tmp_path, script, before=""):
    lib = os.path.join(str(tmp_path), "fake_hip.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "fake_hip.c"), "-o", lib], check=True)
    env = {k: v for k, v in os.environ.items() if not k.startswith("APSS_")}
    r = subprocess.run([sys.executable, "-c", PRELUDE % dict(root=ROOT, lib=lib, before=before) + script], capture_output=True,
                       text=True, timeout=300, env=env)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return r.stdout
