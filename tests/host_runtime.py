"""Runs a piece of Python against liblbm_hip.so on the host runtime of
host_runtime.c, in a process of its own (a process that has loaded a HIP runtime
keeps it).

The code finds `L` (the ctypes binding), `solver(grid, ...)` -> handle,
`calls()` -> the log since the last call of it, `kernels()` -> the names of the
launches in it, `fail_launch(n)`, and leaves its answer in `out` (JSON)."""
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

_PRELUDE = '''
import ctypes, importlib.util, json, re
rt = ctypes.CDLL({runtime!r}, mode=ctypes.RTLD_GLOBAL)
rt.host_log.restype = ctypes.c_char_p
rt.host_fail_launch.argtypes = [ctypes.c_long]
spec = importlib.util.spec_from_file_location("lbm", {binding!r})
L = importlib.util.module_from_spec(spec)
spec.loader.exec_module(L)
_cxx = ctypes.CDLL("libstdc++.so.6")
_cxx.__cxa_demangle.restype = ctypes.c_char_p
def _name(mangled):
    s = _cxx.__cxa_demangle(mangled.encode(), None, None, None)
    s = (s or mangled.encode()).decode().split("(anonymous namespace)::")[-1]
    return re.sub(r"\\(.*", "", s)
def calls():
    lines = rt.host_log().decode().split("\\n")[:-1]
    rt.host_log_clear()
    return [("launch " + _name(l.split()[1])) if l.startswith("launch") else l for l in lines]
def kernels():
    return [l[7:] for l in calls() if l.startswith("launch")]
fail_launch = rt.host_fail_launch
A, B, C, D = 1 << 40, 1 << 41, 1 << 42, 1 << 43  # buffers: the host never follows them
def solver(grid, eps=0.1, flags=0, a=A, b=B):
    nu, dx = 0.02, 1.0 / max(grid)
    return L.lb_create(L.make_config(grid, dx, eps * dx * dx / nu, nu, flags), 0, a, b)
out = None
'''


_tmp = None  # holds the built runtime while the tests run


def _runtime() -> str:
    global _tmp
    if _tmp is None:
        _tmp = tempfile.TemporaryDirectory()
        subprocess.run(["gcc", "-O1", "-std=c11", "-Wall", "-shared", "-fPIC", "-o",
                        os.path.join(_tmp.name, "host_runtime.so"),
                        os.path.join(HERE, "host_runtime.c")], check=True)
    return os.path.join(_tmp.name, "host_runtime.so")


def run(code: str):
    binding = os.path.join(ROOT, "paper_2309_02825_amd", "lbm.py")
    src = _PRELUDE.format(runtime=_runtime(), binding=binding) + code + "\nprint(json.dumps(out))\n"
    r = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout.strip().split("\n")[-1])
