"""Which kernels a call of the C ABI launches, without a GPU: the library is
loaded in a child process behind tests/fake_hip.c, which records launches
instead of running them and reports 256 compute units.

record([call(...), ...]) returns, per call, a dict: "status"; "launches", each
a dict of the kernel's name with its template arguments, grid, block and (act-quant
kernels) its first pointers; "allocs" and "frees".
"""
from __future__ import annotations

import ctypes
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2406_02528_amd", "libmmf.so")
AUTO, GEMV, GEMM = 0, 1, 2


def call(fn, *args, capture=False, fail_alloc=False, path=AUTO, switch=None):
    """One call of `fn` with integer arguments (pointers as made-up addresses,
    None for NULL).  `switch` = (n, path): another thread sets `path` while the
    call makes its n-th query of the runtime."""
    return {"fn": fn, "args": [0 if a is None else int(a) for a in args], "capture": capture, "fail": fail_alloc,
            "path": path, "switch": list(switch or (0, 0))}


def record(calls, lib=LIB):
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "fake_hip.so")
        subprocess.run(["gcc", "-O1", "-std=c11", "-Wall", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.c"), "-o", so],
                       check=True)
        r = subprocess.run([sys.executable, os.path.abspath(__file__)], input=json.dumps([so, lib, calls]),
                           capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = json.loads(r.stdout)
    names = sorted({l["kernel"] for c in out for l in c["launches"]})
    plain = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True, check=True).stdout.split("\n")
    # mmf::skinny::skinny_kernel<4, 2, ...>(...) -> skinny_kernel<4, 2, ...>
    short = {n: _short(p) for n, p in zip(names, plain)}
    for c in out:
        for l in c["launches"]:
            l["kernel"] = short[l["kernel"]]
    return out


def _short(name):
    name = name.removeprefix("void ").replace("(anonymous namespace)::", "").replace("(mmf::Epilogue)", "")
    name = name.replace("mmf::skinny::", "").replace("mmf::dec::", "").replace("mmf::", "")
    depth = 0
    for i, c in enumerate(name):  # cut the argument list
        depth += (c == "<") - (c == ">")
        if c == "(" and depth == 0:
            return name[:i]
    return name


def kernels(result):
    """The launched kernels' names, without template arguments."""
    return [l["kernel"].split("<")[0] for l in result["launches"]]


class _Launch(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char_p), ("grid", ctypes.c_uint * 3), ("block", ctypes.c_uint * 3),
                ("args", ctypes.c_uint64 * 6)]


def _child():
    so, lib, calls = json.load(sys.stdin)
    fake = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)  # in front of the HIP runtime the library links
    mmf = ctypes.CDLL(lib)
    fake.fake_launch.restype = ctypes.POINTER(_Launch)
    fake.fake_reset.argtypes = [ctypes.c_int] * 4 + [ctypes.c_void_p]
    set_path = ctypes.cast(mmf.mmf_set_path, ctypes.c_void_p)
    out = []
    for c in calls:
        mmf.mmf_set_path(c["path"])
        fake.fake_reset(c["capture"], c["fail"], *c["switch"], set_path)
        f = getattr(mmf, c["fn"])
        f.restype = ctypes.c_size_t if c["fn"].endswith("_bytes") else ctypes.c_int
        status = f(*[ctypes.c_int64(a) for a in c["args"]])
        ls = [fake.fake_launch(i).contents for i in range(fake.fake_launches())]
        out.append({"status": status, "allocs": fake.fake_allocs(), "frees": fake.fake_frees(),
                    "launches": [{"kernel": l.name.decode(), "grid": list(l.grid), "block": list(l.block),
                                  "args": list(l.args)} for l in ls]})
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _child()
