"""Which kernels a call launches, read without a GPU: libqn.so is loaded in a
process of its own behind a stand-in for the HIP runtime (launch_trace.cpp)
whose launches only write a log."""

import atexit
import ctypes
import functools
import json
import os
import shutil
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CLANG = "/opt/rocm/llvm/bin/clang++"
ADDR = 1 << 20  # any aligned address: nothing is read or written


@functools.lru_cache(maxsize=None)
def _stand_in():
    d = tempfile.mkdtemp(prefix="qn_trace_")
    atexit.register(shutil.rmtree, d, True)
    so = os.path.join(d, "trace.so")
    subprocess.run([CLANG, "-O1", "-std=c++17", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2502_03611_amd", "csrc"),
                    os.path.join(HERE, "launch_trace.cpp"), "-o", so], check=True)
    return so


def trace(calls, lib=None):
    """calls: dicts with "shape" (array order), "do" (a list of "solve",
    "iterate", "autotune", ["pin", launch], ["device", d]) and, as for Solver,
    "problem", "precision", "boundary", "sem_order"; or "sizes", "ncomp" and
    "precision" of a batch.  One list of log entries per call, each a dict with
    kind, device, grid, block, lds, span, name."""
    env = {k: v for k, v in os.environ.items() if k != "PYTHONPATH"}
    out = subprocess.run([sys.executable, os.path.abspath(__file__), _stand_in(), lib or ""],
                         input=json.dumps(calls), capture_output=True, text=True, env=env)
    assert out.returncode == 0, out.stderr[-2000:]
    res = []
    for text in json.loads(out.stdout):
        rows = []
        for ln in text.splitlines():
            f = ln.split(" ", 2 if ln.startswith("raise") else 6)
            if f[0] == "raise":
                rows.append({"kind": "raise", "device": int(f[1]), "name": f[2]})
            else:
                d, g, b, l, s = (int(v) for v in f[1:6])
                rows.append({"kind": "launch", "device": d, "grid": g, "block": b, "lds": l, "span": s,
                             "name": f[6]})
        res.append(rows)
    return res


def argument_bytes():
    """Bytes of the structs that the launches of dense, line and row passes copy."""
    return [ctypes.CDLL(_stand_in()).trace_argument_bytes(k) for k in range(3)]


FORMS = {"k_fast": "F", "k_strip": "S", "k_fold": "T", "k_gemm": "D"}


def forms(rows):
    """The mode products of one solve, in order: F factored, S strip, T tile, D
    dense split-bf16."""
    return "".join(v for r in rows if r["kind"] == "launch"
                   for k, v in FORMS.items() if k in r["name"])


def _main(stand_in, path, calls):
    import types
    T = ctypes.CDLL(stand_in, mode=ctypes.RTLD_GLOBAL)
    T.trace_text.restype = ctypes.c_char_p
    sys.modules["torch"] = types.ModuleType("torch")  # its libraries would bring the real runtime in
    sys.path.insert(0, ROOT)
    from paper_2502_03611_amd import _binding as qn
    from paper_2502_03611_amd import batched
    if path:
        qn.LIB_PATH = path
    L = qn.lib()

    def single(c):
        shape = c["shape"]
        g, o, ctx = qn.QNGrid(), qn.QNOptions(), ctypes.c_void_p()
        g.dim = len(shape)
        for a, n in enumerate(list(reversed(shape)) + [1] * (3 - len(shape))):
            g.n[a] = n
        prob = c.get("problem", "cubic")
        g.ncomp = 2 if prob in ("system", "grayscott") else 1
        o.precision = qn.PRECISIONS[c.get("precision", "fp64")]
        o.boundary = qn.BOUNDARIES[c.get("boundary", "dirichlet")]
        o.discretization = 1 if c.get("sem_order") else 0
        o.sem_order = c.get("sem_order", 0)
        qn.check(L.qn_setup(ctypes.byref(g), 1.0, qn.NONLINEARITIES[prob], ctypes.byref(o),
                            ctypes.byref(ctx)))
        qn.check(L.qn_bind_workspace(ctx, ADDR, 1 << 46))
        T.trace_clear()
        for d in c["do"]:
            if d == "solve":
                qn.check(L.qn_fdm_solve(ctx, ADDR, 1.0, 1.0, ADDR))
            elif d == "iterate":  # one step's launches; the scalars never arrive
                L.qn_iterate(ctx, ADDR, ADDR, 0.0, 1, None)
            elif d == "autotune":
                qn.check(L.qn_autotune(ctx))
                T.trace_clear()
            elif d[0] == "device":
                T.trace_device(d[1])
            else:  # ["pin", launch]: to its own tile
                info = (ctypes.c_int32 * 4)()
                qn.check(L.qn_tile_info(ctx, d[1], info))
                qn.check(L.qn_set_tile(ctx, d[1], info))
        L.qn_destroy(ctx)

    def batch(c):
        B = batched._qnb()
        sizes, ctx = c["sizes"], ctypes.c_void_p()
        arr = ctypes.c_int32 * len(sizes)
        qn.check(B.qnb_setup(len(sizes), arr(*sizes), arr(*c["ncomp"]),
                             qn.PRECISIONS[c.get("precision", "fp64")], 1, 0.0, ctypes.byref(ctx)))
        qn.check(B.qnb_bind_workspace(ctx, ADDR, 1 << 46))
        T.trace_clear()
        qn.check(B.qnb_fdm_solve(ctx, ADDR, 1.0, 1.0, ADDR))
        B.qnb_destroy(ctx)

    out = []
    for c in calls:
        T.trace_device(0)
        batch(c) if "sizes" in c else single(c)
        out.append(T.trace_text().decode())
    print(json.dumps(out))


if __name__ == "__main__":
    _main(sys.argv[1], sys.argv[2], json.load(sys.stdin))
