"""Which launches a call of the library leads to, without a GPU: ``launches``
runs calls in a process of its own, where launch_recorder.cpp stands in for
the HIP runtime (a device of 256 compute units), and returns every launch's
kernel, grid, work-group and LDS.  Addresses are made up: nothing is run."""

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


@functools.lru_cache(maxsize=None)


def _recorder():
    out = os.path.join(tempfile.mkdtemp(prefix="dpia_launches_"), "recorder.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC",
                    os.path.join(HERE, "launch_recorder.cpp"), "-o", out, "-ldl"], check=True)
    atexit.register(shutil.rmtree, os.path.dirname(out), ignore_errors=True)
    return out


def launches(calls):
    """``calls``: (entry point, strategy fields, other arguments by name); a
    list of [{"kernel", "grid", "block", "lds"}] for each, or its status."""
    r = subprocess.run([sys.executable, os.path.abspath(__file__), _recorder()],
                       input=json.dumps(calls), capture_output=True, text=True,
                       cwd=os.path.dirname(HERE))
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.splitlines()[-1])


def _demangle(names):
    r = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True,
                       check=True)
    return dict(zip(names, r.stdout.splitlines()))


def _call(L, dp, entry, strategy, a):
    # made-up device addresses, 256-byte aligned and far apart
    A, x, y, out, ws, scale = (ctypes.c_void_p((i + 1) << 42) for i in range(6))
    s = dp.Strategy(**strategy)
    r = ctypes.byref(s.c())
    dt = a.get("dtype", dp.F32)
    if entry == "scal":
        return L.dpia_scal(r, dt, a["n"], 0.5, x, y, None)
    if entry == "gemv":
        lda = a.get("lda", a["k"])
        return L.dpia_gemv(r, dt, a["m"], a["k"], lda, A, scale if dt == dp.FP8_E4M3 else None, x, y,
                           None, 0, None)
    if entry == "asum":
        return L.dpia_asum(r, dt, a["n"], x, out, dp.F32, ws, 1 << 50, None)
    if entry == "dot":
        return L.dpia_dot(r, dt, a["n"], x, y, out, dp.I32 if dt == dp.I32 else dp.F32, ws, 1 << 50,
                          None)
    if entry == "fold":
        return L.dpia_fold(r, dp.OP_DOT, dt, a["n"], x, out, dp.I32 if dt == dp.I32 else dp.F32, None)
    raise ValueError(entry)


def _main():
    rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # (before the library is loaded)
    rec.launch_kernel.restype = ctypes.c_char_p
    for f in (rec.launch_grid, rec.launch_block, rec.launch_lds):
        f.restype = ctypes.c_uint64
    sys.path.insert(0, os.path.dirname(HERE))
    import paper_1710_08332_amd as dp
    from paper_1710_08332_amd import _lib
    L = _lib.lib()
    done = []
    for entry, strategy, args in json.load(sys.stdin):
        rec.launches_clear()
        st = _call(L, dp, entry, strategy, args)
        done.append(st if st != _lib.OK else
                    [dict(kernel=rec.launch_kernel(i).decode(), grid=rec.launch_grid(i),
                          block=rec.launch_block(i), lds=rec.launch_lds(i))
                     for i in range(rec.launches_made())])
    names = sorted({l["kernel"] for d in done if isinstance(d, list) for l in d})
    plain = _demangle(names) if names else {}
    for d in done:
        if isinstance(d, list):
            for l in d:
                l["kernel"] = plain[l["kernel"]]
    print(json.dumps(done))

if __name__ == "__main__":
    _main()
