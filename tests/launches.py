"""Which kernels a call of the library launches, found out without a GPU: a child process loads libhq.so on top of
tests/launch_recorder.cpp, which writes launches down instead of carrying them out.

    calls([("fwd", problem fields), ...])  ->  one list of Launch per call
"""
import collections
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
Launch = collections.namedtuple("Launch", "kernel blocks threads lds lds_allowed")
_recorder = None


def recorder():
    """The stand-in runtime, built once per test run."""
    global _recorder
    if _recorder is None:
        folder = tempfile.mkdtemp(prefix="hq_launches_")
        _recorder = os.path.join(folder, "launch_recorder.so")
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", _recorder,
                        os.path.join(HERE, "launch_recorder.cpp")], check=True)
    return _recorder


def calls(wanted):
    """wanted: (operation, the ten fields of an hq_problem or, for weight_quantize, the element count[, device index]) each.
    Operations: fwd, dgrad, dgrad_sr, wgrad, dynamic_fwd, dynamic_dgrad, weight_prepare, weight_quantize."""
    r = subprocess.run([sys.executable, os.path.abspath(__file__), recorder()], input=json.dumps(wanted), cwd=ROOT,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    return [[Launch(*l) for l in launches] for launches in json.loads(r.stdout)]


def _main():
    import ctypes as C
    rec = C.CDLL(sys.argv[1], mode=os.RTLD_GLOBAL | os.RTLD_NOW)
    rec.recorder_lines.restype = C.c_char_p
    sys.path.insert(0, ROOT)
    import paper_2105_04246_amd as hq
    ptr = 0x10000                                                        # aligned; nothing dereferences it
    out = []
    for op, what, *dev in json.load(sys.stdin):
        rec.recorder_reset(dev[0] if dev else 0)
        if op == "weight_quantize":
            hq.hq_weight_quantize(ptr, what, ptr, ptr, 0)
        else:
            p = hq.problem(*what)
            one = (p, ptr, ptr, ptr, ptr, ptr, ptr)
            if op == "fwd":
                hq.hq_gemm_fwd(*one, ptr, ptr, ptr, 0)
            elif op == "dgrad":
                hq.hq_gemm_dgrad(*one, ptr, ptr, ptr, 0)
            elif op == "dgrad_sr":
                hq.hq_gemm_dgrad_sr(*one, 5, ptr, ptr, ptr, 0)
            elif op == "wgrad":
                hq.hq_gemm_wgrad(p, ptr, ptr, ptr, ptr, ptr, None, ptr, 1 << 40, 0)
            elif op in ("dynamic_fwd", "dynamic_dgrad"):
                entry = hq.HQ_ENTRY_DYNAMIC_FWD if op == "dynamic_fwd" else hq.HQ_ENTRY_DYNAMIC_DGRAD
                hq.hq_gemm_dynamic(entry, 0, *one, ptr, ptr, ptr, ptr, 1 << 40, 0)
            elif op == "weight_prepare":
                hq.hq_weight_prepare(p, ptr, None if p.kind == hq.HQ_DEPTHWISE or p.C == 3 else ptr, ptr, ptr, 0)
        lines = rec.recorder_lines().decode().splitlines()
        out.append([[f[0]] + [int(v) for v in f[1:]] for f in (l.split("\t") for l in lines)])
    print(json.dumps(out))


if __name__ == "__main__":
    _main()
