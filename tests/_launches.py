"""Which kernels a call launches, in a process without a GPU: the library on the stand-in runtime of launch_recorder.c, in a
process of its own.  Tensors are addresses that nothing follows."""
import ctypes
import json
import os
import re
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
START, STOP = 71, 72  # event handles of the timer


def _serve(recorder):
    """Reads calls from stdin, one list of dicts, and writes [status, lines] of each."""
    rec = ctypes.CDLL(recorder, mode=ctypes.RTLD_GLOBAL)  # before the library: its imports are found here
    rec.recorder_text.restype = ctypes.c_char_p
    sys.path.insert(0, ROOT)
    from paper_1909_09577_amd import binding as nm
    L = nm.lib()
    at = {n: i + 1 << 40 for i, n in enumerate(("x", "w", "scale", "shift", "res", "y", "dy", "dx", "dres", "dw", "z", "mean", "invstd", "dgamma",
                                                "dbeta", "lengths", "ws", "sx", "sw", "sg", "swt"))}
    out = []
    for c in json.load(sys.stdin):
        p = dict(at, res=None, dres=None)
        p.update({n: at[n] for n in c.get("with", [])})
        p["w"] += c.get("w_offset", 0)
        d, dt, flags, ln = c["dims"], c.get("dtype", 0), c.get("flags", 0), ["lengths"] if c.get("masked") else []
        m = "_masked" if ln else ""
        op = {"fwd": 0, "static": 0, "bwd_data": 1, "bwd_weight": 2, "bwd": 3, "bn_fwd": 4, "bn_bwd": 5}.get(c["call"])
        if op is not None:
            size = c.get("ws_bytes", L.nm_conv1d_workspace_bytes(op, *d, dt, flags))
        tail = lambda: (flags, dt, p["ws"], size, None)
        calls = {
            "fwd": lambda: getattr(L, "nm_conv1d_block_fwd" + m)(*d, *(p[n] for n in ln + ["x", "w", "scale", "shift", "res", "y"]), *tail()),
            "static": lambda: L.nm_conv1d_block_fwd_static(*d, *(p[n] for n in ("x", "w", "scale", "shift", "res", "y")), flags, dt, None),
            "bwd_data": lambda: getattr(L, "nm_conv1d_bwd_data" + m)(*d, *(p[n] for n in ln + ["dy", "y", "scale", "w", "dx", "dres"]), *tail()),
            "bwd_weight": lambda: getattr(L, "nm_conv1d_bwd_weight" + m)(*d, *(p[n] for n in ln + ["x", "dy", "y", "scale", "dw"]), *tail()),
            "bwd": lambda: getattr(L, "nm_conv1d_bwd" + m)(*d, *(p[n] for n in ln + ["x", "dy", "y", "scale", "w", "dx", "dres", "dw"]), *tail()),
            "bn_fwd": lambda: L.nm_conv1d_bn_fwd(*d, *(p[n] for n in ("x", "w", "scale", "shift")), 1e-3,
                                                 *(p[n] for n in ("res", "z", "y", "mean", "invstd")), *tail()),
            "bn_bwd": lambda: L.nm_conv1d_bn_bwd(*d, *(p[n] for n in ("x", "w", "scale", "z", "y", "mean", "invstd", "dy", "dx", "dres", "dw", "dgamma",
                                                                      "dbeta")), *tail()),
            "fp8_fwd": lambda: L.nm_conv1d_block_fwd_fp8(*d, *(p[n] for n in ("x", "sx", "w", "sw", "scale", "shift", "res", "y")), flags, p["ws"],
                                                         L.nm_conv1d_fp8_workspace_bytes(*d), None),
            "fp8_bwd": lambda: L.nm_conv1d_bwd_fp8(*d, *(p[n] for n in ("x", "sx", "dy", "y", "sg", "w", "scale", "swt", "dx", "dres", "dw")), flags,
                                                   p["ws"], L.nm_conv1d_fp8_bwd_workspace_bytes(*d), None),
            "decoder": lambda: L.nm_decoder_logsoftmax_fwd(*d, *(p[n] for n in ("x", "w", "shift", "y")), flags, dt, None),
        }
        rec.recorder_reset(c.get("refuse", 0))
        if "timer" in c:
            L.nm_conv1d_time_next_kernel_of(START, STOP, c["timer"])
        status = calls[c["call"]]()
        out.append([status, rec.recorder_text().decode().splitlines()])
    json.dump(out, sys.stdout)


def run(calls, instances=False):
    """[(status, [(kind, kernel or event handle, grid), ...]), ...]; kind: launch, refused, event.  instances: kernels with their template
    arguments, ("f32_conv_kernel", 1, 0, 11, 1)."""
    with tempfile.TemporaryDirectory() as tmp:
        rec = os.path.join(tmp, "librecorder.so")
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", rec, os.path.join(ROOT, "tests", "launch_recorder.c")], check=True)
        r = subprocess.run([sys.executable, os.path.abspath(__file__), rec], input=json.dumps(calls), capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    res = []
    for status, lines in json.loads(r.stdout):
        seq = []
        for l in lines:
            kind, name, *grid = l.rsplit(" ", 4) if l.count(" ") == 4 else l.split(" ")
            k = re.search(r"\d([a-z][a-z0-9_]*_kernel)(?:I((?:L[ib]\d+E)+)E)?", name)
            what = k.group(1) if k else name
            if k and instances:
                what = (what, *map(int, re.findall(r"L[ib](\d+)E", k.group(2) or "")))
            seq.append((kind, int(name) if kind == "event" else what, tuple(map(int, grid))))
        res.append((status, seq))
    return res


if __name__ == "__main__":
    _serve(sys.argv[1])
