"""Which kernels the library launches for a convolution call, found without a GPU: the built library, in a process of its own,
on launch_recorder.c in the place of the HIP runtime.

`python launches.py` reads one JSON list of [call, N, H, W, C, K, R, stride, pad, zero padding] a line ("bwd_weight_batched": and
workgroups, a batched call of one layer; "layer_step": and bytes of workspace), channel pitches rounded up to 8, and writes one list of launches for each, a status and the number of launches for a refused "layer_step"; `of_calls` does that from a test."""
import ctypes as C
import json
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


class Launch(C.Structure):
    _fields_ = [("kernel", C.c_char * 192), ("grid", C.c_uint32 * 3), ("block", C.c_uint32), ("lds", C.c_uint32)]


def _template(mangled):
    """Name and template arguments of a mangled kernel name: integers and truth values in the order they are declared."""
    m = re.match(r"_ZN2pt\d+(k_[a-z0-9_]+?)(?:I((?:L[a-z]\w+?E)+)E|E)", mangled)
    return [m.group(1)] + [int(v) for v in re.findall(r"L[a-z](\d+)E", m.group(2) or "")] if m else [mangled]


def _main():
    rec = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)
    rec.launch_at.restype = C.POINTER(Launch)
    sys.path.insert(0, ROOT)
    from paper_1901_09290_amd import binding as B
    at = 1 << 20   # (an aligned address: nothing is read)
    for line in sys.stdin:
        call, N, H, W, Ch, K, R, stride, pad, zero, *more = json.loads(line)
        p8 = lambda n: (n + 7) // 8 * 8
        d = B.conv_desc(N, H, W, Ch, K, R, R, stride, pad, p8(Ch), p8(K), p8(Ch), B.CONV_PAD_ZERO if zero else 0)
        rec.forget()
        if call == "fwd":
            B.conv_fwd_at(d, at, at, at, (None, 0), None)
        elif call == "fwd_stats":
            assert B.lib().pt_conv_fwd_stats(C.byref(d), at, at, at, at, 1 << 40, None) == 0
        elif call == "bwd_data":
            B.conv_bwd_data_crsk_at(d, at, at, at, None)
        elif call in ("fwd_batched", "bwd_data_batched"):
            one, fn = (C.c_void_p * 1)(at), B.lib().pt_conv_fwd_batched if call == "fwd_batched" else B.lib().pt_conv_bwd_data_crsk_batched
            assert fn((B.ConvDesc * 1)(d), one, one, one, 1, None) == 0
        elif call == "bwd_weight_batched":
            jobs = (B.LayerWgrad * 1)(B.LayerWgrad(d, at, at, at, None, None, None, 0, 0))
            size = C.c_size_t()
            assert B.lib().pt_conv_bwd_weight_batched_workspace_bytes(jobs, 1, more[0], C.byref(size)) == 0
            assert B.lib().pt_conv_bwd_weight_batched(jobs, 1, 0.0, more[0], at, size.value, None) == 0
        elif call == "layer_step":
            rc = B.lib().pt_conv_layer_step(C.byref(d), at, at, at, at, at, at, 1e-3, 3, at, at, at, at, more[0], None)
            if rc:
                print(json.dumps([rc, rec.recorded()]), flush=True)
                continue
        else:
            ws = B.conv_bwd_weight_workspace_bytes(d)
            assert B.lib().pt_conv_bwd_weight(C.byref(d), at, at, at, at, ws, None) == 0
        got = [rec.launch_at(i).contents for i in range(rec.recorded())]
        print(json.dumps([dict(kernel=_template(g.kernel.decode()), grid=list(g.grid), lds=g.lds) for g in got]), flush=True)


def of_calls(calls, so):
    """[call, N, H, W, C, K, R, stride, pad, zero] each -> the launches of each; so: the built recorder."""
    r = subprocess.run([sys.executable, os.path.abspath(__file__), so], input="\n".join(json.dumps(c) for c in calls), text=True,
                       capture_output=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    return [json.loads(l) for l in r.stdout.splitlines()]


if __name__ == "__main__":
    _main()
