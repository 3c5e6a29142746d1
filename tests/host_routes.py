"""What a call would launch, without a GPU: the library's host side built with a runtime that launches nothing (host_routes.hip)."""
import ctypes
import os
import re
import subprocess

from paper_2604_27124_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
P = 1 << 20                                                            # an aligned address that nothing looks behind


class Launch(ctypes.Structure):
    _fields_ = ([("kernel", ctypes.c_char * 128)] + [(n, ctypes.c_int) for n in
                ("grid", "block", "lds", "B", "N", "N_str", "in_order", "groups")] +
                [(n, ctypes.c_void_p) for n in ("q", "part", "plan", "flags")])

    @property
    def name(self):
        """namespace and kernel, with the pass where it is a template argument: pair.sigattn_pair<0>"""
        m = re.match(r"_ZN7sigattn(?:\d+(onepass|pair|half128))?\d+(sigattn_\w+?)(?:ILi(\d+)E.*|E\w*|v?RK?\w*)?$", self.kernel.decode())
        space, kernel, mode = m.groups() if m else (None, self.kernel.decode(), None)
        return (space + "." if space else "") + kernel + (f"<{mode}>" if mode else "")


class Routes:
    def __init__(self, folder):
        obj, lib = str(folder / "routes.o"), str(folder / "routes.so")
        flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-O3")]
        subprocess.run([B.hipcc(), *flags, "--offload-host-only", "-I", os.path.join(ROOT, "include"), "-I", B.CSRC, "-c", "-o", obj,
                        os.path.join(HERE, "host_routes.hip")], check=True, capture_output=True)
        device = re.findall(r"__hip_fatbin\w*", subprocess.run(["nm", "-u", obj], check=True, capture_output=True, text=True).stdout)
        subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", *[f"-Wl,--defsym={d}=0" for d in device], "-o", lib, obj], check=True, capture_output=True)
        self.lib = ctypes.CDLL(lib)
        self.lib.sigmoid_attn_bwd_onepass_workspace_bytes.restype = ctypes.c_size_t

    def _run(self, fn, *args):
        out = (Launch * 4096)()
        self.lib.routes_take(out, 0)
        rc = fn(*[ctypes.c_void_p(a) if a is None or isinstance(a, int) and a >= P else a for a in args])
        n = self.lib.routes_take(out, len(out))
        return rc, list(out[:n])

    def _ok(self, fn, *args):
        rc, out = self._run(fn, *args)
        assert rc == 0, rc
        return out

    def fwd(self, B, Lq, Lk, H, d):
        return self._ok(self.lib.sigmoid_attn_cross_fwd, *[P] * 7, ctypes.c_float(0.125), B, Lq, Lk, H, d, None)

    def cross_bwd(self, B, Lq, Lk, H, d):
        return self._ok(self.lib.sigmoid_attn_cross_bwd, *[P] * 10, ctypes.c_float(0.125), B, Lq, Lk, H, d, None)

    def bwd(self, B, N, H, d, workspace=True):
        need = self.lib.sigmoid_attn_bwd_onepass_workspace_bytes(B, N, H, d) if workspace else 0
        return self._ok(self.lib.sigmoid_attn_bwd, *[P] * 9, ctypes.c_float(0.125), B, N, H, d, 2 * P if need else None, ctypes.c_size_t(need), None)

    def half(self, which, B, N, H, d):
        n = 8 if which == "dkdv" else 7
        return self._ok(getattr(self.lib, "sigmoid_attn_bwd_" + which), *[P] * n, ctypes.c_float(0.125), B, N, H, d, None)
